// homg_tail.hip -- the parts of a cycle that one workgroup runs alone: the
// leading coarse levels of the schedule (the coarse tail) and, on grids of
// side up to TAIL_MAX_2D / TAIL_MAX_3D, whole solves.
//
// What bounds them is latency, not bandwidth or arithmetic: a few thousand
// nodes at most, some 35 iterations, restrictions and hand-overs one after
// the other, each ending in a barrier.  So the split is chosen for short
// phases:
//  * the finest level (up to 63^2 or 15^3 interior nodes) stays in registers,
//    four nodes per lane.  2D: a wave is a row of 64 columns by 4 rows, x
//    neighbours by DPP wave shifts, and only its first and last row go through
//    LDS (2 writes and 2 reads per lane and iteration; with every node in LDS
//    it was 5 reads and a write per node, bound by LDS throughput: 0.96 us an
//    iteration at 65^2).  3D: a wave is one plane of 16 columns by 4 groups of
//    4 rows, x neighbours by DPP row shifts, y neighbours from the lane's own
//    rows and the lanes 16 away, and the planes above and below through LDS;
//  * the coarser levels have at most 31^2 or 7^3 interior nodes: one per lane,
//    its value, right-hand side and position kept in registers, neighbours
//    through LDS;
//  * levels of at most 64 interior nodes (sides 9, 5, 3; in 3D 5, 3), their
//    restrictions and hand-overs are run by the first wave alone without
//    barriers: a third of all phases.
// Node formulas, summation orders and rounding points are those of the
// multi-workgroup kernels, so every form gives the same bits.
#include "homg_device.h"
#include "homg_internal.h"

namespace homg {

namespace {

constexpr int TAIL_NT = 1024;

// Per-level constants, worked out on the host (the reciprocals and h^2 are
// the correctly rounded values the device division would give), so that no
// level starts with a division.
struct TailLevel {
  int it;        // iterations of level ms + k
  int off;       // element offset of the level's R, P, Q arrays in LDS (k >= 1)
  float inv_ni;  // 1 / (nk - 2): splits the level's interior nodes
  int pad;
  double hl2;    // h^2 = (1 / (nk - 1))^2
};

template <typename T>
struct TailArgs {
  TailLevel lv[BATCH_MAX_LEVELS];
  int nms, nlev;          // side of the finest level, number of levels
  double w;               // omega / 2d, or omega with a variable coefficient
  int x_off, a_off, t_off, s_off;  // byte offsets in LDS: exchange, coefficient, FP64 coarsest level, sums
  const double* a;        // nodal coefficient of the finest level (node 0), or null
  int64_t ap;
  DevState* st;
  double* hist;
  // coarse tail
  const T* r;             // level ms's right-hand side
  T* sprev;               // its final x_{it-1} and x_it
  T* scur;
  int64_t rp, rpl, sp, spl;
  const double* partials; // the previous residual's sums
  int count;
  // whole solves
  int rr;                 // order of the norms' sums (see below)
  int prob, pad;
  double inv_h2;
  DevState* hst;          // pinned mirrors, or null
  double* hhist;
};

// What changes from launch to launch.
struct TailRun {
  int cycle;        // coarse tail: the cycle whose norm is not reduced yet, or -1
  const double* f;  // whole solves: dense, side nms
  double* u;
  double tol;
  int c0, c1, stop; // cycles c0 .. c1
};

template <int D>
__host__ __device__ constexpr int tail_count(int nk) { return D == 2 ? nk * nk : nk * nk * nk; }

// Orders the LDS accesses of one wave (its LDS instructions execute in
// order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// x neighbours within rows of 16 lanes (DPP row shifts); the row's end lane
// keeps `edge`.
__device__ __forceinline__ int row16_prev(int edge, int v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x111, 0xf, 0xf, false);
}
__device__ __forceinline__ int row16_next(int edge, int v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x101, 0xf, 0xf, false);
}
template <typename F>
__device__ __forceinline__ double by_halves(double edge, double v, F&& f) {
  const long long b = __double_as_longlong(v), e = __double_as_longlong(edge);
  const unsigned lo = unsigned(f(int(e), int(b))), hi = unsigned(f(int(e >> 32), int(b >> 32)));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename F>
__device__ __forceinline__ float by_halves(float edge, float v, F&& f) {
  return __int_as_float(f(__float_as_int(edge), __float_as_int(v)));
}
template <int D, typename V>
__device__ __forceinline__ V x_prev(V edge, V v) {
  if (D == 2) return lane_prev_or(edge, v);
  return by_halves(edge, v, [](int e, int b) { return row16_prev(e, b); });
}
template <int D, typename V>
__device__ __forceinline__ V x_next(V edge, V v) {
  if (D == 2) return lane_next_or(edge, v);
  return by_halves(edge, v, [](int e, int b) { return row16_next(e, b); });
}

// The lane's four nodes of the finest level: column x, rows y0 .. y0 + 3,
// plane z (3D).
template <int D>
struct TailNodes {
  int lane, wv, x, y0, z, n;
  __device__ __forceinline__ explicit TailNodes(int n_) : n(n_) {
    lane = threadIdx.x & 63;
    wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    x = 1 + (D == 2 ? lane : lane & 15);
    y0 = 1 + 4 * (D == 2 ? wv : lane >> 4);
    z = D == 2 ? 0 : 1 + wv;
  }
  __device__ __forceinline__ bool in(int k) const {
    return x <= n - 2 && y0 + k <= n - 2 && (D == 2 || z <= n - 2);
  }
};

// y (and 3D z) neighbours of the lane's four values through the exchange
// area X.  put() before a barrier, get() after it.  Values outside the
// lane's reach (y or z = 0) come from lo / zlo; the other end's boundary
// nodes are values of lanes of their own.
template <int D, typename V>
struct TailExchange {
  V* X;
  __device__ __forceinline__ void put(const TailNodes<D>& t, const V (&v)[4]) const {
    if (D == 2) {
      X[(2 * t.wv) * 64 + t.lane] = v[0];
      X[(2 * t.wv + 1) * 64 + t.lane] = v[3];
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) X[k * TAIL_NT + int(threadIdx.x)] = v[k];
    }
  }
  __device__ __forceinline__ void get_y(const TailNodes<D>& t, const V (&v)[4], V lo, V& ym, V& yp) const {
    if (D == 2) {
      ym = t.wv > 0 ? X[(2 * t.wv - 1) * 64 + t.lane] : lo;
      yp = t.wv < 15 ? X[(2 * t.wv + 2) * 64 + t.lane] : V(0);
    } else {
      const int g = t.lane >> 4;
      ym = g > 0 ? X[3 * TAIL_NT + int(threadIdx.x) - 16] : lo;
      yp = g < 3 ? X[int(threadIdx.x) + 16] : V(0);
    }
  }
  __device__ __forceinline__ void get_z(const TailNodes<D>& t, const V (&zlo)[4], V (&zm)[4], V (&zp)[4]) const {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      zm[k] = t.wv > 0 ? X[k * TAIL_NT + int(threadIdx.x) - 64] : zlo[k];
      zp[k] = t.wv < 15 ? X[k * TAIL_NT + int(threadIdx.x) + 64] : V(0);
    }
  }
};

// Relaxation factors of a variable-coefficient node: relax_var's face
// coefficients and w / sum, kept over a level's iterations (the same
// operations, so the same bits).
template <typename C>
struct VarNode {
  C xm, xp, ym, yp, ws;
  __device__ __forceinline__ void set(double c, double axm, double axp, double aym, double ayp, C w) {
    xm = C(harm(c, axm));
    xp = C(harm(c, axp));
    ym = C(harm(c, aym));
    yp = C(harm(c, ayp));
    ws = w / ((xm + xp) + (ym + yp));
  }
  __device__ __forceinline__ C relax(C c, C vxm, C vxp, C vym, C vyp, C r, C hl2) const {
    const C flux = fmac(xm, c - vxm, xp * (c - vxp)) + fmac(ym, c - vym, yp * (c - vyp));
    return fmac(ws, fmac(hl2, r, -flux), c);
  }
};

// One interior node of a coarser level, its neighbours in LDS (pitch nk,
// plane nk^2).
template <int D, bool VAR, typename C>
__device__ __forceinline__ C tail_relax(const C* src, int i, int nk, int pl, C c, C r, C w, C hl2, const VarNode<C>& vn) {
  if (VAR) return vn.relax(c, src[i - 1], src[i + 1], src[i - nk], src[i + nk], r, hl2);
  const C q = (src[i - 1] + src[i + 1]) + (src[i - nk] + src[i + nk]);
  if (D == 2) return relax_const<C>(c, q, r, w, hl2, C(4));
  return relax_const<C>(c, q + (src[i - pl] + src[i + pl]), r, w, hl2, C(6));
}

// ---- one workgroup -----------------------------------------------------
// SOLVE = false, the coarse tail: restricts r of level ms to the coarser
// levels, runs the levels from the coarsest to ms and leaves level ms's
// x_{it-1} and x_it for the next level's first pass (or the hand-over
// kernel).  It also reduces the previous residual's norm and decides
// whether the solve is done (k_finalize's arithmetic): as a launch of its
// own that took 4.3 us a cycle.
// SOLVE = true: cycles c0 .. c1 of a whole solve, u and f in registers.
// The norms are summed in the order of the residual kernels and k_finalize
// -- rr: per 62 columns and 2 rows, as k_residual_restrict_2d's waves;
// otherwise per 4 rows (2D) or plane (3D), as k_residual_2d / _3d -- so the
// history does not depend on the form either.
// TOP64 (reduced precision): the coarsest level in FP64 -- its right-hand
// side restricted in FP64 from the stored values of the level below, its
// iterates FP64 -- and only its final pair rounded to the storage type.
template <typename T, int D, bool VAR, bool TOP64, bool SOLVE>
__device__ __forceinline__ void tail_block(const TailArgs<T>& q, const TailRun& run) {
  using C = typename Tr<T>::C;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_done;
  const int n = q.nms, nlev = q.nlev, ktop = nlev - 1;
  const TailNodes<D> tn(n);
  C* base = reinterpret_cast<C*>(smem);
  C* R0 = base;  // level ms's right-hand side; then R, P, Q of every coarser level
  double* A0 = reinterpret_cast<double*>(smem + q.a_off);
  double* top64 = reinterpret_cast<double*>(smem + q.t_off);
  double* sums = reinterpret_cast<double*>(smem + q.s_off);
  auto side = [&](int k) { return ((n - 1) >> k) + 1; };
  auto lvl = [&](int k, int which) {
    return k == 0 ? R0 : base + q.lv[k].off + which * tail_count<D>(side(k));
  };
  const C w = C(q.w);

  DevState st = *q.st;
  if (!SOLVE && st.done) return;
  if (SOLVE && run.c0 > 0 && st.done) return;

  // loads first: the level's right-hand side, or f and u with the boundary
  // values next to the lane's nodes
  C r[4];
  double uv[4], fv[4], ue[4], ulo = 0.0, uzlo[4];
  const int xc = min(tn.x, n - 1), zc = min(tn.z, n - 1);
  if (!SOLVE) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      r[k] = ld(q.r + int64_t(zc) * q.rpl + int64_t(min(tn.y0 + k, n - 1)) * q.rp + xc);
  } else {
    const int64_t pl = int64_t(zc) * n * n * (D == 3);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t row = pl + int64_t(min(tn.y0 + k, n - 1)) * n;
      uv[k] = run.u[row + xc];
      fv[k] = run.f[row + xc];
      ue[k] = run.u[row];  // x = 0, used by the first lane of a row
      uzlo[k] = D == 3 ? run.u[int64_t(min(tn.y0 + k, n - 1)) * n + xc] : 0.0;  // z = 0
    }
    ulo = run.u[pl + xc];  // y = 0
  }
  if (VAR)
    for (int i = threadIdx.x; i < n * n; i += TAIL_NT) A0[i] = q.a[int64_t(i / n) * q.ap + i % n];
  // the coarser levels' arrays start at 0 (their boundary nodes stay so)
  if (nlev > 1) {
    const int end = q.lv[ktop].off + 3 * tail_count<D>(side(ktop));
    for (int i = q.lv[1].off + int(threadIdx.x); i < end; i += TAIL_NT) base[i] = C(0);
  }
  if (TOP64)
    for (int i = threadIdx.x; i < 3 * tail_count<D>(side(ktop)); i += TAIL_NT) top64[i] = 0.0;
  if (!SOLVE && run.cycle >= 0) {
    const double s = fin_sum(q.partials, q.count);
    if (threadIdx.x == 0) {
      q.hist[run.cycle] = fin_update(st, s, run.cycle);
      *q.st = st;
      s_done = st.done;
    }
    __syncthreads();
    if (s_done) return;
  }
  const int o0 = (D == 3 ? zc * n * n : 0) + xc;  // the lane's column in R0
  // VAR: the lane's face coefficients -- west of each node (the east ones
  // are the next lane's: harm is symmetric to the bit) and south of each,
  // then north of the last -- and w / their sum
  double fx[4], fy[5];
  C ws[4];
  if (VAR) {
    __syncthreads();
    const double* col = A0 + xc;
    double a = col[(min(tn.y0, n - 1) - 1) * n];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const double b = col[min(tn.y0 + k, n - 1) * n];
      fy[k] = harm(b, a);
      if (k < 4) fx[k] = harm(b, col[min(tn.y0 + k, n - 1) * n - 1]);
      a = b;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) ws[k] = w / ((C(fx[k]) + C(x_next<D>(1.0, fx[k]))) + (C(fy[k]) + C(fy[k + 1])));
  }

  for (int cyc = SOLVE ? run.c0 : 0;; ++cyc) {
    if constexpr (SOLVE) {
      // ---- residual and its norm
      const TailExchange<D, double> ex{reinterpret_cast<double*>(smem + q.x_off)};
      ex.put(tn, uv);
      __syncthreads();
      double ym0, yp3, zm[4], zp[4];
      ex.get_y(tn, uv, ulo, ym0, yp3);
      if (D == 3) ex.get_z(tn, uzlo, zm, zp);
      double sr[2] = {0.0, 0.0}, sf[2] = {0.0, 0.0};
      const bool first = cyc == 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double c = uv[k];
        const double xm = x_prev<D>(ue[k], c), xp = x_next<D>(0.0, c);
        const double ym = k == 0 ? ym0 : uv[k - 1], yp = k == 3 ? yp3 : uv[k + 1];
        double au;
        if (VAR)
          au = fmac(fx[k], c - xm, x_next<D>(0.0, fx[k]) * (c - xp)) + fmac(fy[k], c - ym, fy[k + 1] * (c - yp));
        else if (D == 2)
          au = fmac(4.0, c, -((xm + xp) + (ym + yp)));
        else
          au = fmac(6.0, c, -(((xm + xp) + (ym + yp)) + (zm[k] + zp[k])));
        const double rv = fmac(-q.inv_h2, au, fv[k]);
        const bool in = tn.in(k);
        r[k] = in ? rnd<T>(C(rv)) : C(0);
        if (in) {
          if (k >= 2 && q.rr) {  // bands of two rows, or of four
            sr[1] = fmac(rv, rv, sr[1]);
            if (first) sf[1] = fmac(fv[k], fv[k], sf[1]);
          } else {
            sr[0] = fmac(rv, rv, sr[0]);
            if (first) sf[0] = fmac(fv[k], fv[k], sf[0]);
          }
        }
      }
      // partial sums of this wave into sums[] (f^2: sums + 64)
      auto partial = [&](const double (&s)[2], double* out) {
        if (D == 3) {
          double v = s[0];
#pragma unroll
          for (int o = 8; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
          // the four row groups of a plane, one after the other
          double t = 0.0;
#pragma unroll
          for (int g = 0; g < 4; ++g) t += __shfl(v, 16 * g, 64);
          if (tn.lane == 0) out[tn.wv] = t;
        } else if (q.rr) {
          const int gx = (n - 2 + 61) / 62;
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const double last = __shfl(s[b], 62, 64);  // column 63: the second 62-column group
            double v = lane_prev(s[b]);
            if (tn.lane == 63) v = 0.0;
            v = wave_sum(v);
            if (tn.lane == 0 && 4 * tn.wv + 2 * b + 1 <= n - 2) {
              out[(2 * tn.wv + b) * gx] = v;
              if (gx == 2) out[(2 * tn.wv + b) * gx + 1] = last;
            }
          }
        } else {
          const double v = wave_sum(s[0]);
          if (tn.lane == 0) out[tn.wv] = v;
        }
      };
      partial(sr, sums);
      if (first) partial(sf, sums + 64);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (tn.in(k)) R0[o0 + (tn.y0 + k) * n] = r[k];
      __syncthreads();
      if (tn.wv == 0) {
        int cnt;
        auto total = [&](double* p) {
          double v;
          if (D == 2 && !q.rr) {  // four waves (16 rows) per partial sum
            v = 0.0;
            if (tn.lane < 4) {
#pragma unroll
              for (int g = 0; g < 4; ++g) v += p[4 * tn.lane + g];
            }
          } else {
            v = tn.lane < cnt ? p[tn.lane] : 0.0;
          }
          return wave_sum(v);
        };
        cnt = D == 3 ? n - 2 : ((n - 2 + 61) / 62) * ((n - 2 + 1) / 2);
        const double s = total(sums);
        if (first) {
          const double fn = sqrt(total(sums + 64));
          st.done = 0;
          st.cycles = -1;
          st.stop_on_tol = run.stop;
          st.pad = 0;
          st.fnorm = fn > 0.0 ? fn : 1.0;
          st.tol = run.tol;
        }
        if (tn.lane == 0) {
          const double rel = fin_update(st, s, cyc);
          q.hist[cyc] = rel;
          if (q.hhist) q.hhist[cyc] = rel;
          s_done = st.done;
        }
      }
      __syncthreads();
      if (s_done || cyc >= run.c1) break;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        r[k] = tn.in(k) ? r[k] : C(0);
        if (tn.in(k)) R0[o0 + (tn.y0 + k) * n] = r[k];
      }
      __syncthreads();
    }

    // ---- restriction pyramid (full weighting, as k_restrict_*), one node per lane
    auto restrict_to = [&](int k) {
      const int nf = side(k - 1), nc = side(k), ni = nc - 2, cnt = tail_count<D>(ni);
      const int i = threadIdx.x;
      if (i >= cnt) return;
      const C* F = lvl(k - 1, 0);
      int I, J, K;
      tail_split<D>(i, ni, q.lv[k].inv_ni, I, J, K);
      ++I, ++J, K += D == 3;
      const int o = (D == 3 ? K * nc * nc : 0) + J * nc + I;
      const int fp = nf, fpl = nf * nf;
      const int c = (D == 3 ? 2 * K * fpl : 0) + 2 * J * fp + 2 * I;
      auto weigh = [&](auto two, auto scale) {  // as k_restrict_*: rows, then planes
        using V = decltype(two);
        auto rs = [&](int p) { return fmac(two, V(F[p]), V(F[p - 1]) + V(F[p + 1])); };
        if (D == 2) {
          const V top = rs(c - fp), mid = rs(c), bot = rs(c + fp);
          return fmac(two, mid, top + bot) * scale;
        }
        auto ps = [&](int p) { return fmac(two, rs(p), rs(p - fp) + rs(p + fp)); };
        const V top = ps(c - fpl), mid = ps(c), bot = ps(c + fpl);
        return fmac(two, mid, top + bot) * scale;
      };
      if (TOP64 && k == ktop)
        top64[o] = weigh(2.0, D == 2 ? 0.0625 : 0.015625);
      else
        lvl(k, 0)[o] = rnd<T>(weigh(C(2), D == 2 ? C(0.0625) : C(0.015625)));
    };

    // ---- a coarser level: hand-over from the level above (or 0) and its
    // iterations, one node per lane; sync() between phases
    auto run_coarse = [&](int k, auto&& sync) {
      const int nk = side(k), pl = nk * nk, ni = nk - 2, cnt = tail_count<D>(ni);
      const bool on = int(threadIdx.x) < cnt;
      int I, J, K;
      tail_split<D>(on ? int(threadIdx.x) : 0, ni, q.lv[k].inv_ni, I, J, K);
      ++I, ++J, K += D == 3;
      const int i = (D == 3 ? K * pl : 0) + J * nk + I;
      C* xa = lvl(k, 1);
      C* xb = lvl(k, 2);
      const int it = q.lv[k].it;
      const int as = 1 << k;
      const double* ap = A0 + J * as * n + I * as;
      if (TOP64 && k == ktop) {
        double* ya = top64 + tail_count<D>(nk);
        double* yb = ya + tail_count<D>(nk);
        const double rv = top64[i], hl2d = q.lv[k].hl2;
        VarNode<double> vn;
        if (VAR) vn.set(ap[0], ap[-as], ap[as], ap[-as * n], ap[as * n], q.w);
        double c = 0.0, prev = 0.0;
        if (on) ya[i] = 0.0;
        sync();
        for (int t = 1; t <= it; ++t) {
          const double* src = (t & 1) ? ya : yb;
          double* dst = (t & 1) ? yb : ya;
          prev = c;
          if (on) {
            c = tail_relax<D, VAR>(src, i, nk, pl, c, rv, q.w, hl2d, vn);
            dst[i] = c;
          }
          sync();
        }
        if (on) {  // the final pair where run_coarse leaves every level's: by the parity of it
          ((it & 1) ? xa : xb)[i] = rnd<T>(C(prev));
          ((it & 1) ? xb : xa)[i] = rnd<T>(C(c));
        }
        sync();
        return;
      }
      const C hl2 = C(q.lv[k].hl2);
      VarNode<C> vn;
      if (VAR) vn.set(ap[0], ap[-as], ap[as], ap[-as * n], ap[as * n], w);
      const C rv = lvl(k, 0)[i];
      C c = C(0);
      if (k < ktop) {
        // lattice nodes of level k + 1 take its x_it, the others the
        // interpolant of its x_{it-1}
        const int nh = side(k + 1), ph = nh * nh, ith = q.lv[k + 1].it;
        const C* cur = lvl(k + 1, (ith & 1) ? 2 : 1);
        const C* prv = lvl(k + 1, (ith & 1) ? 1 : 2);
        const int c0 = (D == 3 ? (K >> 1) * ph : 0) + (J >> 1) * nh + (I >> 1);
        const C tx = C(I & 1) * C(0.5), ty = C(J & 1) * C(0.5), tz = C(K & 1) * C(0.5);
        const C lat = cur[c0];
        C v;
        if (D == 2) {
          const C top = lerp(prv[c0], prv[c0 + 1], tx), bot = lerp(prv[c0 + nh], prv[c0 + nh + 1], tx);
          v = lerp(top, bot, ty);
        } else {
          const C* p = prv + c0;
          const C* p2 = p + ph;
          const C top = lerp(lerp(p[0], p[1], tx), lerp(p[nh], p[nh + 1], tx), ty);
          const C bot = lerp(lerp(p2[0], p2[1], tx), lerp(p2[nh], p2[nh + 1], tx), ty);
          v = lerp(top, bot, tz);
        }
        c = (!(I & 1) && !(J & 1) && !(K & 1)) ? lat : rnd<T>(v);
      }
      if (on) xa[i] = c;
      sync();
      for (int t = 1; t <= it; ++t) {
        const C* src = (t & 1) ? xa : xb;
        C* dst = (t & 1) ? xb : xa;
        if (on) {
          c = rnd<T>(tail_relax<D, VAR>(src, i, nk, pl, c, rv, w, hl2, vn));
          dst[i] = c;
        }
        sync();
      }
    };

    // levels ks .. ktop have at most 64 interior nodes: the first wave's
    int ks = 1;
    while (ks < nlev && tail_count<D>(side(ks) - 2) > 64) ++ks;
    for (int k = 1; k < ks; ++k) {
      restrict_to(k);
      __syncthreads();
    }
    if (ks < nlev) {
      if (tn.wv == 0) {
        for (int k = ks; k < nlev; ++k) {
          restrict_to(k);
          wave_sync();
        }
        for (int k = ktop; k >= ks; --k) run_coarse(k, [] { wave_sync(); });
      }
      __syncthreads();
    }
    for (int k = ks - 1; k >= 1; --k) run_coarse(k, [] { __syncthreads(); });

    // ---- the finest level, in registers
    C v[4] = {C(0), C(0), C(0), C(0)}, pv[4];
    if (nlev > 1) {
      const int nh = side(1), ph = nh * nh, ith = q.lv[1].it;
      const C* cur = lvl(1, (ith & 1) ? 2 : 1);
      const C* prv = lvl(1, (ith & 1) ? 1 : 2);
      // rows y0 .. y0 + 3 (y0 odd) lie in coarser rows j0, j0 + 1, j0 + 1,
      // j0 + 2; indices of lanes off the grid are clamped, their values dropped
      const int xi = min(tn.x >> 1, nh - 2), j0 = tn.y0 >> 1, zk = D == 3 ? min(tn.z >> 1, nh - 2) : 0;
      const C tx = C(tn.x & 1) * C(0.5), tz = C(tn.z & 1) * C(0.5);
      C yi[2][4];
#pragma unroll
      for (int e = 0; e < (D == 3 ? 2 : 1); ++e) {
        C xr[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const C* p = prv + (D == 3 ? (zk + e) * ph : 0) + min(j0 + d, nh - 1) * nh + xi;
          xr[d] = lerp(p[0], p[1], tx);
        }
        yi[e][0] = lerp(xr[0], xr[1], C(0.5));
        yi[e][1] = lerp(xr[1], xr[2], C(0));
        yi[e][2] = lerp(xr[1], xr[2], C(0.5));
        yi[e][3] = lerp(xr[2], xr[3], C(0));
      }
      const bool even = !(tn.x & 1) && (D == 2 || !(tn.z & 1));
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        C t = D == 3 ? lerp(yi[0][k], yi[1][k], tz) : yi[0][k];
        if (k & 1) {  // an even row: a lattice node of level 1 where x (and z) are even
          const C lat = cur[(D == 3 ? zk * ph : 0) + min(j0 + 1 + (k >> 1), nh - 1) * nh + xi];
          t = even ? lat : rnd<T>(t);
        } else {
          t = rnd<T>(t);
        }
        v[k] = tn.in(k) ? t : C(0);
      }
    }
    const C hl2 = C(q.lv[0].hl2);
    const int it = q.lv[0].it;
    constexpr int XN = D == 2 ? 2 * 16 * 64 : 4 * TAIL_NT;
    C last[4];
    for (int t = 1; t <= it; ++t) {
      // two exchange buffers in turn: one barrier per iteration
      const TailExchange<D, C> ex{reinterpret_cast<C*>(smem + q.x_off) + (t & 1) * XN};
      ex.put(tn, v);
      __syncthreads();
      C ym0, yp3, zm[4], zp[4];
      const C zero4[4] = {C(0), C(0), C(0), C(0)};
      ex.get_y(tn, v, C(0), ym0, yp3);
      if (D == 3) ex.get_z(tn, zero4, zm, zp);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const C c = v[k];
        const C xm = x_prev<D>(C(0), c), xp = x_next<D>(C(0), c);
        const C ym = k == 0 ? ym0 : v[k - 1], yp = k == 3 ? yp3 : v[k + 1];
        if (VAR)
          last[k] = VarNode<C>{C(fx[k]), C(x_next<D>(0.0, fx[k])), C(fy[k]), C(fy[k + 1]), ws[k]}.relax(c, xm, xp, ym, yp, r[k], hl2);
        else if (D == 2)
          last[k] = relax_const<C>(c, (xm + xp) + (ym + yp), r[k], w, hl2, C(4));
        else
          last[k] = relax_const<C>(c, ((xm + xp) + (ym + yp)) + (zm[k] + zp[k]), r[k], w, hl2, C(6));
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        pv[k] = v[k];
        v[k] = tn.in(k) ? rnd<T>(last[k]) : C(0);
      }
    }
    if constexpr (SOLVE) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (tn.in(k)) uv[k] += double(last[k]);  // unrounded, as the passes that add into u
      __syncthreads();  // the exchange area changes its type
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (tn.in(k)) {
          const int64_t o = int64_t(tn.z) * q.spl + int64_t(tn.y0 + k) * q.sp + tn.x;
          st_w(q.sprev + o, pv[k]);
          st_w(q.scur + o, v[k]);
        }
      break;
    }
  }
  if constexpr (SOLVE) {
    const int64_t pl = int64_t(tn.z) * n * n * (D == 3);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (tn.in(k)) run.u[pl + int64_t(tn.y0 + k) * n + tn.x] = uv[k];
    if (threadIdx.x == 0) {
      *q.st = st;
      if (q.hst) *q.hst = st;
    }
  }
}

template <typename T, int D, bool VAR, bool TOP64, bool SOLVE>
__global__ __launch_bounds__(TAIL_NT) void k_coarse_tail(TailArgs<T> q, TailRun run) {
  tail_block<T, D, VAR, TOP64, SOLVE>(q, run);
}

// One workgroup per problem of a batch.
template <typename T, bool TOP64>
__global__ __launch_bounds__(TAIL_NT) void k_batch_tail(const TailArgs<T>* __restrict__ args, int cycle) {
  tail_block<T, 2, false, TOP64, false>(args[blockIdx.x], TailRun{cycle, nullptr, nullptr, 0.0, 0, 0, 0});
}
template <typename T, bool TOP64>
__global__ __launch_bounds__(TAIL_NT) void k_batch_small(const TailArgs<T>* __restrict__ args,
                                                         const double* const* __restrict__ f,
                                                         double* const* __restrict__ u, double tol, int c0, int c1) {
  const TailArgs<T>& q = args[blockIdx.x];
  tail_block<T, 2, false, TOP64, true>(q, TailRun{-1, f[q.prob], u[q.prob], tol, c0, c1, 1});
}

// LDS layout: byte offsets of the areas behind the C arrays.
struct TailLds {
  int off[BATCH_MAX_LEVELS];
  int x_off, a_off, t_off, s_off;
  size_t bytes;
};
TailLds tail_lds(int prec, int d, int nms, int nlev, bool top64, bool var, bool solve) {
  TailLds L{};
  const size_t cs = prec == PREC_F64 ? 8 : 4;
  auto nodes = [&](int k) {
    const size_t nk = size_t((nms - 1) >> k) + 1;
    return d == 2 ? nk * nk : nk * nk * nk;
  };
  size_t cnt = nodes(0);
  for (int k = 1; k < nlev; ++k) {
    L.off[k] = int(cnt);
    cnt += 3 * nodes(k);
  }
  auto take = [&](size_t& at, size_t bytes) {
    at = (at + 15) & ~size_t(15);
    const size_t o = at;
    at += bytes;
    return int(o);
  };
  size_t at = cnt * cs;
  const size_t xn = d == 2 ? 2 * 16 * 64 : 4 * size_t(TAIL_NT);  // one exchange buffer
  L.x_off = take(at, std::max(2 * xn * cs, solve ? xn * 8 : size_t(0)));
  L.a_off = take(at, var ? nodes(0) * 8 : 0);
  L.t_off = take(at, top64 && prec != PREC_F64 ? 3 * nodes(nlev - 1) * 8 : 0);
  L.s_off = take(at, solve ? 128 * 8 : 0);
  L.bytes = at;
  return L;
}

template <typename T, int D, bool VAR, bool TOP64, bool SOLVE>
hipError_t launch_t(const TailArgs<T>& a, const TailRun& run, size_t lds, hipStream_t s) {
  hipError_t e = allow_lds(k_coarse_tail<T, D, VAR, TOP64, SOLVE>, lds);
  if (e != hipSuccess) return e;
  HOMG_LAUNCH_SMEM((k_coarse_tail<T, D, VAR, TOP64, SOLVE>), dim3(1), dim3(TAIL_NT), lds, s, a, run);
}

template <typename T, bool SOLVE>
hipError_t launch_d(int d, bool top64, bool var, const TailArgs<T>& a, const TailRun& run, size_t lds, hipStream_t s) {
  constexpr bool RED = sizeof(T) != 8;  // reduced precision: the FP64 coarsest level exists
  const bool t64 = RED && top64;
  if (d == 3)
    return t64 ? launch_t<T, 3, false, RED, SOLVE>(a, run, lds, s) : launch_t<T, 3, false, false, SOLVE>(a, run, lds, s);
  if (var)
    return t64 ? launch_t<T, 2, true, RED, SOLVE>(a, run, lds, s) : launch_t<T, 2, true, false, SOLVE>(a, run, lds, s);
  return t64 ? launch_t<T, 2, false, RED, SOLVE>(a, run, lds, s) : launch_t<T, 2, false, false, SOLVE>(a, run, lds, s);
}

template <typename T>
TailArgs<T> make_args(const TailLds& L, int d, int nms, int nlev, const int* its, double omega, const double* a,
                      const Lay& al, DevState* st, double* hist) {
  TailArgs<T> q{};
  for (int k = 0; k < nlev; ++k) {
    const int nk = ((nms - 1) >> k) + 1;
    const double h = 1.0 / double(nk - 1);
    q.lv[k] = TailLevel{its[k], L.off[k], 1.0f / float(nk - 2), 0, h * h};
  }
  q.nms = nms;
  q.nlev = nlev;
  q.w = a ? omega : omega / double(2 * d);
  q.x_off = L.x_off;
  q.a_off = L.a_off;
  q.t_off = L.t_off;
  q.s_off = L.s_off;
  q.a = a ? a + al.off : nullptr;
  q.ap = al.pitch;
  q.st = st;
  q.hist = hist;
  return q;
}

bool tail_ok(int d, int nms, int nlev) {
  return nms >= 3 && nms <= tail_max_side(d) && nlev >= 1 && nlev <= BATCH_MAX_LEVELS &&
         ((nms - 1) >> (nlev - 1)) + 1 >= 3;
}

}  // namespace

size_t coarse_tail_lds(int prec, int d, int nms, int nlev, bool top64, bool var, bool solve) {
  return tail_lds(prec, d, nms, nlev, top64, var, solve).bytes;
}

template <typename T>
static hipError_t tail_t(int prec, int d, int nms, int nlev, const int* its, double omega, const double* a,
                         const Lay& al, const void* rms, const Lay& rl, void* sprev, void* scur, const Lay& sl,
                         bool top64, DevState* st, double* hist, const double* partials, int count, int cycle,
                         hipStream_t s) {
  const TailLds L = tail_lds(prec, d, nms, nlev, top64, a != nullptr, false);
  TailArgs<T> q = make_args<T>(L, d, nms, nlev, its, omega, a, al, st, hist);
  q.r = static_cast<const T*>(rms) + rl.off;
  q.rp = rl.pitch;
  q.rpl = rl.plane;
  q.sprev = static_cast<T*>(sprev) + sl.off;
  q.scur = static_cast<T*>(scur) + sl.off;
  q.sp = sl.pitch;
  q.spl = sl.plane;
  q.partials = partials;
  q.count = count;
  const TailRun run{partials ? cycle : -1, nullptr, nullptr, 0.0, 0, 0, 0};
  return launch_d<T, false>(d, top64, a != nullptr, q, run, L.bytes, s);
}

hipError_t launch_coarse_tail(int prec, int d, int nms, int nlev, const int* its, double omega, const double* a,
                              const Lay& al, const void* rms, const Lay& rl, void* sprev, void* scur, const Lay& sl,
                              bool top64, DevState* st, double* hist, const double* partials, int count, int cycle,
                              hipStream_t s) {
  if (!tail_ok(d, nms, nlev) || nlev < 2 || (a && d != 2) || !rms || !sprev || !scur || sl.side != nms ||
      rl.side != nms || (a && al.side != nms))
    return hipErrorInvalidValue;
#define TAIL_CASE(T)                                                                                           \
  return tail_t<T>(prec, d, nms, nlev, its, omega, a, al, rms, rl, sprev, scur, sl, top64, st, hist, partials, \
                   count, cycle, s)
  switch (prec) {
    case PREC_F64: TAIL_CASE(double);
    case PREC_F32: TAIL_CASE(float);
    default: TAIL_CASE(bf16);
  }
#undef TAIL_CASE
}

template <typename T>
static hipError_t small_solve_t(int prec, int d, int n, int nlev, const int* its, double omega, const double* a,
                                const Lay& al, const double* f, double* u, bool top64, bool rr, int c0, int c1,
                                double tol, int stop, DevState* st, double* hist, DevState* hst, double* hhist,
                                hipStream_t s) {
  const TailLds L = tail_lds(prec, d, n, nlev, top64, a != nullptr, true);
  TailArgs<T> q = make_args<T>(L, d, n, nlev, its, omega, a, al, st, hist);
  const double h = 1.0 / double(n - 1);
  q.inv_h2 = 1.0 / (h * h);
  q.rr = rr;
  q.hst = hst;
  q.hhist = hhist;
  return launch_d<T, true>(d, top64, a != nullptr, q, TailRun{-1, f, u, tol, c0, c1, stop}, L.bytes, s);
}

hipError_t launch_small_solve(int prec, int d, int n, int nlev, const int* its, double omega, const double* a,
                              const Lay& al, const double* f, double* u, bool top64, bool rr, int c0, int c1,
                              double tol, int stop, DevState* st, double* hist, DevState* hst, double* hhist,
                              hipStream_t s) {
  if (!tail_ok(d, n, nlev) || (a && (d != 2 || al.side != n)) || !f || !u || c1 < c0 || (top64 && nlev < 2))
    return hipErrorInvalidValue;
#define SMALL_CASE(T)                                                                                            \
  return small_solve_t<T>(prec, d, n, nlev, its, omega, a, al, f, u, top64, rr, c0, c1, tol, stop, st, hist, hst, \
                          hhist, s)
  switch (prec) {
    case PREC_F64: SMALL_CASE(double);
    case PREC_F32: SMALL_CASE(float);
    default: SMALL_CASE(bf16);
  }
#undef SMALL_CASE
}

size_t batch_tail_bytes(int prec) {
  return prec == PREC_F64 ? sizeof(TailArgs<double>) : (prec == PREC_F32 ? sizeof(TailArgs<float>) : sizeof(TailArgs<bf16>));
}

template <typename T>
static void batch_tail_t(int prec, void* dst, int n, int nlev, const int* its, double omega, const void* r, int64_t rp,
                         void* sprev, void* scur, int64_t sp, bool top64, DevState* st, double* hist,
                         const double* partials, int count) {
  TailArgs<T> q = make_args<T>(tail_lds(prec, 2, n, nlev, top64, false, false), 2, n, nlev, its, omega, nullptr, Lay(),
                               st, hist);
  q.r = static_cast<const T*>(r);
  q.rp = rp;
  q.sprev = static_cast<T*>(sprev);
  q.scur = static_cast<T*>(scur);
  q.sp = sp;
  q.partials = partials;
  q.count = count;
  *static_cast<TailArgs<T>*>(dst) = q;
}

void batch_tail_fill(int prec, void* dst, int n, int nlev, const int* its, double omega, const void* r, int64_t rp,
                     void* sprev, void* scur, int64_t sp, bool top64, DevState* st, double* hist,
                     const double* partials, int count) {
#define TAIL_FILL(T) \
  batch_tail_t<T>(prec, dst, n, nlev, its, omega, r, rp, sprev, scur, sp, top64, st, hist, partials, count)
  switch (prec) {
    case PREC_F64: TAIL_FILL(double); break;
    case PREC_F32: TAIL_FILL(float); break;
    default: TAIL_FILL(bf16); break;
  }
#undef TAIL_FILL
}

template <typename T>
static void batch_small_t(int prec, void* dst, int n, int nlev, const int* its, double omega, bool top64, bool rr,
                          int prob, DevState* st, double* hist) {
  TailArgs<T> q = make_args<T>(tail_lds(prec, 2, n, nlev, top64, false, true), 2, n, nlev, its, omega, nullptr, Lay(),
                               st, hist);
  const double h = 1.0 / double(n - 1);
  q.inv_h2 = 1.0 / (h * h);
  q.rr = rr;
  q.prob = prob;
  *static_cast<TailArgs<T>*>(dst) = q;
}

void batch_small_fill(int prec, void* dst, int n, int nlev, const int* its, double omega, bool top64, bool rr, int prob,
                      DevState* st, double* hist) {
  switch (prec) {
    case PREC_F64: batch_small_t<double>(prec, dst, n, nlev, its, omega, top64, rr, prob, st, hist); break;
    case PREC_F32: batch_small_t<float>(prec, dst, n, nlev, its, omega, top64, rr, prob, st, hist); break;
    default: batch_small_t<bf16>(prec, dst, n, nlev, its, omega, top64, rr, prob, st, hist); break;
  }
}

template <typename T, bool TOP64>
static hipError_t batch_tails_t(const void* args, int count, size_t lds, int cycle, hipStream_t s) {
  hipError_t e = allow_lds(k_batch_tail<T, TOP64>, lds);
  if (e != hipSuccess) return e;
  HOMG_LAUNCH_SMEM((k_batch_tail<T, TOP64>), dim3(count), dim3(TAIL_NT), lds, s, static_cast<const TailArgs<T>*>(args),
                   cycle);
}

hipError_t launch_batch_tails(int prec, bool top64, const void* args, int count, size_t lds, int cycle, hipStream_t s) {
  switch (prec) {
    case PREC_F64: return batch_tails_t<double, false>(args, count, lds, cycle, s);
    case PREC_F32:
      return top64 ? batch_tails_t<float, true>(args, count, lds, cycle, s)
                   : batch_tails_t<float, false>(args, count, lds, cycle, s);
    default:
      return top64 ? batch_tails_t<bf16, true>(args, count, lds, cycle, s)
                   : batch_tails_t<bf16, false>(args, count, lds, cycle, s);
  }
}

template <typename T, bool TOP64>
static hipError_t batch_small_launch(const void* args, int count, size_t lds, const double* const* f, double* const* u,
                                     double tol, int c0, int c1, hipStream_t s) {
  hipError_t e = allow_lds(k_batch_small<T, TOP64>, lds);
  if (e != hipSuccess) return e;
  HOMG_LAUNCH_SMEM((k_batch_small<T, TOP64>), dim3(count), dim3(TAIL_NT), lds, s, static_cast<const TailArgs<T>*>(args),
                   f, u, tol, c0, c1);
}

hipError_t launch_batch_small(int prec, bool top64, const void* args, int count, size_t lds, const double* const* f,
                              double* const* u, double tol, int c0, int c1, hipStream_t s) {
  switch (prec) {
    case PREC_F64: return batch_small_launch<double, false>(args, count, lds, f, u, tol, c0, c1, s);
    case PREC_F32:
      return top64 ? batch_small_launch<float, true>(args, count, lds, f, u, tol, c0, c1, s)
                   : batch_small_launch<float, false>(args, count, lds, f, u, tol, c0, c1, s);
    default:
      return top64 ? batch_small_launch<bf16, true>(args, count, lds, f, u, tol, c0, c1, s)
                   : batch_small_launch<bf16, false>(args, count, lds, f, u, tol, c0, c1, s);
  }
}

}  // namespace homg
