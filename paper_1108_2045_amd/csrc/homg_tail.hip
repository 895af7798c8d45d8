// homg_tail.hip -- the parts of a cycle that one workgroup runs alone: the
// leading coarse levels of the schedule (the coarse tail) and, on grids of
// side up to tail_max_side (2D 65, 3D 17), whole solves.
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
//  * 2D: the coarser levels keep one node per lane in registers, rows of 32,
//    16 or 8 lanes (sides 33, 17 and up to 9; the last lane of a row is the
//    boundary, so DPP shifts give the x neighbours).  Sides 33 and 17 exchange
//    rows through LDS with a barrier per iteration; sides up to 9 are one
//    wave's, rows by lane shuffles, no barrier and no LDS.  The code is
//    written out per side (33, 17, 9, 5, 3), with sides, offsets and spacings
//    known at compile time: as a loop over levels each began with scalar
//    loads and taken branches, 600 of its 1700 clocks.  The first restriction
//    is formed from the finest level's registers.
//    (Four nodes per lane on the coarser levels too were slower: one wave's
//    instruction issue.)
//  * 3D: the coarser levels have at most 7^3 interior nodes, one per lane, its
//    value, right-hand side and position in registers, neighbours through
//    LDS; sides 5 and 3 run in the first wave alone.  Written out per side too.
// Node formulas, summation orders and rounding points are those of the
// multi-workgroup kernels, so every form gives the same bits.
#include <type_traits>

#include "homg_device.h"
#include "homg_internal.h"

namespace homg {

namespace {

constexpr int TAIL_NT = 1024;

template <typename T>
struct TailArgs {
  int it[BATCH_MAX_LEVELS];  // iterations of level ms + k
  int nms, nlev;          // side of the finest level, number of levels
  double hl2;             // h^2 of the finest level
  double w;               // omega / 2d, or omega with a variable coefficient
  int x_off, a_off, t_off, s_off;  // byte offsets in LDS: exchange, coarser levels' factors, FP64 coarsest level, sums
  const double* faces;    // variable coefficient: the levels' factors (launch_faces), or null
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

// Relaxation of a variable-coefficient node from its face coefficients and
// w / their sum, kept over a level's iterations (relax_var's operations, so
// the same bits).
template <typename C>
struct VarNode {
  C xm, xp, ym, yp, ws;
  __device__ __forceinline__ C relax(C c, C vxm, C vxp, C vym, C vyp, C r, C hl2) const {
    const C flux = fmac(xm, c - vxm, xp * (c - vxp)) + fmac(ym, c - vym, yp * (c - vyp));
    return fmac(ws, fmac(hl2, r, -flux), c);
  }
};

// The coarser levels' arrays in LDS (offsets in elements): R, P and Q of every
// side below the largest, largest first; in 3D after R of the finest level.
// Sides and offsets are compile-time, one instance of the code per side.
template <int D, int S>
constexpr int LEV_OFF = LEV_OFF<D, 2 * S - 1> + 3 * (D == 2 ? 1 : 2 * S - 1) * (2 * S - 1) * (2 * S - 1);
template <>
constexpr int LEV_OFF<2, 33> = 1024;  // after an exchange row per wave
template <>
constexpr int LEV_OFF<3, 9> = 17 * 17 * 17;
template <int D>
constexpr int LEV_END = LEV_OFF<D, 3> + 3 * (D == 2 ? 9 : 27);

// The starting values of rows y0 .. y0 + 3 (y0 odd) of column x of a 2D level
// from the coarser level's pair (pitch = side nh): its lattice nodes take cur,
// the others the interpolant of prv.  Positions off the grid are clamped
// (their values are dropped by the caller).
template <typename T, typename C = typename Tr<T>::C>
__device__ __forceinline__ void hand_over_2d(const C* prv, const C* cur, int nh, int x, int y0, C (&v)[4]) {
  const int xi = min(x >> 1, nh - 2), j0 = y0 >> 1;
  const C tx = C(x & 1) * C(0.5);
  C xr[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const C* p = prv + min(j0 + d, nh - 1) * nh + xi;
    xr[d] = lerp(p[0], p[1], tx);
  }
  const C l1 = cur[min(j0 + 1, nh - 1) * nh + xi], l3 = cur[min(j0 + 2, nh - 1) * nh + xi];
  const bool even = !(x & 1);
  v[0] = rnd<T>(lerp(xr[0], xr[1], C(0.5)));
  v[1] = even ? l1 : rnd<T>(lerp(xr[1], xr[2], C(0)));
  v[2] = rnd<T>(lerp(xr[1], xr[2], C(0.5)));
  v[3] = even ? l3 : rnd<T>(lerp(xr[2], xr[3], C(0)));
}

// 2D coarser levels: lanes per row of a level of side S.
template <int S>
constexpr int ROW_W = S > 17 ? 32 : S > 9 ? 16 : 8;

// A 2D level of side S, one node per lane, rows of W lanes (lane W - 1 of a
// row holds x = W, the boundary or beyond: 0).  W = 8: the first wave alone.
// W = 16, 32: the first four or all waves hold rows, every wave of the
// workgroup calls it (barriers); X: two exchange buffers of W + 1 rows.  V:
// the arithmetic (FP64 for the coarsest level of reduced-precision cycles,
// whose iterates are not rounded).  hi: the next coarser level's arrays (side
// (S + 1) / 2, ith iterations), unread if zero.  Leaves the final pair, rounded
// to T, where its parity puts it (x_it in Q if it is odd), interior nodes only.
template <typename T, typename V, bool VAR, int S>
__device__ __forceinline__ void row_level(const V* R, typename Tr<T>::C* me, int it, V w, bool zero,
                                          const typename Tr<T>::C* hi, int ith, const double* fac, V* X) {
  using C = typename Tr<T>::C;
  constexpr bool EXACT = sizeof(V) != sizeof(C);  // FP64 iterates in a reduced-precision cycle
  constexpr int W = ROW_W<S>, BUF = (W + 1) * W, H = (S + 1) / 2;
  constexpr double h = 1.0 / double(S - 1);
  const V hl2 = V(h * h);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const bool on = wv < W * W / 64;
  const int x = 1 + (lane & (W - 1)), y = 1 + (W == 8 ? 0 : wv * (64 / W)) + lane / W;
  const bool in = on && x <= S - 2 && y <= S - 2;
  const int i = min(y, S - 2) * S + min(x, S - 2);
  V v = V(0), pv = V(0), cw = V(0), ce = V(0), cs = V(0), cn = V(0), ws = V(0), r = V(0);
  V* const mine = X + y * W + (x - 1);
  if (on) {  // (whole waves)
    r = R[i];
    if constexpr (VAR) {
      cw = V(fac[i]);
      ce = V(fac[i + 1]);
      cs = V(fac[S * S + i]);
      cn = V(fac[S * S + i + S]);
      ws = V(fac[2 * S * S + i]);
    }
    if constexpr (!EXACT && S > 3) {
      if (!zero) {
        const C* prv = hi + ((ith & 1) ? H * H : 2 * H * H);
        const C* cur = hi + ((ith & 1) ? 2 * H * H : H * H);
        const int c0 = min(y >> 1, H - 2) * H + min(x >> 1, H - 2);
        const C p00 = prv[c0], p01 = prv[c0 + 1], p10 = prv[c0 + H], p11 = prv[c0 + H + 1], lat = cur[c0];
        const C tx = C(x & 1) * C(0.5), ty = C(y & 1) * C(0.5);
        const C t = rnd<T>(lerp(lerp(p00, p01, tx), lerp(p10, p11, tx), ty));
        v = in ? (((x | y) & 1) ? t : lat) : V(0);
      }
    }
    if (W > 8 && y == 1) mine[-W] = mine[BUF - W] = V(0);  // row 0 of both buffers
  }
  auto step = [&](int buf) {
    V ym, yp;
    if constexpr (W == 8) {
      const V dn = __shfl_up(v, 8, 64), up = __shfl_down(v, 8, 64);
      ym = lane < 8 ? V(0) : dn;
      yp = lane < 56 ? up : V(0);
    } else {
      if (on) mine[buf * BUF] = v;
      __syncthreads();
      if (!on) return;
      ym = mine[buf * BUF - W];
      yp = mine[buf * BUF + (y < W ? W : 0)];  // (row W is the boundary's)
    }
    const V xm = lane_prev(v), xp = lane_next(v);
    V nv;
    if constexpr (VAR) {
      const V flux = fmac(cw, v - xm, ce * (v - xp)) + fmac(cs, v - ym, cn * (v - yp));
      nv = fmac(ws, fmac(hl2, r, -flux), v);
    } else {
      nv = relax_const<V>(v, (xm + xp) + (ym + yp), r, w, hl2, V(4));
    }
    pv = v;
    if constexpr (EXACT)
      v = in ? nv : V(0);
    else
      v = in ? rnd<T>(nv) : V(0);
  };
  int t = 0;
  for (; t + 2 <= it; t += 2) {  // a taken branch costs as much as four FP64 operations
    step(1);
    step(0);
  }
  if (t < it) step(1);
  if (in) {
    C* oc = me + ((it & 1) ? 2 * S * S : S * S);
    C* op = me + ((it & 1) ? S * S : 2 * S * S);
    oc[i] = EXACT ? rnd<T>(C(v)) : C(v);
    op[i] = EXACT ? rnd<T>(C(pv)) : C(pv);
  }
}

// Full weighting of side 2 S - 1 (F) onto the 2D level of side S in the same
// rows of lanes (as k_restrict_2d: rows, then their sum).
template <typename T, typename V, int S>
__device__ __forceinline__ void row_restrict(const typename Tr<T>::C* F, V* R) {
  constexpr int W = ROW_W<S>, NF = 2 * S - 1;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  if (wv >= W * W / 64) return;
  const int x = 1 + (lane & (W - 1)), y = 1 + (W == 8 ? 0 : wv * (64 / W)) + lane / W;
  if (x > S - 2 || y > S - 2) return;
  const typename Tr<T>::C* p = F + 2 * y * NF + 2 * x;
  auto rs = [&](int o) { return fmac(V(2), V(p[o]), V(p[o - 1]) + V(p[o + 1])); };
  const V top = rs(-NF), mid = rs(0), bot = rs(NF);
  const V v = fmac(V(2), mid, top + bot) * V(0.0625);
  R[y * S + x] = sizeof(V) != sizeof(typename Tr<T>::C) ? v : V(rnd<T>(typename Tr<T>::C(v)));
}

// The interior node of a 3D level of side S that the lane holds (x, y, z from 1).
template <int S>
__device__ __forceinline__ bool box_node(int& I, int& J, int& K) {
  constexpr int NI = S - 2;
  const bool on = int(threadIdx.x) < NI * NI * NI;
  const int i = on ? int(threadIdx.x) : 0;
  K = 1 + i / (NI * NI);
  J = 1 + i / NI % NI;
  I = 1 + i % NI;
  return on;
}

// Full weighting of side 2 S - 1 (F) onto the 3D level of side S, one node per
// lane (as k_restrict_3d: rows, planes, then their sum).
template <typename T, typename V, int S>
__device__ __forceinline__ void box_restrict(const typename Tr<T>::C* F, V* R) {
  constexpr int NF = 2 * S - 1, FPL = NF * NF;
  int I, J, K;
  if (!box_node<S>(I, J, K)) return;
  const typename Tr<T>::C* p = F + 2 * K * FPL + 2 * J * NF + 2 * I;
  auto rs = [&](int o) { return fmac(V(2), V(p[o]), V(p[o - 1]) + V(p[o + 1])); };
  auto ps = [&](int o) { return fmac(V(2), rs(o), rs(o - NF) + rs(o + NF)); };
  const V top = ps(-FPL), mid = ps(0), bot = ps(FPL);
  const V v = fmac(V(2), mid, top + bot) * V(0.015625);
  R[(K * S + J) * S + I] = sizeof(V) != sizeof(typename Tr<T>::C) ? v : V(rnd<T>(typename Tr<T>::C(v)));
}

// A 3D level of side S, one node per lane, its neighbours through LDS: the
// hand-over from the next coarser level's arrays (hi: side (S + 1) / 2, ith
// iterations; 0 if zero) and its iterations.  X holds R, then the two iterates
// V of the FP64 coarsest level (EXACT) or the level's own P, Q; me is the
// level's arrays.  The final pair ends in P and Q where its parity puts it.
template <typename T, typename V, int S, typename Sync>
__device__ __forceinline__ void box_level(V* X, typename Tr<T>::C* me, int it, V w, bool zero,
                                          const typename Tr<T>::C* hi, int ith, Sync&& sync) {
  using C = typename Tr<T>::C;
  constexpr bool EXACT = sizeof(V) != sizeof(C);
  constexpr int PL = S * S, N = S * S * S, H = (S + 1) / 2, HN = H * H * H;
  constexpr double h = 1.0 / double(S - 1);
  const V hl2 = V(h * h);
  int I, J, K;
  const bool on = box_node<S>(I, J, K);
  const int i = (K * S + J) * S + I;
  V* const xa = X + N;
  V* const xb = X + 2 * N;
  const V rv = X[i];
  V c = V(0), prev = V(0);
  if constexpr (!EXACT && S > 3) {
    if (!zero) {
      // lattice nodes of the coarser level take its x_it, the others the
      // interpolant of its x_{it-1}
      const C* cur = hi + ((ith & 1) ? 2 : 1) * HN;
      const C* p = hi + ((ith & 1) ? 1 : 2) * HN;
      const int c0 = ((K >> 1) * H + (J >> 1)) * H + (I >> 1);
      const C tx = C(I & 1) * C(0.5), ty = C(J & 1) * C(0.5), tz = C(K & 1) * C(0.5);
      const C lat = cur[c0];
      p += c0;
      const C* p2 = p + H * H;
      const C top = lerp(lerp(p[0], p[1], tx), lerp(p[H], p[H + 1], tx), ty);
      const C bot = lerp(lerp(p2[0], p2[1], tx), lerp(p2[H], p2[H + 1], tx), ty);
      c = ((I | J | K) & 1) ? rnd<T>(lerp(top, bot, tz)) : lat;
    }
  }
  if (on) xa[i] = c;
  sync();
  auto step = [&](const V* src, V* dst) {
    prev = c;
    if (on) {
      const V q = ((src[i - 1] + src[i + 1]) + (src[i - S] + src[i + S])) + (src[i - PL] + src[i + PL]);
      c = relax_const<V>(c, q, rv, w, hl2, V(6));
      if constexpr (!EXACT) c = rnd<T>(c);
      dst[i] = c;
    }
    sync();
  };
  int t = 0;
  for (; t + 2 <= it; t += 2) {
    step(xa, xb);
    step(xb, xa);
  }
  if (t < it) step(xa, xb);
  if constexpr (EXACT) {
    if (on) {
      me[((it & 1) ? 1 : 2) * N + i] = rnd<T>(C(prev));
      me[((it & 1) ? 2 : 1) * N + i] = rnd<T>(C(c));
    }
    sync();
  }
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
  const int n = q.nms, nlev = q.nlev;
  const int S1 = (n + 1) / 2, Stop = ((n - 1) >> (nlev - 1)) + 1;  // sides of the next level and the coarsest
  const TailNodes<D> tn(n);
  C* base = reinterpret_cast<C*>(smem);
  C* R0 = base;  // 3D: level ms's right-hand side, then R, P, Q of every coarser level
  C* E0 = base;  // 2D: an exchange row per wave, then the coarser levels' arrays
  double* A0 = reinterpret_cast<double*>(smem + q.a_off);  // VAR: the coarser levels' factors
  double* top64 = reinterpret_cast<double*>(smem + q.t_off);
  double* sums = reinterpret_cast<double*>(smem + q.s_off);
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
  // VAR: the factors (launch_faces) of the lane's nodes -- west of each (the
  // east ones are the next lane's), south of each and north of the last, w /
  // sum -- to registers, the coarser levels' to LDS.  Formed here, with some twenty
  // divisions a lane in every launch, whole solves took 371 us at 65^2 (336
  // now) and 220 at 33^2 (207), the tail 18.6 (17.9).
  double fx[4], fy[5];
  C ws[4];
  if (VAR) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const double* p = q.faces + min(tn.y0 + k, n - 1) * n + xc;
      fy[k] = p[n * n];
      if (k < 4) {
        fx[k] = p[0];
        ws[k] = C(p[2 * n * n]);
      }
    }
    const double* next = q.faces + 3 * n * n;
    int cnt = 0;
    for (int k = 1; k < nlev; ++k) cnt += 3 * (((n - 1) >> k) + 1) * (((n - 1) >> k) + 1);
    for (int i = threadIdx.x; i < cnt; i += TAIL_NT) A0[i] = next[i];
  }
  // the coarser levels' arrays start at 0 (their boundary nodes stay so)
  for (int i = LEV_OFF<D, (D == 2 ? 33 : 9)> + int(threadIdx.x); i < LEV_END<D>; i += TAIL_NT) base[i] = C(0);
  if (SOLVE && threadIdx.x < 128) sums[threadIdx.x] = 0.0;
  if (TOP64)
    for (int i = threadIdx.x; i < 3 * tail_count<D>(Stop); i += TAIL_NT) top64[i] = 0.0;
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
  // waves whose nodes all lie off the grid only take part in the barriers
  const bool wave_on = D == 2 ? 4 * tn.wv + 1 <= n - 2 : tn.wv + 1 <= n - 2;
  const bool wave_put = (D == 2 ? 4 * tn.wv : tn.wv) <= n - 2;  // (the boundary's values too)
  // iterations of the level of a side, read once
  constexpr int NSIDE = D == 2 ? 5 : 3;  // sides 3, 5, 9 (17, 33)
  int its[NSIDE];
#pragma unroll
  for (int j = 0, S = 3; j < NSIDE; ++j, S = 2 * S - 1) {
    int k = 1;
    while (((n - 1) >> k) + 1 > S) ++k;
    its[j] = S < n && S >= Stop ? q.it[k] : 0;
  }
  const int it0 = q.it[0];
  const C hl20 = C(q.hl2);
  // 2D: the restriction of level ms's right-hand side, from registers (as
  // k_restrict_2d: row sums, then their sum): a lane's rows y0 + 1 and y0 + 3
  // are coarse rows; the row above the second comes from the next wave
  auto row_sum = [&](auto two, C c) {
    using V = decltype(two);
    return fmac(two, V(c), V(lane_prev(c)) + V(lane_next(c)));
  };
  auto put_first = [&](const C (&rr)[4]) {
    if (wave_on) E0[tn.wv * 64 + tn.lane] = rr[0];
  };
  auto get_first = [&](const C (&rr)[4], auto two, auto* R) {
    if (!wave_on) return;
    using V = decltype(two);
    const int S = S1;
    const C up = 4 * tn.wv + 5 <= n - 2 ? E0[(tn.wv + 1) * 64 + tn.lane] : C(0);
    const V s0 = row_sum(two, rr[0]), s1 = row_sum(two, rr[1]), s2 = row_sum(two, rr[2]), s3 = row_sum(two, rr[3]),
            s4 = row_sum(two, up);
    const V a = fmac(two, s1, s0 + s2) * V(0.0625), b = fmac(two, s3, s2 + s4) * V(0.0625);
    auto put = [&](int J, V v) {
      if (!(tn.x & 1) && tn.x <= n - 3 && J <= S - 2)
        R[J * S + (tn.x >> 1)] = sizeof(V) != sizeof(C) ? v : V(rnd<T>(C(v)));
    };
    put(2 * tn.wv + 1, a);
    put(2 * tn.wv + 2, b);
  };

  for (int cyc = SOLVE ? run.c0 : 0;; ++cyc) {
    if constexpr (SOLVE) {
      // ---- residual and its norm
      const TailExchange<D, double> ex{reinterpret_cast<double*>(smem + q.x_off)};
      if (wave_put) ex.put(tn, uv);
      __syncthreads();
      if (wave_on) {
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
      if (D == 3) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (tn.in(k)) R0[o0 + (tn.y0 + k) * n] = r[k];
      }
      }  // wave_on
      if (D == 2) put_first(r);
      __syncthreads();
      if (tn.wv == 0) {
        int cnt;
        const bool first = cyc == 0;
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
        if (D == 3 && tn.in(k)) R0[o0 + (tn.y0 + k) * n] = r[k];
      }
      if (D == 2) put_first(r);
      __syncthreads();
    }

    // ---- the coarser levels: sides below n, not below the schedule's coarsest
    double* const X64 = reinterpret_cast<double*>(smem + q.x_off);
    C* const X = reinterpret_cast<C*>(smem + q.x_off);
    auto has = [&](int S) { return S <= S1 && S >= Stop; };
    auto down = [&](auto sz) {  // the restriction onto side S
      constexpr int S = decltype(sz)::value;
      const bool t64 = TOP64 && S == Stop;
      if constexpr (D == 2) {
        const C* F = base + LEV_OFF<2, (S < 33 ? 2 * S - 1 : 33)>;
        if (S == S1) {
          if (t64)
            get_first(r, 2.0, top64);
          else
            get_first(r, C(2), base + LEV_OFF<2, S>);
        } else if constexpr (S < 33) {
          if (t64)
            row_restrict<T, double, S>(F, top64);
          else
            row_restrict<T, C, S>(F, base + LEV_OFF<2, S>);
        }
      } else {
        const C* F = S == S1 ? base : base + LEV_OFF<3, (S < 9 ? 2 * S - 1 : 9)>;
        if (t64)
          box_restrict<T, double, S>(F, top64);
        else
          box_restrict<T, C, S>(F, base + LEV_OFF<3, S>);
      }
    };
    auto up = [&](auto sz, int it, int ith, auto&& sync) {  // side S's hand-over and iterations
      constexpr int S = decltype(sz)::value;
      const bool t64 = TOP64 && S == Stop;
      C* const me = base + LEV_OFF<D, S>;
      const C* hi = base + LEV_OFF<D, (S > 3 ? (S + 1) / 2 : 3)>;
      if constexpr (D == 2) {
        const int o1 = S1 == 33 ? LEV_OFF<2, 33> : S1 == 17 ? LEV_OFF<2, 17> : S1 == 9 ? LEV_OFF<2, 9>
                       : S1 == 5 ? LEV_OFF<2, 5> : LEV_OFF<2, 3>;
        const double* fac = A0 + (LEV_OFF<2, S> - o1);  // (three arrays per level too)
        if (t64)
          row_level<T, double, VAR, S>(top64, me, it, q.w, true, hi, 0, fac, X64);
        else
          row_level<T, C, VAR, S>(me, me, it, w, S == Stop, hi, ith, fac, X);
      } else {
        if (t64)
          box_level<T, double, S>(top64, me, it, q.w, true, hi, 0, sync);
        else
          box_level<T, C, S>(me, me, it, w, S == Stop, hi, ith, sync);
      }
    };
    using S33 = std::integral_constant<int, 33>;
    using S17 = std::integral_constant<int, 17>;
    using S9 = std::integral_constant<int, 9>;
    using S5 = std::integral_constant<int, 5>;
    using S3 = std::integral_constant<int, 3>;
    auto one_wave = [] { wave_sync(); };
    auto all_waves = [] { __syncthreads(); };
    if (nlev > 1) {
      if constexpr (D == 2) {
        if (has(33)) {
          down(S33());
          __syncthreads();
        }
        if (has(17)) {
          down(S17());
          __syncthreads();
        }
        // the first restriction takes every wave's registers; the rest of the
        // levels of one wave is that wave's
        if (S1 <= 9) {
          if (S1 == 9)
            down(S9());
          else if (S1 == 5)
            down(S5());
          else
            down(S3());
          __syncthreads();
        }
        if (Stop <= 9) {
          if (tn.wv == 0) {
            if (has(9)) {
              if (S1 > 9) down(S9());
              wave_sync();
            }
            if (has(5)) {
              if (S1 > 5) down(S5());
              wave_sync();
            }
            if (has(3)) {
              if (S1 > 3) down(S3());
              wave_sync();
              up(S3(), its[0], 0, one_wave);
              wave_sync();
            }
            if (has(5)) {
              up(S5(), its[1], its[0], one_wave);
              wave_sync();
            }
            if (has(9)) up(S9(), its[2], its[1], one_wave);
          }
          __syncthreads();
        }
        if (has(17)) {
          up(S17(), its[NSIDE > 3 ? 3 : 0], its[2], all_waves);
          __syncthreads();
        }
        if (has(33)) {
          up(S33(), its[NSIDE > 3 ? 4 : 0], its[NSIDE > 3 ? 3 : 0], all_waves);
          __syncthreads();
        }
      } else {
        if (has(9)) {
          down(S9());
          __syncthreads();
        }
        if (Stop <= 5) {  // sides 5 and 3: the first wave's
          if (tn.wv == 0) {
            if (has(5)) {
              down(S5());
              wave_sync();
            }
            if (has(3)) {
              down(S3());
              wave_sync();
              up(S3(), its[0], 0, one_wave);
            }
            if (has(5)) up(S5(), its[1], its[0], one_wave);
          }
          __syncthreads();
        }
        if (has(9)) up(S9(), its[2], its[1], all_waves);
      }
    }

    // ---- the finest level, in registers
    C v[4] = {C(0), C(0), C(0), C(0)}, pv[4];
    if (nlev > 1 && wave_on) {
      const int nh = S1, ph = nh * nh;
      const int ith = q.it[1];
      const C* base1;
      if (D == 2)
        base1 = base + (nh == 33 ? LEV_OFF<2, 33> : nh == 17 ? LEV_OFF<2, 17> : nh == 9 ? LEV_OFF<2, 9>
                        : nh == 5 ? LEV_OFF<2, 5> : LEV_OFF<2, 3>);
      else
        base1 = base + (nh == 9 ? LEV_OFF<3, 9> : nh == 5 ? LEV_OFF<3, 5> : LEV_OFF<3, 3>);
      const C* cur = base1 + ((ith & 1) ? 2 : 1) * tail_count<D>(nh);
      const C* prv = base1 + ((ith & 1) ? 1 : 2) * tail_count<D>(nh);
      if constexpr (D == 2) {
        hand_over_2d<T>(prv, cur, nh, tn.x, tn.y0, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = tn.in(k) ? v[k] : C(0);
      } else {
        // rows y0 .. y0 + 3 (y0 odd) lie in coarser rows j0, j0 + 1, j0 + 1,
        // j0 + 2; indices of lanes off the grid are clamped, their values dropped
        const int xi = min(tn.x >> 1, nh - 2), j0 = tn.y0 >> 1, zk = min(tn.z >> 1, nh - 2);
        const C tx = C(tn.x & 1) * C(0.5), tz = C(tn.z & 1) * C(0.5);
        C yi[2][4];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          C xr[4];
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            const C* p = prv + (zk + e) * ph + min(j0 + d, nh - 1) * nh + xi;
            xr[d] = lerp(p[0], p[1], tx);
          }
          yi[e][0] = lerp(xr[0], xr[1], C(0.5));
          yi[e][1] = lerp(xr[1], xr[2], C(0));
          yi[e][2] = lerp(xr[1], xr[2], C(0.5));
          yi[e][3] = lerp(xr[2], xr[3], C(0));
        }
        const bool even = !(tn.x & 1) && !(tn.z & 1);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          C t = rnd<T>(lerp(yi[0][k], yi[1][k], tz));
          if (k & 1) {  // an even row: a lattice node of level 1 where x and z are even
            const C lat = cur[zk * ph + min(j0 + 1 + (k >> 1), nh - 1) * nh + xi];
            t = even ? lat : t;
          }
          v[k] = tn.in(k) ? t : C(0);
        }
      }
    }
    const C hl2 = hl20;
    const int it = it0;
    constexpr int XN = D == 2 ? 2 * 16 * 64 : 4 * TAIL_NT;
    C last[4];
    for (int t = 1; t <= it; ++t) {
      // two exchange buffers in turn: one barrier per iteration
      const TailExchange<D, C> ex{reinterpret_cast<C*>(smem + q.x_off) + (t & 1) * XN};
      if (wave_put) ex.put(tn, v);
      __syncthreads();
      if (!wave_on) continue;
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
  const size_t cnt = d == 2 ? LEV_END<2> : LEV_END<3>;
  auto take = [&](size_t& at, size_t bytes) {
    at = (at + 15) & ~size_t(15);
    const size_t o = at;
    at += bytes;
    return int(o);
  };
  size_t at = cnt * cs;
  const size_t xn = d == 2 ? 2 * 16 * 64 : 4 * size_t(TAIL_NT);  // one exchange buffer
  const bool t64 = top64 && prec != PREC_F64;
  const size_t rows64 = d == 2 && t64 ? 2 * 33 * 32 * 8 : 0;  // an FP64 level's exchange
  L.x_off = take(at, std::max({2 * xn * cs, solve ? xn * 8 : size_t(0), rows64}));
  size_t facs = 0;
  for (int k = 1; k < nlev; ++k) facs += 3 * nodes(k);
  L.a_off = take(at, var ? facs * 8 : 0);
  L.t_off = take(at, t64 ? 3 * nodes(nlev - 1) * 8 : 0);
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
TailArgs<T> make_args(const TailLds& L, int d, int nms, int nlev, const int* its, double omega, const double* faces,
                      DevState* st, double* hist) {
  TailArgs<T> q{};
  for (int k = 0; k < nlev; ++k) q.it[k] = its[k];
  q.nms = nms;
  q.nlev = nlev;
  q.hl2 = (1.0 / double(nms - 1)) * (1.0 / double(nms - 1));
  q.w = faces ? omega : omega / double(2 * d);
  q.x_off = L.x_off;
  q.a_off = L.a_off;
  q.t_off = L.t_off;
  q.s_off = L.s_off;
  q.faces = faces;
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
static hipError_t tail_t(int prec, int d, int nms, int nlev, const int* its, double omega, const double* faces,
                         const void* rms, const Lay& rl, void* sprev, void* scur, const Lay& sl,
                         bool top64, DevState* st, double* hist, const double* partials, int count, int cycle,
                         hipStream_t s) {
  const TailLds L = tail_lds(prec, d, nms, nlev, top64, faces != nullptr, false);
  TailArgs<T> q = make_args<T>(L, d, nms, nlev, its, omega, faces, st, hist);
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
  return launch_d<T, false>(d, top64, faces != nullptr, q, run, L.bytes, s);
}

hipError_t launch_coarse_tail(int prec, int d, int nms, int nlev, const int* its, double omega, const double* faces,
                              const void* rms, const Lay& rl, void* sprev, void* scur, const Lay& sl,
                              bool top64, DevState* st, double* hist, const double* partials, int count, int cycle,
                              hipStream_t s) {
  if (!tail_ok(d, nms, nlev) || nlev < 2 || (faces && d != 2) || !rms || !sprev || !scur || sl.side != nms ||
      rl.side != nms)
    return hipErrorInvalidValue;
#define TAIL_CASE(T)                                                                                           \
  return tail_t<T>(prec, d, nms, nlev, its, omega, faces, rms, rl, sprev, scur, sl, top64, st, hist, partials, \
                   count, cycle, s)
  switch (prec) {
    case PREC_F64: TAIL_CASE(double);
    case PREC_F32: TAIL_CASE(float);
    default: TAIL_CASE(bf16);
  }
#undef TAIL_CASE
}

template <typename T>
static hipError_t small_solve_t(int prec, int d, int n, int nlev, const int* its, double omega, const double* faces,
                                const double* f, double* u, bool top64, bool rr, int c0, int c1,
                                double tol, int stop, DevState* st, double* hist, DevState* hst, double* hhist,
                                hipStream_t s) {
  const TailLds L = tail_lds(prec, d, n, nlev, top64, faces != nullptr, true);
  TailArgs<T> q = make_args<T>(L, d, n, nlev, its, omega, faces, st, hist);
  const double h = 1.0 / double(n - 1);
  q.inv_h2 = 1.0 / (h * h);
  q.rr = rr;
  q.hst = hst;
  q.hhist = hhist;
  return launch_d<T, true>(d, top64, faces != nullptr, q, TailRun{-1, f, u, tol, c0, c1, stop}, L.bytes, s);
}

hipError_t launch_small_solve(int prec, int d, int n, int nlev, const int* its, double omega, const double* faces,
                              const double* f, double* u, bool top64, bool rr, int c0, int c1,
                              double tol, int stop, DevState* st, double* hist, DevState* hst, double* hhist,
                              hipStream_t s) {
  if (!tail_ok(d, n, nlev) || (faces && d != 2) || !f || !u || c1 < c0 || (top64 && nlev < 2))
    return hipErrorInvalidValue;
#define SMALL_CASE(T)                                                                                            \
  return small_solve_t<T>(prec, d, n, nlev, its, omega, faces, f, u, top64, rr, c0, c1, tol, stop, st, hist, hst, \
                          hhist, s)
  switch (prec) {
    case PREC_F64: SMALL_CASE(double);
    case PREC_F32: SMALL_CASE(float);
    default: SMALL_CASE(bf16);
  }
#undef SMALL_CASE
}

// ---- variable coefficient: the factors of the levels one workgroup may run

struct FaceLevel {
  const double* a;  // nodal coefficient at (0, 0)
  int64_t ap;
  int side, off, wide;  // wide: w / sum in FP64 whatever the storage type
};
struct FaceArgs {
  FaceLevel lv[8];
  double* out;
  double w;
  int f32;  // w / sum in FP32
};
__global__ __launch_bounds__(256) void k_faces(FaceArgs q) {
  const FaceLevel& L = q.lv[blockIdx.y];
  const int S = L.side, i = blockIdx.x * 256 + threadIdx.x;
  if (i >= S * S) return;
  const int y = i / S, x = i % S;
  const double* p = L.a + y * L.ap + x;
  const double c = p[0];
  // (face coefficients are symmetric to the bit: each is formed once)
  const double w = x > 0 ? harm(c, p[-1]) : 0.0, s = y > 0 ? harm(c, p[-L.ap]) : 0.0;
  double d = 0.0;
  if (x > 0 && y > 0 && x < S - 1 && y < S - 1) {
    const double e = harm(c, p[1]), n = harm(c, p[L.ap]);
    d = q.f32 && !L.wide ? double(float(q.w) / ((float(w) + float(e)) + (float(s) + float(n))))
                         : q.w / ((w + e) + (s + n));
  }
  double* o = q.out + L.off + i;
  o[0] = w;
  o[S * S] = s;
  o[2 * S * S] = d;
}

hipError_t launch_faces(int prec, int levels, const double* const* a, const Lay* al, bool wide_last, double omega,
                        double* out, hipStream_t s) {
  if (levels < 1 || levels > 8) return hipErrorInvalidValue;
  FaceArgs q{};
  int off = 0;
  for (int k = 0; k < levels; ++k) {
    if (al[k].side > tail_max_side(2)) return hipErrorInvalidValue;
    q.lv[k] = FaceLevel{a[k] + al[k].off, al[k].pitch, al[k].side, off, wide_last && k == levels - 1};
    off += 3 * al[k].side * al[k].side;
  }
  q.out = out;
  q.w = omega;
  q.f32 = prec != PREC_F64;
  HOMG_LAUNCH(k_faces, dim3(unsigned(al[0].side * al[0].side + 255) / 256, unsigned(levels)), dim3(256), s, q);
}

size_t batch_tail_bytes(int prec) {
  return prec == PREC_F64 ? sizeof(TailArgs<double>) : (prec == PREC_F32 ? sizeof(TailArgs<float>) : sizeof(TailArgs<bf16>));
}

template <typename T>
static void batch_tail_t(int prec, void* dst, int n, int nlev, const int* its, double omega, const void* r, int64_t rp,
                         void* sprev, void* scur, int64_t sp, bool top64, DevState* st, double* hist,
                         const double* partials, int count) {
  TailArgs<T> q = make_args<T>(tail_lds(prec, 2, n, nlev, top64, false, false), 2, n, nlev, its, omega, nullptr,
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
  TailArgs<T> q = make_args<T>(tail_lds(prec, 2, n, nlev, top64, false, true), 2, n, nlev, its, omega, nullptr,
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
