// homg_learned_tiles.hip -- the learned relaxation, several iterations or
// levels per launch (2D, chained execution).
//
// What bounds it: on lattices up to 129^2 the launch and the chain of phases
// of one block; above that the phases between barriers with 16 waves on a CU:
// at 1025^2 vector issue (1290 instructions a wave for two iterations) fills 31
// of a pass's 50 us, LDS 20 and the matrix cores 11, and dropping the masks of
// blocks away from the boundary (60 instructions) left it at 50.  One launch per
// iteration with a hand-over launch per level takes 396 us a cycle at 1025^2
// (FP64, 10 levels); with these two kernels it is 231.  A workgroup keeps a 32 x 32
// block of the hidden layer and
//  * k_learned_tiles runs up to four iterations of one level on it, the block
//    shrinking by three nodes a side each, the coefficient factors of a lane's
//    nodes kept in registers, the first iterate taken from the next coarser
//    level's compact state.  Per level and cycle, four iterations, before and
//    after: 65^2 and 129^2 24 -> 13 us, 257^2 30 -> 20, 513^2 50 -> 31,
//    1025^2 124 -> 103 (and 4 us per hand-over);
//  * k_learned_tail runs the leading coarse levels of sides up to 33 (one
//    block holds the interior) with their restrictions, hand-overs and the
//    previous norm: 30 us, before 113 in 21 launches.
// Node formulas are those of the single-iteration kernel, so the bits are too.
#include <algorithm>

#include "homg_device.h"
#include "homg_learned_device.h"

namespace homg {

namespace {

constexpr int LB_NT = 1024;
constexpr int LB_H = 32;         // hidden-layer block
constexpr int LB_F = LB_H + 2;   // features
constexpr int LB_X = LB_H + 4;   // iterate and coefficient
constexpr int LB_FPL = LB_F * LB_F;

// ---- several iterations of one level ------------------------------------

template <typename T>
struct LearnedTileArgs {
  const T* xo;  // x_0, or null: 0 or the coarser level's state
  T* xn;
  T* xp;        // x_{it-1} (nullable)
  int cp, rp, ap, up;
  const T* r;
  const double* a;
  double* u;    // given: u += x_it instead of the stores
  const T* lprev;  // the coarser level's pair (lprev null: x_{it-1} = 0)
  const T* lcur;   // (null: none)
  int lp;
  int n, nb, it;
  typename Tr<T>::C hl2;
  const float* w;
  const int* done;
};

// Blocks above which 8 waves take one, two to a CU: one workgroup of 16 waves
// to a CU leaves it idle at its barriers; fewer blocks than CUs finish sooner
// with 16 waves.  Level 0's last pass with 16 and with 8 waves (FP64): 129^2 (four
// iterations, 121 blocks) 13.5 and 15.0 us, 257^2 (two, 121) 9.4 and 10.1; 513^2
// (two, 484) 18.5 and 15.5, 1025^2 67 and 49, 2049^2 241 and 165.
constexpr int LB_WIDE_BLOCKS = 256;

template <typename C>
struct LearnedTileLds {
  static constexpr int ZPL = LB_H * LB_H + 4;
  uint64_t fb[3 * LB_FPL];
  C x[LB_X * LB_X];
  union {
    float z[9 * ZPL];
    float a[LB_X * LB_X];  // until the factors are formed
  };
};

template <typename T, bool VAR, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_learned_tiles(LearnedTileArgs<T> q) {
  using C = typename Tr<T>::C;
  constexpr int ZPL = LearnedTileLds<C>::ZPL;
  constexpr int NX = (LB_X * LB_X + NT - 1) / NT, NF = (LB_FPL + NT - 1) / NT, NO = LB_H * LB_H / NT;
  extern __shared__ __align__(16) unsigned char smem[];
  LearnedTileLds<C>& L = *reinterpret_cast<LearnedTileLds<C>*>(smem);
  const int t = threadIdx.x, n = q.n;
  const int m0 = 3 * q.it - 2, own = LB_H - 2 * m0;  // owned block: hidden nodes m0 .. 31 - m0
  const unsigned lb = xcd_order(blockIdx.x, gridDim.x);
  // hidden node (j, i) is lattice node (J0 + j, I0 + i)
  const int J0 = 1 + int(lb / unsigned(q.nb)) * own - m0, I0 = 1 + int(lb % unsigned(q.nb)) * own - m0;
  auto interior = [&](int J, int I) { return unsigned(J - 1) < unsigned(n - 2) && unsigned(I - 1) < unsigned(n - 2); };

  // x_0 and a on the 36^2 region, r of the lane's feature nodes, the weights:
  // clamped loads, all in flight together
  const int done = *q.done;
  C xl[NX];
  double al[NX];
#pragma unroll
  for (int k = 0; k < NX; ++k) {
    const int p = t + k * NT;
    const int J = J0 - 2 + p / LB_X, I = I0 - 2 + p % LB_X;
    const int cj = min(max(J, 0), n - 1), ci = min(max(I, 0), n - 1);
    xl[k] = C(0);
    if (q.xo) xl[k] = ld(q.xo + cj * q.cp + ci);
    if constexpr (VAR) al[k] = q.a[cj * q.ap + ci];
  }
  C rv[NF];
  bool fin[NF];
  int fx[NF];  // the feature node's place in x
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    const int p = t + k * NT, fj = p / LB_F, fi = p % LB_F;
    const int J = J0 - 1 + fj, I = I0 - 1 + fi;
    fin[k] = p < LB_FPL && interior(J, I);
    fx[k] = p < LB_FPL ? (fj + 1) * LB_X + fi + 1 : LB_X + 1;
    rv[k] = ld(q.r + min(max(J, 1), n - 2) * q.rp + min(max(I, 1), n - 2));
  }
  const int hi = t & 31, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int I = I0 + hi;
  bool owned[NO];
  double uo[NO];
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    const int hj = (t >> 5) + k * (NT / 32);
    owned[k] = hj >= m0 && hj < LB_H - m0 && hi >= m0 && hi < LB_H - m0 && interior(J0 + hj, I);
    uo[k] = q.u ? q.u[min(max(J0 + hj, 0), n - 1) * q.up + min(max(I, 0), n - 1)] : 0.0;
  }
  const LaneConst kc = lane_const(q.w);
  if (q.lcur) {  // the coarser level's state: its nodes as they are, others interpolated
    const int nc = (n - 1) / 2 + 1;
    C c00[NX], p00[NX], p01[NX], p10[NX], p11[NX];
    const T* const pv = q.lprev ? q.lprev : q.lcur;  // (x_{it-1} = 0: loads a valid array, drops it)
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      const int p = t + k * NT;
      const int cj = min(max(J0 - 2 + p / LB_X, 0), n - 1), ci = min(max(I0 - 2 + p % LB_X, 0), n - 1);
      const int o = min(cj >> 1, nc - 2) * q.lp + min(ci >> 1, nc - 2);
      c00[k] = ld(q.lcur + o);
      p00[k] = ld(pv + o);
      p01[k] = ld(pv + o + 1);
      p10[k] = ld(pv + o + q.lp);
      p11[k] = ld(pv + o + q.lp + 1);
    }
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      const int p = t + k * NT;
      const int ci = I0 - 2 + p % LB_X, cj = J0 - 2 + p / LB_X;
      const C tx = C(ci & 1) * C(0.5), ty = C(cj & 1) * C(0.5);
      const C v = lerp(lerp(p00[k], p01[k], tx), lerp(p10[k], p11[k], tx), ty);
      xl[k] = ((ci | cj) & 1) ? (q.lprev ? rnd<T>(v) : C(0)) : c00[k];
    }
  }
#pragma unroll
  for (int k = 0; k < NX; ++k) {
    const int p = t + k * NT;
    const int J = J0 - 2 + p / LB_X, I = I0 - 2 + p % LB_X;
    if (p < LB_X * LB_X) {
      L.x[p] = interior(J, I) ? xl[k] : C(0);
      if constexpr (VAR) L.a[p] = unsigned(J) < unsigned(n) && unsigned(I) < unsigned(n) ? float(al[k]) : 1.f;
    }
  }
  if (done) return;
  __syncthreads();
  FaceFactors ff[NF];
  if constexpr (VAR) {
#pragma unroll
    for (int k = 0; k < NF; ++k)
      if (t + k * NT < LB_FPL) {
        const float* a = L.a + fx[k];
        ff[k].set(a[0], a[-1], a[1], a[-LB_X], a[LB_X]);
      }
  }

  C xv[NO], pv[NO];
  for (int s = 0; s < q.it; ++s) {
    const int lo = 3 * s;  // the block shrinks: hidden nodes lo .. 31 - lo
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const int p = t + k * NT, fj = p / LB_F;
      if (p < LB_FPL && fj >= lo && fj < LB_F - lo) {
        const C* x = L.x + fx[k];
        const C xc = x[0];
        float f0, f1, f2;
        node_feature<VAR, C>(ff[k], xc - x[-1], xc - x[1], xc - x[-LB_X], xc - x[LB_X], rv[k], q.hl2, f0, f1, f2);
        store_features<LB_FPL>(L.fb + p, fin[k] ? f0 : 0.f, fin[k] ? f1 : 0.f, fin[k] ? f2 : 0.f);
      }
    }
    __syncthreads();
    // rows of one or two groups of 16 columns (the second overlaps the first
    // and writes the same values there)
    const int width = LB_H - 2 * lo, two = width > 16;
    for (int c = wave; c < width << two; c += NT / 64) {
      const int j = lo + (c >> two), i = two && (c & 1) ? LB_H - 16 - lo : lo;
      contract16<LB_F, LB_FPL, ZPL>(L.z + j * LB_H + i, L.fb + j * LB_F + i, kc, interior(J0 + j, I0 + i + (t & 15)));
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NO; ++k) {
      const int hj = (t >> 5) + k * (NT / 32);
      if (hj > lo && hj < LB_H - 1 - lo && hi > lo && hi < LB_H - 1 - lo && interior(J0 + hj, I)) {
        C* x = L.x + (hj + 2) * LB_X + hi + 2;
        pv[k] = *x;
        xv[k] = pv[k] + C(sum_taps<LB_H, ZPL>(L.z + (hj - 1) * LB_H + hi - 1));
        if (!(q.u && s == q.it - 1)) xv[k] = rnd<T>(xv[k]);
        *x = xv[k];
      }
    }
    if (s < q.it - 1) __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    const int J = J0 + (t >> 5) + k * (NT / 32);
    if (!owned[k]) continue;
    if (q.u) {
      q.u[J * q.up + I] = uo[k] + double(xv[k]);
    } else {
      st_w(q.xn + J * q.cp + I, xv[k]);
      if (q.xp) st_w(q.xp + J * q.cp + I, pv[k]);
    }
  }
}

// ---- the leading coarse levels ------------------------------------------

constexpr int LT_P = LB_F;          // pitch of x, features and Z: lattice columns 0 .. 33
constexpr int LT_A = LEARNED_TAIL_SIDE;

template <typename T>
struct LearnedTailArgs {
  int it[8];
  int n, nlev;  // side of the finest level, number of levels
  const T* r;
  const double* a;
  T* sprev;
  T* scur;
  int rp, ap, sp;
  const float* w;
  DevState* st;
  double* hist;
  const double* partials;  // of the previous cycle's residual norm (cycle < 0: none)
  int count, cycle;
};

template <typename C>
struct LearnedTailLds {
  uint64_t fb[3 * LB_FPL];
  C x[LT_P * LT_P], xp[LT_P * LT_P];
  C r[33 * 33 + 17 * 17 + 9 * 9 + 5 * 5 + 3 * 3 + 2];
  float z[9 * LB_FPL];
  float a[LT_A * LT_A];
};

template <typename T, bool VAR>
__global__ __launch_bounds__(LB_NT) void k_learned_tail(LearnedTailArgs<T> q) {
  using C = typename Tr<T>::C;
  extern __shared__ __align__(16) unsigned char smem[];
  LearnedTailLds<C>& L = *reinterpret_cast<LearnedTailLds<C>*>(smem);
  __shared__ int s_done;
  DevState st = *q.st;
  if (st.done) return;
  const int t = threadIdx.x, n = q.n, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int J = 1 + (t >> 5), I = 1 + (t & 31);  // the lane's node at every level
  // right-hand side and coefficient of the finest level; the rest starts at 0
  // (features and Z of boundary nodes stay so)
  for (int i = t; i < n * n; i += LB_NT) {
    L.r[i] = ld(q.r + (i / n) * q.rp + i % n);
    if (VAR) L.a[i] = float(q.a[(i / n) * q.ap + i % n]);
  }
  for (int i = t; i < 3 * LB_FPL; i += LB_NT) L.fb[i] = 0;
  for (int i = t; i < 9 * LB_FPL; i += LB_NT) L.z[i] = 0.f;
  for (int i = t; i < LT_P * LT_P; i += LB_NT) L.x[i] = L.xp[i] = C(0);
  const LaneConst kc = lane_const(q.w);
  if (q.cycle >= 0) {
    const double s = fin_sum(q.partials, q.count);
    if (t == 0) {
      q.hist[q.cycle] = fin_update(st, s, q.cycle);
      *q.st = st;
      s_done = st.done;
    }
    __syncthreads();
    if (s_done) return;
  }
  __syncthreads();
  // restrictions (full weighting, as k_restrict_2d)
  int off = 0;
  for (int k = 1; k < q.nlev; ++k) {
    const int nf = ((n - 1) >> (k - 1)) + 1, nc = ((n - 1) >> k) + 1;
    const C* F = L.r + off + 2 * J * nf + 2 * I;
    off += nf * nf;
    if (J <= nc - 2 && I <= nc - 2) {
      auto rs = [&](int o) { return fmac(C(2), F[o], F[o - 1] + F[o + 1]); };
      const C top = rs(-nf), mid = rs(0), bot = rs(nf);
      L.r[off + J * nc + I] = rnd<T>(fmac(C(2), mid, top + bot) * C(0.0625));
    }
    __syncthreads();
  }
  const int me = J * LT_P + I;
  for (int k = q.nlev - 1; k >= 0; --k) {
    const int S = ((n - 1) >> k) + 1, it = q.it[k];
    const bool in = J <= S - 2 && I <= S - 2;
    const double h = 1.0 / double(S - 1);
    const C hl2 = C(h * h);
    C v = C(0), rv = C(0), pv = C(0);
    FaceFactors ff;
    if (in) {
      rv = L.r[off + J * S + I];
      if constexpr (VAR) {
        const int as = 1 << k;
        const float* a = L.a + (J * n + I) * as;
        ff.set(a[0], a[-as], a[as], a[-as * n], a[as * n]);
      }
      if (k < q.nlev - 1) {  // the hand-over from side (S + 1) / 2
        const int o = (J >> 1) * LT_P + (I >> 1);
        const C* p = L.xp + o;
        const C tx = C(I & 1) * C(0.5), ty = C(J & 1) * C(0.5);
        const C top = lerp(p[0], p[1], tx), bot = lerp(p[LT_P], p[LT_P + 1], tx);
        v = ((J | I) & 1) ? rnd<T>(lerp(top, bot, ty)) : L.x[o];
      }
    }
    __syncthreads();
    if (in) L.x[me] = v;
    __syncthreads();
    const int two = S - 2 > 16;
    for (int s = 0; s < it; ++s) {
      if (in) {
        const C* x = L.x + me;
        float f0, f1, f2;
        node_feature<VAR, C>(ff, v - x[-1], v - x[1], v - x[-LT_P], v - x[LT_P], rv, hl2, f0, f1, f2);
        store_features<LB_FPL>(L.fb + me, f0, f1, f2);
      }
      __syncthreads();
      for (int c = wave; c < (S - 2) << two; c += LB_NT / 64) {
        const int j = c >> two, i = two && (c & 1) ? 16 : 0;
        contract16<LT_P, LB_FPL, LB_FPL>(L.z + (j + 1) * LT_P + i + 1, L.fb + j * LT_P + i, kc,
                                         i + (t & 15) <= S - 3);
      }
      __syncthreads();
      if (in) {
        pv = v;
        v = rnd<T>(v + C(sum_taps<LT_P, LB_FPL>(L.z + me - LT_P - 1)));
        L.x[me] = v;
        if (s == it - 1) L.xp[me] = pv;
      }
      __syncthreads();
    }
    if (k == 0 && in) {
      st_w(q.sprev + J * q.sp + I, pv);
      st_w(q.scur + J * q.sp + I, v);
    }
    if (k > 0) {
      const int SF = 2 * S - 1;
      off -= SF * SF;
    }
  }
}

template <typename T, bool VAR, int NT>
hipError_t tiles_launch(const LearnedTileArgs<T>& q, int blocks, size_t lds, hipStream_t s) {
  hipError_t e = allow_lds(k_learned_tiles<T, VAR, NT>, lds);
  if (e != hipSuccess) return e;
  HOMG_LAUNCH_SMEM((k_learned_tiles<T, VAR, NT>), dim3(unsigned(blocks)), dim3(NT), lds, s, q);
}

template <typename T>
hipError_t learned_tiles_t(int n, int it, double hl, const void* xo, void* xn, void* xp, const Lay& cl, const void* r,
                           const Lay& rl, const double* a, const Lay& al, double* u, const Lay& ul, const L1State* l1,
                           const float* w, const int* done, hipStream_t s) {
  using C = typename Tr<T>::C;
  // 32-bit element offsets inside the kernel
  const int64_t lim = int64_t(1) << 31;
  if (cl.pitch * n >= lim || rl.pitch * n >= lim || (a && al.pitch * n >= lim) || (u && ul.pitch * n >= lim))
    return hipErrorInvalidValue;
  LearnedTileArgs<T> q{};
  if (xo) q.xo = static_cast<const T*>(xo) + cl.off;
  if (xn) q.xn = static_cast<T*>(xn) + cl.off;
  if (xp) q.xp = static_cast<T*>(xp) + cl.off;
  q.cp = int(cl.pitch);
  q.rp = int(rl.pitch);
  q.r = static_cast<const T*>(r) + rl.off;
  if (a) {
    q.a = a + al.off;
    q.ap = int(al.pitch);
  }
  if (u) {
    q.u = u + ul.off;
    q.up = int(ul.pitch);
  }
  if (l1) {
    q.lcur = static_cast<const T*>(l1->cur) + l1->cl.off;
    if (!l1->zero_old) q.lprev = static_cast<const T*>(l1->prev) + l1->cl.off;
    q.lp = int(l1->cl.pitch);
  }
  q.n = n;
  const int own = LB_H - 2 * (3 * it - 2);
  q.nb = (n - 2 + own - 1) / own;
  q.it = it;
  q.hl2 = C(hl * hl);
  q.w = w;
  q.done = done;
  const size_t lds = sizeof(LearnedTileLds<C>);
  const int blocks = q.nb * q.nb;
  if (blocks > LB_WIDE_BLOCKS) return a ? tiles_launch<T, true, 512>(q, blocks, lds, s) : tiles_launch<T, false, 512>(q, blocks, lds, s);
  return a ? tiles_launch<T, true, 1024>(q, blocks, lds, s) : tiles_launch<T, false, 1024>(q, blocks, lds, s);
}

template <typename T>
hipError_t learned_tail_t(int n, int nlev, const int* its, const double* a, const Lay& al, const void* r, const Lay& rl,
                          void* sprev, void* scur, const Lay& sl, const float* w, DevState* st, double* hist,
                          const double* partials, int count, int cycle, hipStream_t s) {
  using C = typename Tr<T>::C;
  LearnedTailArgs<T> q{};
  for (int k = 0; k < nlev; ++k) q.it[k] = its[k];
  q.n = n;
  q.nlev = nlev;
  q.r = static_cast<const T*>(r) + rl.off;
  q.rp = int(rl.pitch);
  if (a) {
    q.a = a + al.off;
    q.ap = int(al.pitch);
  }
  q.sprev = static_cast<T*>(sprev) + sl.off;
  q.scur = static_cast<T*>(scur) + sl.off;
  q.sp = int(sl.pitch);
  q.w = w;
  q.st = st;
  q.hist = hist;
  q.partials = partials;
  q.count = count;
  q.cycle = partials ? cycle : -1;
  const size_t lds = sizeof(LearnedTailLds<C>);
  hipError_t e;
  if (a) {
    if ((e = allow_lds(k_learned_tail<T, true>, lds)) != hipSuccess) return e;
    HOMG_LAUNCH_SMEM((k_learned_tail<T, true>), dim3(1), dim3(LB_NT), lds, s, q);
  }
  if ((e = allow_lds(k_learned_tail<T, false>, lds)) != hipSuccess) return e;
  HOMG_LAUNCH_SMEM((k_learned_tail<T, false>), dim3(1), dim3(LB_NT), lds, s, q);
}

}  // namespace

size_t learned_tiles_lds(int prec) {
  return prec == PREC_F64 ? std::max(sizeof(LearnedTileLds<double>), sizeof(LearnedTailLds<double>))
                          : std::max(sizeof(LearnedTileLds<float>), sizeof(LearnedTailLds<float>));
}

hipError_t launch_learned_tiles(int prec, int n, int it, double hl, const void* xo, void* xn, void* xp, const Lay& cl,
                                const void* r, const Lay& rl, const double* a, const Lay& al, double* u, const Lay& ul,
                                const L1State* l1, const float* w, const int* done, hipStream_t s) {
  if (n < 3 || it < 1 || it > LEARNED_TILE_IT || (l1 && (n < 5 || l1->cl.side != (n - 1) / 2 + 1)) || (u != nullptr) == (xn != nullptr))
    return hipErrorInvalidValue;
#define LT_CASE(T) return learned_tiles_t<T>(n, it, hl, xo, xn, xp, cl, r, rl, a, al, u, ul, l1, w, done, s)
  switch (prec) {
    case PREC_F64: LT_CASE(double);
    case PREC_F32: LT_CASE(float);
    default: LT_CASE(bf16);
  }
#undef LT_CASE
}

hipError_t launch_learned_tail(int prec, int n, int nlev, const int* its, const double* a, const Lay& al, const void* r,
                               const Lay& rl, void* sprev, void* scur, const Lay& sl, const float* w, DevState* st,
                               double* hist, const double* partials, int count, int cycle, hipStream_t s) {
  if (n < 3 || n > LEARNED_TAIL_SIDE || nlev < 1 || nlev > 8 || ((n - 1) >> (nlev - 1)) + 1 < 3 || sl.side != n ||
      rl.side != n || (a && al.side != n))
    return hipErrorInvalidValue;
#define LT_CASE(T) return learned_tail_t<T>(n, nlev, its, a, al, r, rl, sprev, scur, sl, w, st, hist, partials, count, cycle, s)
  switch (prec) {
    case PREC_F64: LT_CASE(double);
    case PREC_F32: LT_CASE(float);
    default: LT_CASE(bf16);
  }
#undef LT_CASE
}

}  // namespace homg
