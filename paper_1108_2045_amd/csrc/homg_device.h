// homg_device.h -- device code shared by the HIP sources: storage types,
// node formulas, lane exchange, reductions, and the launch macros.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "homg_internal.h"

namespace homg {

// ------------------------------------------------------------ storage types

struct bf16 {
  uint16_t bits;
};

template <typename T> struct Tr;
template <> struct Tr<double> { using C = double; };
template <> struct Tr<float> { using C = float; };
template <> struct Tr<bf16> { using C = float; };

__device__ __forceinline__ double ld(const double* p) { return *p; }
__device__ __forceinline__ float ld(const float* p) { return *p; }
__device__ __forceinline__ float ld(const bf16* p) {
  return __uint_as_float(uint32_t(p->bits) << 16);
}
// Stores are streaming (non-temporal): every kernel here writes each output
// element once and the next kernel reads it from memory, so the written
// lines need not stay in the caches (on MI355X this lifts a read+write
// stream from about 5.2 to 7.5 TB/s).
__device__ __forceinline__ void st(double* p, double v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ void st(float* p, float v) { __builtin_nontemporal_store(v, p); }
// FP32 -> BF16, round to nearest even; NaN stays NaN (quieted: the upper
// half of its bits with bit 6 set).  One v_cvt_pk_bf16_f32: on MI355X it
// gives exactly that result for every one of the 2^32 FP32 bit patterns,
// where the same rounding done with integer operations took five or six
// instructions per value.
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, __bf16(f)); }
__device__ __forceinline__ void st(bf16* p, float v) { __builtin_nontemporal_store(f2bf(v), &p->bits); }
// Write-only passes (a level's whole-grid write, the coarse-level sweeps)
// keep ordinary stores: on MI355X a pure write stream runs faster with them
// (5.6 against 4.5 TB/s), while streams that also read gain from streaming
// stores.
__device__ __forceinline__ void st_w(double* p, double v) { *p = v; }
__device__ __forceinline__ void st_w(float* p, float v) { *p = v; }
__device__ __forceinline__ void st_w(bf16* p, float v) { p->bits = f2bf(v); }
// u += v on the caller's FP64 array (the last iteration of a cycle).
__device__ __forceinline__ void add_to(double* p, double v) { __builtin_nontemporal_store(*p + v, p); }

// Value as it reads back after a store in storage type T.
template <typename T> __device__ __forceinline__ typename Tr<T>::C rnd(typename Tr<T>::C v) { return v; }
template <> __device__ __forceinline__ float rnd<bf16>(float v) {
  return __uint_as_float(uint32_t(f2bf(v)) << 16);
}

__device__ __forceinline__ double fmac(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmac(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// ------------------------------------------------------------ node formulas
// Shared by every kernel that evaluates a node, so results agree bit for bit.

// Damped Jacobi at a lattice node, constant coefficient (Sec. 2, level-m
// relaxation with the sign that converges): c + w (h_l^2 r - (2d c - sum nb)),
// w = omega / 2d.  q is the neighbour sum, added pairwise per axis.
template <typename C>
__device__ __forceinline__ C relax_const(C c, C q, C r, C w, C hl2, C two_d) {
  C lap = fmac(two_d, c, -q);           // 2d c - sum nb
  C res = fmac(hl2, r, -lap);           // h_l^2 r - (2d c - sum nb)
  return fmac(w, res, c);
}

// Harmonic mean of two nodal coefficients (the face coefficient).
__device__ __forceinline__ double harm(double a, double b) { return 2.0 * a * b / (a + b); }

// Damped Jacobi for -div(a grad) at a lattice node: c + w (h_l^2 r - flux) / sum_a
// with face coefficients the harmonic means of the nodal coefficient
// (w = omega here).  Neighbours in the order -x, +x, -y, +y.
template <typename C>
__device__ __forceinline__ C relax_var(C c, C xm, C xp, C ym, C yp, double ac, double axm,
                                       double axp, double aym, double ayp, C r, C w, C hl2) {
  const C cxm = C(harm(ac, axm)), cxp = C(harm(ac, axp));
  const C cym = C(harm(ac, aym)), cyp = C(harm(ac, ayp));
  const C sa = (cxm + cxp) + (cym + cyp);
  const C flux = fmac(cxm, c - xm, cxp * (c - xp)) + fmac(cym, c - ym, cyp * (c - yp));
  return fmac(w / sa, fmac(hl2, r, -flux), c);
}

// Linear interpolation a + t (b - a), t in [0, 1).
template <typename C>
__device__ __forceinline__ C lerp(C a, C b, C t) { return fmac(t, b - a, a); }

// ------------------------------------------------------------ lane exchange
// The value of the previous / next lane of the wave (lane i gets lane i - 1
// / i + 1) by a DPP wave shift (a VALU move; no LDS round trip as with
// __shfl_up / __shfl_down).  The lane at the wave's end reads 0; every
// caller discards what those lanes compute.
__device__ __forceinline__ int dpp_prev(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true);  // wave_shr:1
}
__device__ __forceinline__ int dpp_next(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true);  // wave_shl:1
}
__device__ __forceinline__ float lane_prev(float v) { return __int_as_float(dpp_prev(__float_as_int(v))); }
__device__ __forceinline__ float lane_next(float v) { return __int_as_float(dpp_next(__float_as_int(v))); }
__device__ __forceinline__ double lane_prev(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = unsigned(dpp_prev(int(b))), hi = unsigned(dpp_prev(int(b >> 32)));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double lane_next(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = unsigned(dpp_next(int(b))), hi = unsigned(dpp_next(int(b >> 32)));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// The same shifts where the end lane takes `edge` instead: the DPP move
// leaves a lane without a source lane at its old value (bound_ctrl off), so
// no lane-dependent select follows the shift (the compiler may turn such a
// select into a branch that runs the shift with the end lane switched off,
// and an inactive source lane reads 0).
__device__ __forceinline__ double lane_prev_or(double edge, double v) {
  const long long b = __double_as_longlong(v), e = __double_as_longlong(edge);
  const unsigned lo = unsigned(__builtin_amdgcn_update_dpp(int(e), int(b), 0x138, 0xf, 0xf, false));
  const unsigned hi = unsigned(__builtin_amdgcn_update_dpp(int(e >> 32), int(b >> 32), 0x138, 0xf, 0xf, false));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double lane_next_or(double edge, double v) {
  const long long b = __double_as_longlong(v), e = __double_as_longlong(edge);
  const unsigned lo = unsigned(__builtin_amdgcn_update_dpp(int(e), int(b), 0x130, 0xf, 0xf, false));
  const unsigned hi = unsigned(__builtin_amdgcn_update_dpp(int(e >> 32), int(b >> 32), 0x130, 0xf, 0xf, false));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ float lane_prev_or(float edge, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_next_or(float edge, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xf, 0xf, false));
}

// ------------------------------------------------------------ reductions

// v + the value `n` lanes on in its row of 16 (DPP rotation).
template <int N>
__device__ __forceinline__ double add_rot16(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = unsigned(__builtin_amdgcn_update_dpp(0, int(b), 0x120 + N, 0xf, 0xf, true));
  const unsigned hi = unsigned(__builtin_amdgcn_update_dpp(0, int(b >> 32), 0x120 + N, 0xf, 0xf, true));
  return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over the wave, in every lane: pairs 32 lanes apart, then 16, 8, 4, 2, 1.
// Once lanes 8 apart hold the same sum, the lane 4 on in a row of 16 holds
// what the lane with bit 2 flipped does, and so on down: the last four steps
// are row rotations (VALU moves; six steps of lane shuffles, two LDS crossbar
// operations each, were bound by the crossbar where 16 waves summed at once).
__device__ __forceinline__ double wave_sum(double v) {
  v += __shfl_xor(v, 32, 64);
  v += __shfl_xor(v, 16, 64);
  v = add_rot16<8>(v);
  v = add_rot16<4>(v);
  v = add_rot16<2>(v);
  return add_rot16<1>(v);
}

// Deterministic block sum (fixed order for a fixed block size); result valid
// in thread 0.  Every thread of the block must call it.
template <int NT>
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double red[NT / 64];
  v = wave_sum(v);
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (tid == 0) {
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) s += red[w];
  }
  return s;
}

constexpr int FIN_NT = 1024;
__device__ __forceinline__ double fin_sum(const double* __restrict__ partials, int count) {
  double s = 0.0;
  for (int i = threadIdx.x; i < count; i += FIN_NT) s += partials[i];
  return block_sum<FIN_NT>(s);
}

// The state after the norm of cycle `cycle`'s residual (one thread): v holds
// the state before it.
__device__ __forceinline__ double fin_update(DevState& v, double s, int cycle) {
  const double rel = sqrt(s) / v.fnorm;
  v.cycles = cycle;
  if (!(rel <= 1.7976931348623157e308)) v.done = 2;  // NaN or Inf
  else if (v.stop_on_tol && rel <= v.tol) v.done = 1;
  return rel;
}

// i -> (I, J, K) in a box of side s (x fastest); a single-precision
// reciprocal is exact here: i < 2^24 and (i + 1/2) / s stays at least
// 1/(2 s) away from an integer.
template <int D>
__device__ __forceinline__ void tail_split(int i, int s, float inv_s, int& I, int& J, int& K) {
  const int q = int((float(i) + 0.5f) * inv_s);
  I = i - q * s;
  if (D == 2) {
    J = q;
    K = 0;
  } else {
    K = int((float(q) + 0.5f) * inv_s);
    J = q - K * s;
  }
}

// ------------------------------------------------------------ launch shapes

constexpr int BX2 = 256;          // 2D: lanes per block
// 2D tiles: a block's four waves take TW2 = 64 columns each on four
// consecutive bands of `len` rows (wave w of block row `by` walks band
// 4 by + w), so the waves of one block write different rows.  Measured on
// MI355X with a padded 4097^2 FP64 array: a pure write stream runs at 5.9
// TB/s this way against 4.2 TB/s with the four waves side by side on the
// same rows, and a two-read one-write stream with streaming stores at 7.8
// against 6.9 TB/s.
constexpr int TW2 = 64;
__device__ __forceinline__ int t2_x(int bx) { return 1 + bx * TW2 + int(threadIdx.x & 63); }
__device__ __forceinline__ int t2_y0(int by, int len) { return 1 + (by * 4 + int(threadIdx.x >> 6)) * len; }
__host__ __device__ inline int t2_gx(int n) { return (n - 2 + TW2 - 1) / TW2; }
__host__ __device__ inline int t2_gy(int n, int len) { return (n - 2 + 4 * len - 1) / (4 * len); }

// Workgroups of a launch are dealt to the 8 XCDs round-robin (workgroup h
// runs on XCD h % 8).  xcd_order maps h to a logical index so that each XCD
// receives one contiguous range of logical workgroups (a bijection on
// [0, count)).
__device__ __forceinline__ unsigned xcd_order(unsigned h, unsigned count) {
  const unsigned q = count / 8, rem = count % 8, x = h % 8;
  return x * q + min(x, rem) + h / 8;
}

// ------------------------------------------------------------ launches

#define HOMG_LAUNCH_SMEM(kernel, grid, block, smem, stream, ...)                              \
  do {                                                                                        \
    hipEvent_t ev_a_, ev_b_;                                                                  \
    current_launch_events(&ev_a_, &ev_b_);                                                    \
    hipExtLaunchKernelGGL(kernel, grid, block, smem, stream, ev_a_, ev_b_, 0,        \
                          __VA_ARGS__);                                                       \
    return hipGetLastError();                                                                 \
  } while (0)

#define HOMG_LAUNCH(kernel, grid, block, stream, ...) \
  HOMG_LAUNCH_SMEM(kernel, grid, block, 0, stream, __VA_ARGS__)

// Opt a kernel in to more than 64 KB of dynamic LDS.
template <typename K>
static hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
}

}  // namespace homg
