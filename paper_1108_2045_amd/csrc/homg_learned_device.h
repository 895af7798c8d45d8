// homg_learned_device.h -- the learned relaxation's inference on the matrix
// cores, shared by its kernels.
//
// The two channel contractions run on the matrix cores
// (v_mfma_f32_16x16x32_bf16: D = A B + D with A 16 x 32, B 32 x 16, BF16
// operands, FP32 accumulation).  Operand layout (one wave, lane l,
// g = l / 16): A[i][k] with i = l % 16, k = 8 g + e; B[k][j] with
// j = l % 16, same k; D[i][j] with j = l % 16, i = 4 g + r.  The weights
// are BF16 values already; each FP32 activation is split exactly into three
// BF16 parts (hi = its top 8 significant bits, mid = the next 8 of the
// remainder, lo = the rest, which fits BF16 exactly since 24 = 3 x 8), so
// every product is exact and only the FP32 accumulation rounds: FP32
// arithmetic on the matrix cores.
//
// Per 16 nodes of a row:
//   first layer  D1[c][node] = sum_s W1[c][s] F[s][node] over K slots
//     s = 12 dy + 4 dx + ci of the 3 x 3 window (27 of 64 slots carry
//     weights), with the features F read from LDS already split, four BF16
//     per node (two MFMAs per part, six in all);
//   H = max(D1, 0) on interior nodes, 0 elsewhere -- the lane holds
//     channels 4g .. 4g+3 of its node, which is exactly the B operand the
//     second layer needs, so H never leaves registers;
//   second layer Z[tap][node] = sum_c W2[c][tap] H[c][node] (K slots
//     8 g + e: hi / mid of channel 4 g + e % 4, then lo of channel 4 g + e
//     and zeros: two MFMAs), written to LDS, a plane per tap;
// and after a barrier the output at a node is y = sum_k Z[k][node + o_k].
// Planes ZPL floats apart with ZPL = 4 mod 16: the 16 nodes by four taps a
// wave writes, and the row a wave reads, both fall into different banks (a
// node's taps side by side, 12 floats a node, read four to a bank).
// (A wave going down the rows with a feature row's three words serving three
// rows of nodes took 3 LDS reads a row and lane in place of 9 and rounded in
// another order; it was no faster, the vector instructions are the same.)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "homg_internal.h"

namespace homg {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct Parts {  // an FP32 value as three BF16 parts, in the upper halves of FP32 words
  uint32_t hi, mid, lo;
};

__device__ __forceinline__ Parts split3(float v) {
  Parts p;
  p.hi = __float_as_uint(v) & 0xffff0000u;
  const float r1 = v - __uint_as_float(p.hi);
  p.mid = __float_as_uint(r1) & 0xffff0000u;
  p.lo = __float_as_uint(r1 - __uint_as_float(p.mid));
  return p;
}

// Eight BF16-valued FP32 numbers as a BF16 vector (exact).
__device__ __forceinline__ bf16x8 pack8(const float (&v)[8]) {
  uint32_t p[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    p[k] = (__float_as_uint(v[2 * k]) >> 16) | (__float_as_uint(v[2 * k + 1]) & 0xffff0000u);
  return __builtin_bit_cast(bf16x8, p);
}

__device__ __forceinline__ uint32_t pair16(uint32_t lo_word, uint32_t hi_word) {
  return __builtin_amdgcn_perm(hi_word, lo_word, 0x07060302u);
}

// The lane's operands that do not change from tile to tile.  First-layer K
// slot s (two MFMAs, s in [0, 64)) holds channel s % 4 of feature node
// (dy, dx) = (s / 12, (s % 12) / 4) of the 3 x 3 window (channel 3 and
// s >= 36 are zero weights): with the features stored as four BF16 per
// node, a lane's eight slots of the first MFMA are two whole nodes and
// those of the second one node (lanes 0-15) or nothing.
struct LaneConst {
  bf16x8 w1a, w1b, w2a, w2b;  // A operands: first layer (two MFMAs); second layer (two)
};

__device__ __forceinline__ LaneConst lane_const(const float* __restrict__ w) {
  const int lane = threadIdx.x & 63;
  const int ii = lane & 15, g = lane >> 4;
  LaneConst k;
  // every lane loads (clamped) and then keeps or drops, so the loads carry no
  // branches and are in flight together
  float wa[2][3], wb[3], w2[4];
  auto w1 = [&](int node, int ci) { return w[ii * 27 + ci * 9 + node]; };  // W1[c = ii][ci][tap]
#pragma unroll
  for (int ci = 0; ci < 3; ++ci) {
    wa[0][ci] = w1(2 * g, ci);
    wa[1][ci] = w1(2 * g + 1, ci);
    wb[ci] = w1(8, ci);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) w2[e] = w[NW1 + (4 * g + e) * 9 + min(ii, 8)];  // W2[c][tap = ii]
  float va1[8], vb1[8], va[8], vb[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    va1[e] = (e & 3) < 3 ? wa[e >> 2][(e & 3) < 3 ? e & 3 : 0] : 0.f;
    vb1[e] = e < 3 && g == 0 ? wb[e < 3 ? e : 0] : 0.f;
    va[e] = ii < 9 ? w2[e & 3] : 0.f;
    vb[e] = e < 4 ? va[e] : 0.f;
  }
  k.w1a = pack8(va1);
  k.w1b = pack8(vb1);
  k.w2a = pack8(va);
  k.w2b = pack8(vb);
  return k;
}

__device__ __forceinline__ float frcp(float v) { return __builtin_amdgcn_rcpf(v); }

// The coefficient factors of a node's features: face harmonic means, one over
// their sum and the two ratios, in FP32 with the hardware reciprocal -- all of
// it is rounded to FP32 for the network.
struct FaceFactors {
  float w, e, s, n, inv, gx, gy;
  __device__ __forceinline__ void set(float ac, float aw, float ae, float as, float an) {
    w = 2.f * ac * aw * frcp(ac + aw);
    e = 2.f * ac * ae * frcp(ac + ae);
    s = 2.f * ac * as * frcp(ac + as);
    n = 2.f * ac * an * frcp(ac + an);
    inv = frcp(((w + e) + s) + n);
    gx = (e - w) * frcp(e + w);
    gy = (n - s) * frcp(n + s);
  }
};

// The features of a node from its differences to W, E, S, N and its
// right-hand side, the residual part in the cycle's precision C.
template <bool VAR, typename C>
__device__ __forceinline__ void node_feature(const FaceFactors& k, C dw, C de, C ds, C dn, C rv, C hl2, float& f0,
                                             float& f1, float& f2) {
  if constexpr (!VAR) {
    f0 = float((hl2 * rv - (((dw + de) + ds) + dn)) * C(0.25));
    f1 = f2 = 0.f;
  } else {
    const C flux = ((C(k.w) * dw + C(k.e) * de) + C(k.s) * ds) + C(k.n) * dn;
    f0 = float((hl2 * rv - flux) * C(k.inv));
    f1 = f0 * k.gx;
    f2 = f0 * k.gy;
  }
}

// Features split into their parts and stored: per part (planes FPL apart) one
// 8-byte word per node, channels 0, 1, 2 and a zero.
template <int FPL>
__device__ __forceinline__ void store_features(uint64_t* fb, float f0, float f1, float f2) {
  const Parts p0 = split3(f0), p1 = split3(f1), p2 = split3(f2);
  auto node = [](uint32_t c0, uint32_t c1, uint32_t c2) {
    return uint64_t(pair16(c0, c1)) | (uint64_t(c2 >> 16) << 32);
  };
  fb[0] = node(p0.hi, p1.hi, p2.hi);
  fb[FPL] = node(p0.mid, p1.mid, p2.mid);
  fb[2 * FPL] = node(p0.lo, p1.lo, p2.lo);
}

// Both layers for 16 nodes of a row, one per lane % 16: fb is the feature at
// the first node's window corner (row pitch FP, parts FPL apart), z the first
// node's place in the first Z plane (planes ZPL apart), in: the lane's node is
// interior.
template <int FP, int FPL, int ZPL>
__device__ __forceinline__ void contract16(float* z, const uint64_t* fb, const LaneConst& k, bool in) {
  const int lane = threadIdx.x & 63;
  const int ii = lane & 15, g = lane >> 4;
  // the lane's window nodes (see lane_const): first MFMA nodes 2 g and 2 g + 1,
  // second MFMA node 8 (every lane reads it, the weights keep lanes 0-15's)
  const int na = g == 0 ? 0 : g == 1 ? 2 : g == 2 ? FP + 1 : 2 * FP;
  const int nb = g == 0 ? 1 : g == 1 ? FP : g == 2 ? FP + 2 : 2 * FP + 1;
  fb += ii;
  f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int part = 0; part < 3; ++part) {
    const uint64_t* fp = fb + part * FPL;
    const uint64_t b1[2] = {fp[na], fp[nb]};
    const uint64_t b2[2] = {fp[2 * FP + 2], uint64_t(0)};
    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k.w1a, __builtin_bit_cast(bf16x8, b1), d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k.w1b, __builtin_bit_cast(bf16x8, b2), d, 0, 0, 0);
  }
  Parts h[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) h[r] = split3((in & (d[r] > 0.f)) ? d[r] : 0.f);  // no short circuit: a select
  const uint32_t ba[4] = {pair16(h[0].hi, h[1].hi), pair16(h[2].hi, h[3].hi), pair16(h[0].mid, h[1].mid),
                          pair16(h[2].mid, h[3].mid)};
  const uint32_t bb[4] = {pair16(h[0].lo, h[1].lo), pair16(h[2].lo, h[3].lo), 0u, 0u};
  f32x4 y = {0.f, 0.f, 0.f, 0.f};
  y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k.w2a, __builtin_bit_cast(bf16x8, ba), y, 0, 0, 0);
  y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k.w2b, __builtin_bit_cast(bf16x8, bb), y, 0, 0, 0);
  z += 4 * g * ZPL + ii;  // taps 4 g .. 4 g + 3, nine in all
  if (g < 3) z[0] = y[0];
  if (g < 2) {
#pragma unroll
    for (int r = 1; r < 4; ++r) z[r * ZPL] = y[r];
  }
}

// y at a node: z is the first plane at its window's corner (row pitch ZP).
template <int ZP, int ZPL>
__device__ __forceinline__ float sum_taps(const float* z) {
  float y = 0.f;
#pragma unroll
  for (int k = 0; k < 9; ++k) y += z[k * ZPL + (k / 3) * ZP + k % 3];
  return y;
}

}  // namespace homg
