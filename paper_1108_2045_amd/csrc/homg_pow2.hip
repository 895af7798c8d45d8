// homg_pow2.hip -- power-of-two grids (Sec. 3): the whole-grid iterations,
// the restriction families, and the compact form in which a level's
// iterations touch its marks alone.
#include "homg_device.h"
#include "homg_internal.h"

namespace homg {

// ------------------------------------------------------------ power-of-two grids
// Sec. 3: a 2D grid of N = 2^k nodes per side in four quadrants.  Level-m
// marks of quadrant (sx, sy) are the nodes whose coordinates, measured from
// the quadrant's external corner (index 0 on side 0, N-1 on side 1), are
// multiples of l = 2^m no larger than N/2 -- the last one just outside the
// quadrant.  Every interior mark relaxes (5-point stencil at distance l on
// the whole grid, a neighbour outside the grid reads 0) with its quadrant's
// restricted residual; every other interior node interpolates bilinearly
// from the marks of the quadrant that owns it (no cross-quadrant reads).
// The marks of side 0 are even and those of side 1 odd on every axis, so
// each node has at most one owner lattice.  Each quadrant's residuals form
// a nested sequence anchored at its corner ("family"): level j is the full
// weighting of level j-1 on compact arrays of side N >> j whose index 0 (the
// domain boundary) stays 0.

// Mark side (0 or 1) of coordinate x at stride l = 2^m, or -1.
__device__ __forceinline__ int p2_side(int x, int N, int m) {
  const int mask = (1 << m) - 1, half = N >> 1;
  if ((x & mask) == 0 && x <= half) return 0;
  const int a = N - 1 - x;
  if ((a & mask) == 0 && a <= half) return 1;
  return -1;
}

constexpr int P2_ROWS = 8;  // rows walked per block by the whole-grid passes

// One iteration at level m >= 1 over the whole grid.  fam[q] points at node
// (0, 0) of family q's level-m array (pitch fp).
template <int MODE>
__global__ __launch_bounds__(256) void k_p2_sweep(const double* __restrict__ eo, double* __restrict__ en,
                                                  int64_t ep, const double* __restrict__ f0,
                                                  const double* __restrict__ f1, const double* __restrict__ f2,
                                                  const double* __restrict__ f3, int64_t fp, int N, int m,
                                                  double w, double hl2, double* __restrict__ u, int64_t up,
                                                  const int* __restrict__ done) {
  if (*done) return;
  const int x = t2_x(blockIdx.x);
  if (x > N - 2) return;
  const int l = 1 << m, half = N >> 1;
  // 1 / l is exact (l a power of two), so the weights below equal the
  // quotients (ax - cx) / l bit for bit without a division per node
  const double inv_l = 1.0 / double(l);
  const int sx = p2_side(x, N, m);
  const int tx = x >= half ? 1 : 0;
  const int ax = tx ? N - 1 - x : x, cx = (ax >> m) << m;
  const int gx0 = tx ? N - 1 - cx : cx, gx1 = tx ? N - 1 - (cx + l) : cx + l;
  const double fx = double(ax - cx) * inv_l;
  const int y0 = t2_y0(blockIdx.y, P2_ROWS), y1 = min(N - 1, y0 + P2_ROWS);
  // the corners of the lattice cell last interpolated from (the walk
  // reloads them only when a row lies in another cell)
  int cell = -1;
  double c00 = 0.0, c01 = 0.0, c10 = 0.0, c11 = 0.0;
  for (int y = y0; y < y1; ++y) {
    const int sy = p2_side(y, N, m);
    double v;
    if (sx >= 0 && sy >= 0) {
      const double* fam = sy ? (sx ? f3 : f2) : (sx ? f1 : f0);
      const int a = sx ? N - 1 - x : x, b = sy ? N - 1 - y : y;
      const double rv = fam[int64_t(b >> m) * fp + (a >> m)];
      double c = 0.0, q = 0.0;
      if (!(MODE & SW_ZERO_OLD)) {
        const double* row = eo + int64_t(y) * ep;
        c = row[x];
        const double xm = x - l >= 0 ? row[x - l] : 0.0;
        const double xp = x + l <= N - 1 ? row[x + l] : 0.0;
        const double ym = y - l >= 0 ? eo[int64_t(y - l) * ep + x] : 0.0;
        const double yp = y + l <= N - 1 ? eo[int64_t(y + l) * ep + x] : 0.0;
        q = (xm + xp) + (ym + yp);
      }
      v = relax_const<double>(c, q, rv, w, hl2, 4.0);
    } else if (MODE & SW_ZERO_OLD) {
      v = 0.0;
    } else {
      const int ty = y >= half ? 1 : 0;
      const int ay = ty ? N - 1 - y : y, cy = (ay >> m) << m;
      const int gy0 = ty ? N - 1 - cy : cy, gy1 = ty ? N - 1 - (cy + l) : cy + l;
      const double fy = double(ay - cy) * inv_l;
      const int key = gy0 * 2 + ty;
      if (key != cell) {
        const double* r0 = eo + int64_t(gy0) * ep;
        const double* r1 = eo + int64_t(gy1) * ep;
        c00 = r0[gx0];
        c01 = r0[gx1];
        c10 = r1[gx0];
        c11 = r1[gx1];
        cell = key;
      }
      v = lerp(lerp(c00, c01, fx), lerp(c10, c11, fx), fy);
    }
    if (MODE & SW_ACCUM)
      add_to(u + int64_t(y) * up + x, v);
    else
      st_w(en + int64_t(y) * ep + x, v);
  }
}

hipError_t launch_p2_sweep(int N, int m, double omega, const double* eo, double* en, const Lay& el,
                           const double* const* fam, const Lay& fl, double* u, const Lay& ul, int mode,
                           const int* done, hipStream_t s) {
  if (m < 1 || N < 4 || (N & (N - 1)) || fl.side != (N >> m)) return hipErrorInvalidValue;
  const double hl = double(1 << m) / double(N - 1);
  const dim3 g(t2_gx(N), t2_gy(N, P2_ROWS));
  const double* e = eo + el.off;
  double* o = en + el.off;
  double* uu = u ? u + ul.off : nullptr;
  const double *f0 = fam[0] + fl.off, *f1 = fam[1] + fl.off, *f2 = fam[2] + fl.off, *f3 = fam[3] + fl.off;
#define P2_CASE(MODE)                                                                                       \
  HOMG_LAUNCH((k_p2_sweep<MODE>), g, dim3(256), s, e, o, el.pitch, f0, f1, f2, f3, fl.pitch, N, m, omega / 4.0, \
              hl * hl, uu, ul.pitch, done)
  switch (mode & (SW_ZERO_OLD | SW_ACCUM)) {
    case 0: P2_CASE(0);
    case SW_ZERO_OLD: P2_CASE(SW_ZERO_OLD);
    case SW_ACCUM: P2_CASE(SW_ACCUM);
    default: P2_CASE(SW_ZERO_OLD | SW_ACCUM);
  }
#undef P2_CASE
}

// ------------------------------------------------------------ restriction families

// Level 1 of all four families from the whole-grid r_0, read once.  A lane
// owns the fine columns 2k and 2k + 1 -- the centres of x-side 0's node k and
// of x-side 1's node N/2 - 1 - k -- and walks pairs of rows the same way; the
// columns beside its own come from the neighbour lanes.  One launch per
// family read r_0 four times (108 us at 4096^2 against 55).
constexpr int P2R_ROWS = 8;  // row pairs per wave
__global__ __launch_bounds__(256) void k_p2_restrict_first(const double* __restrict__ F, int64_t fp,
                                                           double* __restrict__ c0, double* __restrict__ c1,
                                                           double* __restrict__ c2, double* __restrict__ c3,
                                                           int64_t cp, int N, const int* __restrict__ done) {
  if (*done) return;
  const int half = N >> 1, lane = threadIdx.x & 63;
  const int k = blockIdx.x * 64 + lane;
  const int K0 = (blockIdx.y * 4 + int(threadIdx.x >> 6)) * P2R_ROWS;
  if (K0 >= half) return;  // the whole wave
  const int K1 = min(half, K0 + P2R_ROWS);
  const bool kin = k < half;
  const int kc = min(k, half - 1);
  const int xl = max(2 * kc - 1, 0), xr = min(2 * kc + 2, N - 1);
  double s0, s1;  // row sums of x-sides 0 and 1
  auto row = [&](int y) {
    const double* p = F + int64_t(min(max(y, 0), N - 1)) * fp;
    const double a = p[2 * kc], b = p[2 * kc + 1];
    double el = 0.0, er = 0.0;
    if (lane == 0) el = p[xl];
    if (lane == 63) er = p[xr];
    const double l = lane_prev_or(el, b);  // column 2k - 1
    const double r = lane_next_or(er, a);  // column 2k + 2
    s0 = fmac(2.0, a, l + b);
    s1 = fmac(2.0, b, a + r);
  };
  // (k = 0 and k = N/2 - 1 read 0 or a clamped column beyond the grid for the
  // side whose node is the boundary: that node is not written)
  double t0, t1, m0, m1, b0, b1, n0, n1;
  row(2 * K0 - 1);
  t0 = s0; t1 = s1;
  row(2 * K0);
  m0 = s0; m1 = s1;
  for (int K = K0; K < K1; ++K) {
    row(2 * K + 1);
    b0 = s0; b1 = s1;
    row(2 * K + 2);
    n0 = s0; n1 = s1;
    if (kin) {
      const int A1 = half - 1 - k, B1 = half - 1 - K;
      if (K > 0) {
        if (k > 0) c0[int64_t(K) * cp + k] = fmac(2.0, m0, t0 + b0) * 0.0625;
        if (A1 > 0) c1[int64_t(K) * cp + A1] = fmac(2.0, m1, t1 + b1) * 0.0625;
      }
      if (B1 > 0) {
        if (k > 0) c2[int64_t(B1) * cp + k] = fmac(2.0, b0, m0 + n0) * 0.0625;
        if (A1 > 0) c3[int64_t(B1) * cp + A1] = fmac(2.0, b1, m1 + n1) * 0.0625;
      }
    }
    t0 = b0; t1 = b1;
    m0 = n0; m1 = n1;
  }
}

// Level j >= 2 of the four families (blockIdx.z) from level j - 1.  Row and
// column 0 (the domain boundary) stay 0.
struct P2Fams {
  const double* f[4];
  double* c[4];
};
__global__ __launch_bounds__(256) void k_p2_restrict(P2Fams p, int64_t fp, int64_t cp, int nc,
                                                     const int* __restrict__ done) {
  if (*done) return;
  const int A = 1 + blockIdx.x * 64 + threadIdx.x, B = 1 + blockIdx.y * 4 + threadIdx.y;
  if (A >= nc || B >= nc) return;
  const double* F = p.f[blockIdx.z];
  auto rs = [&](int b) {
    const double* q = F + int64_t(b) * fp + 2 * A;
    return fmac(2.0, q[0], q[-1] + q[1]);
  };
  const double top = rs(2 * B - 1), mid = rs(2 * B), bot = rs(2 * B + 1);
  p.c[blockIdx.z][int64_t(B) * cp + A] = fmac(2.0, mid, top + bot) * 0.0625;
}

// ------------------------------------------------------------ compact levels
// The level-m state of a quadrant on its marks alone, seen from its corner:
// index i is the coordinate i l, marks 1 .. h = N / 2l on each axis, index 0
// the boundary (0).  A mark next to the quadrant's far end also relaxes with
// the node at N/2 + l, which another quadrant interpolates: its value is kept
// as index h + 1 (a ghost) and evolves like the whole grid's node -- at
// iteration t the interpolant of that quadrant's marks at iteration t - 1 --
// so one iteration needs the state before it and nothing else.  The same
// formulas on the same values as the whole-grid iteration: the same bits.
// (At h = 1 the node lies outside the grid: 0.)
template <typename P>
struct P2State {
  P* p;  // quadrant 0 at index (0, 0); quadrant 2 sy + sx lies (2 sy + sx) planes on
  int64_t plane, pitch;
  __device__ __forceinline__ P* at(int z, int j, int i) const { return p + z * plane + j * pitch + i; }
};
using P2Marks = P2State<const double>;
using P2Out = P2State<double>;

// Whole-grid value of a non-mark node given by its distances (px, py) from
// the corner of quadrant (sx, sy): the bilinear interpolant of the marks of
// the quadrant that owns it (of the other side when at or past N/2).
__device__ __forceinline__ double p2_interp(const P2Marks& s, int N, int m, int sx, int sy, int px, int py) {
  const int half = N >> 1, l = 1 << m;
  const bool ox = px >= half, oy = py >= half;
  const int tx = ox ? 1 - sx : sx, ty = oy ? 1 - sy : sy;
  const int ax = ox ? N - 1 - px : px, ay = oy ? N - 1 - py : py;
  const int ix = ax >> m, iy = ay >> m;
  const double inv_l = 1.0 / double(l);
  const double fx = double(ax - (ix << m)) * inv_l, fy = double(ay - (iy << m)) * inv_l;
  const double* p = s.at(2 * ty + tx, iy, ix);
  return lerp(lerp(p[0], p[1], fx), lerp(p[s.pitch], p[s.pitch + 1], fx), fy);
}

// Whole-grid value of any interior node after a level-m iteration: x_it at
// the marks, else the interpolant of x_{it-1}.
__device__ __forceinline__ double p2_state(const P2Marks& prev, const P2Marks& cur, int N, int m, int sx, int sy,
                                           int px, int py) {
  // the node as seen from the far corners: a mark of side s has its distance
  // from that corner a multiple of l, at most N/2
  const int mask = (1 << m) - 1, half = N >> 1;
  const int qx = N - 1 - px, qy = N - 1 - py;
  const int kx = (px & mask) == 0 && px <= half ? 0 : ((qx & mask) == 0 && qx <= half ? 1 : -1);
  const int ky = (py & mask) == 0 && py <= half ? 0 : ((qy & mask) == 0 && qy <= half ? 1 : -1);
  if (kx >= 0 && ky >= 0) {
    const int tx = kx ? 1 - sx : sx, ty = ky ? 1 - sy : sy;
    return *cur.at(2 * ty + tx, (ky ? qy : py) >> m, (kx ? qx : px) >> m);
  }
  return p2_interp(prev, N, m, sx, sy, px, py);
}

// One iteration of level m: marks relax, ghosts interpolate.
__device__ __forceinline__ double p2_node(const P2Marks& in, const double* __restrict__ fam, int64_t fp, int N, int m,
                                          int sx, int sy, int i, int j, int h, double w, double hl2) {
  if (i <= h && j <= h) {
    const double* p = in.at(2 * sy + sx, j, i);
    const double q = (p[-1] + p[1]) + (p[-in.pitch] + p[in.pitch]);
    return relax_const<double>(p[0], q, fam[int64_t(j) * fp + i], w, hl2, 4.0);
  }
  const int px = i << m, py = j << m;
  return px > N - 1 || py > N - 1 ? 0.0 : p2_interp(in, N, m, sx, sy, px, py);
}

struct P2Fam4 {
  const double* f[4];
};
__global__ __launch_bounds__(256) void k_p2_iter(P2Marks in, P2Out out, P2Fam4 fam, int64_t fp, int N, int m,
                                                 double w, double hl2, const int* __restrict__ done) {
  if (*done) return;
  const int h = N >> (m + 1);
  const int i = 1 + blockIdx.x * 64 + threadIdx.x, j = 1 + blockIdx.y * 4 + threadIdx.y;
  if (i > h + 1 || j > h + 1 || (i > h && j > h)) return;
  const int z = blockIdx.z;
  *out.at(z, j, i) = p2_node(in, fam.f[z], fp, N, m, z & 1, z >> 1, i, j, h, w, hl2);
}

// ---- several iterations of a level in one launch
// A workgroup owns B x B marks of a quadrant and iterates on them with a halo
// of one mark per iteration, the tile nodes in registers and their
// neighbours' values through LDS.  A tile at the quadrant's far end holds the
// ghost at h + 1 too, and beside its own marks (in x, in y or both) the last
// marks of the other side, whose interpolant the ghost is and whose ghost its
// own marks give in turn: [h - 1 - it, h + 1] feed it iterations.  So an axis
// of a tile is one segment of own indices and, at the seam, one of the other
// side's: at most B + 12 positions.  The starting state is formed in the tile
// from the coarser level's pair.  What bounds it is latency: a block loads,
// then runs four short phases.  One launch in place of a hand-over and a
// launch per iteration, four iterations: 21 -> 5 us at h = 32, 33 -> 27 at
// h = 512, 100 -> 88 at h = 1024.  B = 16 (a node per lane, the shortest
// phases) while its blocks fit the chip about once; from h = 256 on B = 32 (two
// nodes per lane), which repeats 1.6 nodes per owned one in place of 2.3 (h =
// 1024: 92 us against 153, before the offsets were 32-bit).
constexpr int P2T_WIDE = 256;
constexpr int p2t_side(int B) { return B + 3 * P2T_IT; }  // positions per axis at most

struct P2TileArgs {
  P2Marks sp, sc;  // the state before: the final pair of level `from`,
  const double* e;  // the whole grid (from = 0), or 0 (from < 0)
  int64_t ep;
  int from;
  P2Out prev, cur;
  P2Fam4 fam;
  int64_t fp;
  int N, m, it, nb;
  double w, hl2;
  const int* done;
};

// The positions of one axis: own indices from lo, then the other side's from
// lob.
template <int B>
struct P2Axis {
  int own, lo, len, lob, lenb;
  __device__ __forceinline__ P2Axis(int side, int a, int it, int h) {
    own = side;
    lo = max(a - it, 0);
    const int hi = min(a + B - 1 + it, h + 1);
    len = hi - lo + 1;
    lob = max(h - 1 - it, 0);
    lenb = hi == h + 1 ? h + 2 - lob : 0;
  }
  __device__ __forceinline__ bool at(int p, int& side, int& idx) const {
    const bool o = p < len;
    side = o ? own : 1 - own;
    idx = o ? lo + p : lob + p - len;
    return p < len + lenb;
  }
  // The position of an index (clamped: what falls outside feeds no owned mark).
  __device__ __forceinline__ int pos(int side, int idx) const {
    return side == own ? min(max(idx - lo, 0), len - 1) : len + min(max(idx - lob, 0), max(lenb - 1, 0));
  }
};

// B: owned marks per axis, K: tile nodes per lane.
template <int B, int NT, int K>
__global__ __launch_bounds__(NT) void k_p2_tile(P2TileArgs g) {
  constexpr int S = p2t_side(B), W = B + 2 * P2T_IT, PAD = S + 1;
  static_assert(S * S <= K * NT && B + P2T_IT + 1 + P2T_IT + 3 <= S, "K tile nodes per lane");
  __shared__ double X[2][S * S + 2 * PAD];
  const int N = g.N, m = g.m, half = N >> 1, h = N >> (m + 1);
  const unsigned lb = xcd_order(blockIdx.x, gridDim.x);
  const unsigned nb2 = unsigned(g.nb) * unsigned(g.nb);
  const int z = int(lb / nb2), bxy = int(lb % nb2);
  const int a = 1 + (bxy % g.nb) * B, b = 1 + (bxy / g.nb) * B;
  double v[K], pv[K], r[K];
  if (max(a, b) + B - 1 + g.it < h) {  // away from the seams: own marks alone
    const int done = *g.done;
    const double* fam = z & 2 ? (z & 1 ? g.fam.f[3] : g.fam.f[2]) : (z & 1 ? g.fam.f[1] : g.fam.f[0]);
    const int side = B + 2 * g.it;
    // 32-bit offsets from the quadrant's arrays (launch_p2_tile checks them; with
    // 64-bit products and a division per node and use 92 us at h = 1024, now 88)
    const double* const sp = g.sp.p + z * g.sp.plane;
    const double* const sc = g.sc.p + z * g.sc.plane;
    const int fp = int(g.fp), pp = int(g.sp.pitch), op = int(g.cur.pitch);
    int pj[K], pi[K], o[K];
    bool mark[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      pj[k] = k ? pj[k - 1] + NT / W : int(threadIdx.x) / W;
      pi[k] = k ? pi[k - 1] + NT % W : int(threadIdx.x) % W;
      if (k && pi[k] >= W) pi[k] -= W, ++pj[k];
      const int i = a - g.it + pi[k], j = b - g.it + pj[k];
      o[k] = PAD + min(pj[k], S - 1) * S + pi[k];
      mark[k] = i >= 1 && j >= 1 && pi[k] < side && pj[k] < side;
      const int ic = min(max(i, 1), h), jc = min(max(j, 1), h);
      v[k] = 0.0;
      pv[k] = 0.0;
      r[k] = fam[jc * fp + ic];
      if (g.from == m + 1) {  // p2_state here: lattice nodes as they are, others interpolated
        const int at = min(jc >> 1, (h >> 1) - 1) * pp + min(ic >> 1, (h >> 1) - 1);
        const double c = sc[at], p00 = sp[at], p01 = sp[at + 1], p10 = sp[at + pp], p11 = sp[at + pp + 1];
        const double fx = double(ic & 1) * 0.5, fy = double(jc & 1) * 0.5;
        v[k] = (ic | jc) & 1 ? lerp(lerp(p00, p01, fx), lerp(p10, p11, fx), fy) : c;
      } else if (g.from > 0) {
        v[k] = p2_state(g.sp, g.sc, N, g.from, z & 1, z >> 1, ic << m, jc << m);
      } else if (g.from == 0) {
        const int px = ic << m, py = jc << m;
        v[k] = g.e[int64_t(z & 2 ? N - 1 - py : py) * g.ep + (z & 1 ? N - 1 - px : px)];
      }
    }
    if (done) return;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!mark[k]) v[k] = 0.0;
      if (pj[k] < W) {
        X[0][o[k]] = v[k];
        if (!mark[k]) X[1][o[k]] = 0.0;
      }
    }
    __syncthreads();
    auto step = [&](int t, const double* in, double* out) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const double* src = in + o[k];
        pv[k] = v[k];
        v[k] = relax_const<double>(v[k], (src[-1] + src[1]) + (src[-S] + src[S]), r[k], g.w, g.hl2, 4.0);
        if (t < g.it && mark[k]) out[o[k]] = v[k];
      }
      if (t < g.it) __syncthreads();
    };
    for (int t = 1; t <= g.it; t += 2) {
      step(t, X[0], X[1]);
      if (t < g.it) step(t + 1, X[1], X[0]);
    }
    double* const oc = g.cur.p + z * g.cur.plane;
    double* const op_ = g.prev.p + z * g.prev.plane;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = a - g.it + pi[k], j = b - g.it + pj[k];
      if (i < a || j < b || i >= a + B || j >= b + B) continue;
      oc[j * op + i] = v[k];
      op_[j * op + i] = pv[k];
    }
    return;
  }
  if (*g.done) return;
  const P2Axis<B> ax(z & 1, a, g.it, h), ay(z >> 1, b, g.it, h);
  double fx[K], fy[K];
  int o00[K], o01[K], o10[K], o11[K];
  bool live[K], mark[K], inside[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int q = threadIdx.x + k * NT, pj = q / S, pi = q % S;
    int sx, sy, i, j;
    const bool ix = ax.at(pi, sx, i), iy = ay.at(pj, sy, j);
    live[k] = q < S * S && ix && iy && i >= 1 && j >= 1 && (i <= h || j <= h);
    mark[k] = live[k] && i <= h && j <= h;
    const int px = i << m, py = j << m;
    inside[k] = live[k] && px <= N - 1 && py <= N - 1;
    v[k] = pv[k] = r[k] = fx[k] = fy[k] = 0.0;
    o00[k] = o01[k] = o10[k] = o11[k] = 0;
    if (inside[k]) {
      if (g.from > 0)
        v[k] = p2_state(g.sp, g.sc, N, g.from, sx, sy, px, py);
      else if (g.from == 0)
        v[k] = g.e[int64_t(sy ? N - 1 - py : py) * g.ep + (sx ? N - 1 - px : px)];
    }
    if (mark[k]) {
      const double* f = sy ? (sx ? g.fam.f[3] : g.fam.f[2]) : (sx ? g.fam.f[1] : g.fam.f[0]);
      r[k] = f[int64_t(j) * g.fp + i];
    } else if (inside[k]) {  // a ghost (as p2_interp): its cell in the quadrant that owns it
      const bool ox = px >= half, oy = py >= half;
      const int tx = ox ? 1 - sx : sx, ty = oy ? 1 - sy : sy;
      const int qx = ox ? N - 1 - px : px, qy = oy ? N - 1 - py : py;
      const int kx = qx >> m, ky = qy >> m;
      const double inv_l = 1.0 / double(1 << m);
      fx[k] = double(qx - (kx << m)) * inv_l;
      fy[k] = double(qy - (ky << m)) * inv_l;
      const int x0 = ax.pos(tx, kx), x1 = ax.pos(tx, kx + 1), y0 = ay.pos(ty, ky), y1 = ay.pos(ty, ky + 1);
      o00[k] = y0 * S + x0;
      o01[k] = y0 * S + x1;
      o10[k] = y1 * S + x0;
      o11[k] = y1 * S + x1;
    }
    if (q < S * S) {
      X[0][PAD + q] = v[k];
      if (!live[k]) X[1][PAD + q] = 0.0;
    }
  }
  __syncthreads();
  for (int t = 1; t <= g.it; ++t) {
    const double* src = &X[(t - 1) & 1][PAD];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int q = threadIdx.x + k * NT;
      pv[k] = v[k];
      if (mark[k]) {
        const double c = (src[q - 1] + src[q + 1]) + (src[q - S] + src[q + S]);
        v[k] = relax_const<double>(v[k], c, r[k], g.w, g.hl2, 4.0);
      } else if (inside[k]) {
        v[k] = lerp(lerp(src[o00[k]], src[o01[k]], fx[k]), lerp(src[o10[k]], src[o11[k]], fx[k]), fy[k]);
      }
      if (t < g.it && live[k]) X[t & 1][PAD + q] = v[k];
    }
    if (t < g.it) __syncthreads();
  }
  // owned marks, and the ghosts behind them at the far end
  const int ae = min(a + B - 1, h), be = min(b + B - 1, h);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int q = threadIdx.x + k * NT, pj = q / S, pi = q % S;
    int sx, sy, i, j;
    ax.at(pi, sx, i);
    ay.at(pj, sy, j);
    const bool own = live[k] && pi < ax.len && pj < ay.len && i >= a && j >= b && i <= (ae == h ? h + 1 : ae) &&
                     j <= (be == h ? h + 1 : be);
    if (!own) continue;
    *g.cur.at(z, j, i) = v[k];
    if (mark[k]) *g.prev.at(z, j, i) = pv[k];
  }
}

// The whole grid after a level: stored in en, or (u given) added into u.  A
// lane walks rows of one column; the x part of the interpolation and the
// column's mark test are formed once.
__global__ __launch_bounds__(256) void k_p2_write(P2Marks prev, P2Marks cur, int m, int N, double* __restrict__ en,
                                                  int64_t ep, double* __restrict__ u, int64_t up,
                                                  const int* __restrict__ done) {
  if (*done) return;
  const int x = t2_x(blockIdx.x);
  if (x > N - 2) return;
  const int half = N >> 1;
  const double inv_l = 1.0 / double(1 << m);
  const int sx = p2_side(x, N, m);
  const int mx = sx == 1 ? (N - 1 - x) >> m : x >> m;  // the column's mark index, if it is one
  const int tx = x >= half ? 1 : 0, ax = tx ? N - 1 - x : x, ix = ax >> m;
  const double fx = double(ax - (ix << m)) * inv_l;
  const int y0 = t2_y0(blockIdx.y, P2_ROWS), y1 = min(N - 1, y0 + P2_ROWS);
  int cell = -1;
  double r0 = 0.0, r1 = 0.0;  // x-interpolants of the cell's two mark rows
  for (int y = y0; y < y1; ++y) {
    const int sy = p2_side(y, N, m);
    double v;
    if (sx >= 0 && sy >= 0) {
      const int my = (sy ? N - 1 - y : y) >> m;
      v = *cur.at(2 * sy + sx, my, mx);
    } else {
      const int ty = y >= half ? 1 : 0, ay = ty ? N - 1 - y : y, iy = ay >> m;
      const int key = 2 * iy + ty;
      if (key != cell) {
        const double* p = prev.at(2 * ty + tx, iy, ix);
        r0 = lerp(p[0], p[1], fx);
        r1 = lerp(p[prev.pitch], p[prev.pitch + 1], fx);
        cell = key;
      }
      v = lerp(r0, r1, double(ay - (iy << m)) * inv_l);
    }
    if (u)
      add_to(u + int64_t(y) * up + x, v);
    else
      st_w(en + int64_t(y) * ep + x, v);
  }
}

// ---- the leading coarse levels in one workgroup
// Levels ms .. top of the schedule's start (each once, descending), h <=
// P2_TAIL_H at level ms: the families of level ms in LDS, restricted to the
// coarser levels there, and every level's iterations; leaves level ms's
// final pair.  As launches these levels took some 30 of 4 us each per cycle;
// here a mark per lane keeps its value, right-hand side and place in registers
// (16.7 us at h = 16 .. 1; 21 with every node's place worked out again in each
// iteration).
// Also reduces the previous residual's norm (as k_coarse_tail).
constexpr int P2_TAIL_H = 16;
constexpr int P2_TAIL_NT = 1024;
constexpr int P2_TAIL_MP = P2_TAIL_H + 2;  // mark pitch in LDS

struct P2TailArgs {
  const double* f[4];  // families of level ms at (0, 0)
  int64_t fp;
  P2Out prev, cur;     // level ms
  int N, ms, nlev;
  int its[BATCH_MAX_LEVELS];  // of level ms + k
  double w, hl2[BATCH_MAX_LEVELS];
  DevState* st;
  double* hist;
  const double* partials;
  int count, cycle;
};

__global__ __launch_bounds__(P2_TAIL_NT) void k_p2_tail(P2TailArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_done;
  DevState st = *a.st;
  if (st.done) return;
  const int N = a.N;
  double* fam = reinterpret_cast<double*>(smem);  // per level four families of side 2h
  constexpr int MQ = P2_TAIL_MP * P2_TAIL_MP;
  const int S0 = N >> a.ms;  // side of level ms's families
  auto foff = [&](int k) {  // 4 (S0^2 + (S0/2)^2 + ...) before level k
    int o = 0;
    for (int c = 0; c < k; ++c) o += 4 * (S0 >> c) * (S0 >> c);
    return o;
  };
  // four mark states in turn: this level's pair, the coarser level's pair
  double* X = fam + foff(a.nlev);
  auto marks = [&](int b) {
    return P2Marks{X + b * 4 * MQ, MQ, P2_TAIL_MP};
  };
  for (int i = threadIdx.x; i < 4 * S0 * S0; i += P2_TAIL_NT) {
    const int ls = 31 - __builtin_clz(S0), z = i >> (2 * ls), j = (i >> ls) & (S0 - 1), c = i & (S0 - 1);
    const double* f = z & 2 ? (z & 1 ? a.f[3] : a.f[2]) : (z & 1 ? a.f[1] : a.f[0]);
    fam[i] = f[int64_t(j) * a.fp + c];
  }
  for (int i = threadIdx.x; i < 16 * MQ; i += P2_TAIL_NT) X[i] = 0.0;
  if (a.cycle >= 0) {
    const double s = fin_sum(a.partials, a.count);
    if (threadIdx.x == 0) {
      a.hist[a.cycle] = fin_update(st, s, a.cycle);
      *a.st = st;
      s_done = st.done;
    }
    __syncthreads();
    if (s_done) return;
  }
  __syncthreads();
  for (int k = 1; k < a.nlev; ++k) {
    const int sc = S0 >> k, sf = 2 * sc;
    const double* F = fam + foff(k - 1);
    double* Cc = fam + foff(k);
    const int ls = 31 - __builtin_clz(sc);
    for (int i = threadIdx.x; i < 4 * sc * sc; i += P2_TAIL_NT) {
      const int z = i >> (2 * ls), B = (i >> ls) & (sc - 1), A = i & (sc - 1);
      double v = 0.0;
      if (A > 0 && B > 0) {
        const double* p = F + z * sf * sf + 2 * B * sf + 2 * A;
        auto rs = [&](const double* q) { return fmac(2.0, q[0], q[-1] + q[1]); };
        const double top = rs(p - sf), mid = rs(p), bot = rs(p + sf);
        v = fmac(2.0, mid, top + bot) * 0.0625;
      }
      Cc[i] = v;
    }
    __syncthreads();
  }
  int pb = 0;  // mark states pb (x_{t-1}) and pb + 1 (x_t) of the coarser level; the other pair is free
  int it_above = 0;
  for (int k = a.nlev - 1; k >= 0; --k) {
    const int m = a.ms + k, h = N >> (m + 1), lh = 31 - __builtin_clz(h), sk = S0 >> k;
    const int nb = 2 - pb;  // the free pair
    const double* fk = fam + foff(k);
    // a mark per lane (h is a power of two, 4 h^2 <= 1024 of them) and, in the
    // last lanes, a ghost: place, right-hand side or cell and weights, and the
    // mark's value stay in registers over the iterations
    const int n = threadIdx.x;
    const bool mark = n < 4 * h * h;
    const int mz = mark ? n >> (2 * lh) : 0, mi = 1 + (n & (h - 1)), mj = 1 + ((n >> lh) & (h - 1));
    const int mo = mz * MQ + mj * P2_TAIL_MP + mi;
    const int gn = n - (P2_TAIL_NT - 8 * h);
    const bool gap = ((gn >> lh) & 1) != 0;  // ghosts of the y axis, else of x
    const int gc = 1 + (gn & (h - 1)), gz = gn >= 0 ? gn >> (lh + 1) : 0;
    const int gi = gap ? gc : h + 1, gj = gap ? h + 1 : gc;
    const bool ghost = gn >= 0 && (gi << m) <= N - 1 && (gj << m) <= N - 1;
    const int go = gz * MQ + gj * P2_TAIL_MP + gi;
    double rv = 0.0, v = 0.0, gv = 0.0, gfx = 0.0, gfy = 0.0;
    int g0 = 0;
    if (mark) rv = fk[mz * sk * sk + mj * sk + mi];
    if (ghost) {  // its cell (as p2_interp)
      const int half = N >> 1, px = gi << m, py = gj << m, sx = gz & 1, sy = gz >> 1;
      const bool ox = px >= half, oy = py >= half;
      const int ax = ox ? N - 1 - px : px, ay = oy ? N - 1 - py : py, ix = ax >> m, iy = ay >> m;
      const double inv_l = 1.0 / double(1 << m);
      gfx = double(ax - (ix << m)) * inv_l;
      gfy = double(ay - (iy << m)) * inv_l;
      g0 = (2 * (oy ? 1 - sy : sy) + (ox ? 1 - sx : sx)) * MQ + iy * P2_TAIL_MP + ix;
    }
    double* const xa = X + nb * 4 * MQ;
    double* const xb = xa + 4 * MQ;
    if (k < a.nlev - 1) {  // hand-over from level m + 1 (the coarsest level starts from 0)
      const P2Marks prev = marks(pb + ((it_above & 1) ? 0 : 1)), cur = marks(pb + ((it_above & 1) ? 1 : 0));
      if (mark) v = p2_state(prev, cur, N, m + 1, mz & 1, mz >> 1, mi << m, mj << m);
      if (ghost) gv = p2_state(prev, cur, N, m + 1, gz & 1, gz >> 1, gi << m, gj << m);
      if (mark) xa[mo] = v;
      if (gn >= 0) xa[go] = gv;
      __syncthreads();
    }
    const int it = a.its[k];
    const double hl2 = a.hl2[k];
    double pv = 0.0;
    auto step = [&](const double* in, double* o) {
      pv = v;
      if (mark) {
        const double* p = in + mo;
        v = relax_const<double>(v, (p[-1] + p[1]) + (p[-P2_TAIL_MP] + p[P2_TAIL_MP]), rv, a.w, hl2, 4.0);
        o[mo] = v;
      }
      if (gn >= 0) {
        const double* p = in + g0;
        const double t = lerp(lerp(p[0], p[1], gfx), lerp(p[P2_TAIL_MP], p[P2_TAIL_MP + 1], gfx), gfy);
        o[go] = ghost ? t : 0.0;
      }
      __syncthreads();
    };
    int t = 0;
    for (; t + 2 <= it; t += 2) {
      step(xa, xb);
      step(xb, xa);
    }
    if (t < it) step(xa, xb);
    if (k == 0 && mark) {
      *a.cur.at(mz, mj, mi) = v;
      *a.prev.at(mz, mj, mi) = pv;
    }
    it_above = it;
    pb = nb;
  }
}

// ------------------------------------------------------------ launchers

Lay p2_mark_layout(int N, int m) {
  const int h = N >> (m + 1);
  Lay L;
  L.side = h;
  L.pitch = ((h + 2 + 15) / 16) * 16;
  L.off = 15;  // index 1 of every row starts a 128-byte line
  L.plane = (h + 2) * L.pitch;  // quadrant to quadrant
  L.alloc = ((L.off + 4 * L.plane + 16 + 15) / 16) * 16;  // arrays side by side keep the phase
  return L;
}

static P2Marks p2_in(const double* p, const Lay& l) { return P2Marks{p ? p + l.off : nullptr, l.plane, l.pitch}; }
static P2Out p2_out(double* p, const Lay& l) { return P2Out{p + l.off, l.plane, l.pitch}; }
static dim3 p2_mark_grid(int h) { return dim3((h + 1 + 63) / 64, (h + 1 + 3) / 4, 4); }

hipError_t launch_p2_restrict(const double* r0, const Lay& rl, const double* const* F, const Lay& fl, int N,
                              double* const* Cc, const Lay& cl, const int* done, hipStream_t s) {
  const int nc = cl.side;
  if (r0) {
    if (nc != N / 2 || rl.side != N) return hipErrorInvalidValue;
    const dim3 g((nc + 63) / 64, (nc + 4 * P2R_ROWS - 1) / (4 * P2R_ROWS));
    HOMG_LAUNCH(k_p2_restrict_first, g, dim3(256), s, r0 + rl.off, rl.pitch, Cc[0] + cl.off, Cc[1] + cl.off,
                Cc[2] + cl.off, Cc[3] + cl.off, cl.pitch, N, done);
  }
  if (!F || fl.side != 2 * nc || nc < 2) return hipErrorInvalidValue;
  P2Fams p{};
  for (int z = 0; z < 4; ++z) {
    p.f[z] = F[z] + fl.off;
    p.c[z] = Cc[z] + cl.off;
  }
  const dim3 g((nc - 1 + 63) / 64, (nc - 1 + 3) / 4, 4);
  HOMG_LAUNCH(k_p2_restrict, g, dim3(64, 4), s, p, fl.pitch, cl.pitch, nc, done);
}

hipError_t launch_p2_iter(int N, int m, double omega, const double* in, double* out, const Lay& ml,
                          const double* const* fam, const Lay& fl, const int* done, hipStream_t s) {
  const int h = N >> (m + 1);
  if (m < 1 || h < 1 || ml.side != h || fl.side != (N >> m)) return hipErrorInvalidValue;
  P2Fam4 f{};
  for (int z = 0; z < 4; ++z) f.f[z] = fam[z] + fl.off;
  const double hl = double(1 << m) / double(N - 1);
  HOMG_LAUNCH(k_p2_iter, p2_mark_grid(h), dim3(64, 4), s, p2_in(in, ml), p2_out(out, ml), f, fl.pitch, N, m,
              omega / 4.0, hl * hl, done);
}

hipError_t launch_p2_tile(int N, int m, int it, double omega, int from, const double* sprev, const double* scur,
                          const Lay& sl, const double* e, const Lay& el, double* prev, double* cur, const Lay& ml,
                          const double* const* fam, const Lay& fl, const int* done, hipStream_t s) {
  const int h = N >> (m + 1);
  if (m < 1 || h < 1 || it < 1 || it > P2T_IT || ml.side != h || fl.side != (N >> m) || (from == 0 && !e) ||
      (from > 0 && (!sprev || !scur || sl.side != (N >> (from + 1)))))
    return hipErrorInvalidValue;
  const int64_t lim = int64_t(1) << 31;  // 32-bit offsets inside a quadrant
  if (fl.pitch * fl.side >= lim || ml.plane >= lim || (from > 0 && sl.plane >= lim)) return hipErrorInvalidValue;
  P2TileArgs g{};
  if (from > 0) {
    g.sp = p2_in(sprev, sl);
    g.sc = p2_in(scur, sl);
  } else if (from == 0) {
    g.e = e + el.off;
    g.ep = el.pitch;
  }
  g.from = from;
  g.prev = p2_out(prev, ml);
  g.cur = p2_out(cur, ml);
  for (int z = 0; z < 4; ++z) g.fam.f[z] = fam[z] + fl.off;
  g.fp = fl.pitch;
  g.N = N;
  g.m = m;
  g.it = it;
  g.w = omega / 4.0;
  const double hl = double(1 << m) / double(N - 1);
  g.hl2 = hl * hl;
  g.done = done;
  if (h >= P2T_WIDE) {
    g.nb = (h + 31) / 32;
    HOMG_LAUNCH((k_p2_tile<32, 1024, 2>), dim3(4u * unsigned(g.nb) * unsigned(g.nb)), dim3(1024), s, g);
  }
  g.nb = (h + 15) / 16;
  HOMG_LAUNCH((k_p2_tile<16, 832, 1>), dim3(4u * unsigned(g.nb) * unsigned(g.nb)), dim3(832), s, g);
}

hipError_t launch_p2_write(int N, int m, const double* prev, const double* cur, const Lay& ml, double* en,
                           const Lay& el, double* u, const Lay& ul, const int* done, hipStream_t s) {
  if (m < 1 || ml.side != (N >> (m + 1))) return hipErrorInvalidValue;
  const dim3 g(t2_gx(N), t2_gy(N, P2_ROWS));
  HOMG_LAUNCH(k_p2_write, g, dim3(256), s, p2_in(prev, ml), p2_in(cur, ml), m, N, en ? en + el.off : nullptr, el.pitch,
              u ? u + ul.off : nullptr, ul.pitch, done);
}

bool p2_tail_fits(int N, int ms) { return (N >> (ms + 1)) <= P2_TAIL_H; }

hipError_t launch_p2_tail(int N, int ms, int nlev, const int* its, double omega, const double* const* fam,
                          const Lay& fl, double* prev, double* cur, const Lay& ml, DevState* st, double* hist,
                          const double* partials, int count, int cycle, hipStream_t s) {
  if (ms < 1 || nlev < 1 || nlev > BATCH_MAX_LEVELS || !p2_tail_fits(N, ms) || (N >> (ms + nlev)) < 1 ||
      fl.side != (N >> ms) || ml.side != (N >> (ms + 1)))
    return hipErrorInvalidValue;
  P2TailArgs a{};
  size_t nodes = 0;
  for (int k = 0; k < nlev; ++k) {
    const double hl = double(1 << (ms + k)) / double(N - 1);
    a.its[k] = its[k];
    a.hl2[k] = hl * hl;
    nodes += 4 * size_t(N >> (ms + k)) * size_t(N >> (ms + k));
  }
  for (int z = 0; z < 4; ++z) a.f[z] = fam[z] + fl.off;
  a.fp = fl.pitch;
  a.prev = p2_out(prev, ml);
  a.cur = p2_out(cur, ml);
  a.N = N;
  a.ms = ms;
  a.nlev = nlev;
  a.w = omega / 4.0;
  a.st = st;
  a.hist = hist;
  a.partials = partials;
  a.count = count;
  a.cycle = partials ? cycle : -1;
  const size_t lds = (nodes + 16 * P2_TAIL_MP * P2_TAIL_MP) * sizeof(double);
  hipError_t e = allow_lds(k_p2_tail, lds);
  if (e != hipSuccess) return e;
  HOMG_LAUNCH_SMEM(k_p2_tail, dim3(1), dim3(P2_TAIL_NT), lds, s, a);
}

}  // namespace homg
