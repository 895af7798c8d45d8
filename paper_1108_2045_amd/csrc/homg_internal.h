// homg_internal.h -- declarations shared by the C-ABI driver (homg_capi.cpp)
// and the HIP kernels (homg_kernels.hip).  Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <vector>

struct homg_ctx;

namespace homg {

enum Prec { PREC_F64 = 0, PREC_F32 = 1, PREC_BF16 = 2 };

inline int prec_bytes(int p) { return p == PREC_F64 ? 8 : (p == PREC_F32 ? 4 : 2); }

// Layout of one d-dimensional array of side `side`, in elements.  Node
// (k,j,i) sits at base + off + k*plane + j*pitch + i.  Internal arrays are
// padded so that node (.,.,1) -- the first interior node of every row --
// starts a 128-byte line and every row starts on the same phase; dense
// arrays (the caller's) have off = 0, pitch = side, plane = side*side.
struct Lay {
  int side = 0;
  int64_t off = 0, pitch = 0, plane = 0, alloc = 0;
};

Lay dense_layout(int d, int side);
Lay padded_layout(int d, int side, int elem_bytes);

// Per-solve device state (one per handle).
struct DevState {
  int done;      // 0 running, 1 converged, 2 non-finite norm
  int cycles;    // last cycle whose residual was recorded
  int stop_on_tol;
  int pad;
  double fnorm;  // ||f||_2 over interior nodes (1 if f == 0)
  double tol;
};

enum SweepMode { SW_ZERO_OLD = 1, SW_ACCUM = 2, SW_TBLOCK = 8 };

// Upper bound on the number of per-block partial sums written by the
// residual launches for a grid of side n, and launch_residual's number.
int partials_bound(int d, int n);
int residual_partials(int d, int n);

// r0 = f - A u (FP64) stored in the precision `prec`; per-block sums of r^2
// -> partials (their number in *count) and, given fpart, of f^2 -> fpart.
// `a` (nullable) is the nodal coefficient for the diffusion operator, in the
// layout al.
hipError_t launch_residual(int prec, int d, int n, const double* u, const Lay& ul,
                           const double* f, const Lay& fl, const double* a, const Lay& al,
                           void* r0, const Lay& rl, double* partials, int* count,
                           const int* done, hipStream_t s, double* fpart = nullptr);
// 2D (n >= 5): the residual of launch_residual and, in the same
// pass, its full-weighting restriction to level 1 (rc, layout cl of side
// (n-1)/2+1), equal bit for bit to launch_restrict applied to the stored r0.
// Per-wave sums of r^2 (their number in *count) and, given fpart, of f^2.
hipError_t launch_residual_restrict_2d(int prec, int n, const double* u, const Lay& ul,
                                       const double* f, const Lay& fl, const double* a, const Lay& al, void* r0,
                                       const Lay& rl, void* rc, const Lay& cl, double* partials, int* count,
                                       const int* done, hipStream_t s, double* fpart = nullptr);
// Sums `count` partials in a fixed order: history[cycle] = sqrt(sum)/fnorm,
// and `done` is updated (nothing if it is set).  Given hst / hhist (pinned
// host memory), the state and history[0 .. the last recorded cycle] are
// stored there as well.  _first: a solve's first residual, with its sums of
// f^2 -- the state starts here (fnorm, tol, stop_on_tol), as cycle 0.
hipError_t launch_finalize(const double* partials, int count, DevState* st, double* history,
                           int cycle, hipStream_t s, DevState* hst = nullptr, double* hhist = nullptr);
hipError_t launch_finalize_first(const double* partials, const double* fpart, int count, double tol,
                                 int stop_on_tol, DevState* st, double* history, hipStream_t s,
                                 DevState* hst = nullptr, double* hhist = nullptr);
// Normalised L1 error (Sec. 4, discrete): *out (device) = sum |uref - v| /
// sum |uref| over all n^d nodes, v = u + e (e: internal iterate of type
// prec, layout el) or v = u when e is null; uref and u dense FP64.  part:
// l1_partials() doubles of workspace.
int l1_partials();
hipError_t launch_l1(int prec, int d, int n, const double* uref, const double* u, const void* e,
                     const Lay& el, double* part, double* out, hipStream_t s);
// One full-weighting restriction: fine level (side nf) -> coarse (side (nf-1)/2+1).
hipError_t launch_restrict(int prec, int d, const void* rf, const Lay& fl, void* rc,
                           const Lay& cl, const int* done, hipStream_t s);
// P consecutive restrictions r_a -> ... -> r_{a+P} in one launch (r[k],
// l[k]: the array and layout of level a + k, k = 0 .. P): the same bits as
// P launch_restrict calls.  Workgroups own blocks of B nodes per axis of
// level a + P; restrict_multi_lds: the LDS bytes that needs.
constexpr int MR_MAX = 6;
size_t restrict_multi_lds(int prec, int d, int P, int B);
// The same for the families of a power-of-two grid: fam[4 k + q] is family q's
// array of level a + k, l[k] its layout.
hipError_t launch_p2_restrict_multi(int P, int B, double* const* fam, const Lay* l, const int* done, hipStream_t s);
hipError_t launch_restrict_multi(int prec, int d, int P, int B, void* const* r, const Lay* l, const int* done,
                                 hipStream_t s);
// One whole-grid relax+interpolate iteration at level m.  eo/en: fine
// arrays (layout el); rm: compact level-m residual (layout rl); am: compact
// level-m nodal coefficient (FP64, layout al) or null; mode: SweepMode bits;
// with SW_ACCUM the iterate is added to u (FP64, layout ul) instead of
// being stored in en.  compact: a level-0 iteration on the compact lattice
// of a coarse level (same arithmetic, a kernel symbol of its own).
hipError_t launch_sweep(int prec, int d, int n, int m, double omega, const void* eo, void* en,
                        const Lay& el, const void* rm, const Lay& rl, const double* am,
                        const Lay& al, double* u, const Lay& ul, int mode, const int* done,
                        hipStream_t s, bool compact = false);
// Level 0 of a 2D constant-coefficient grid: `it` (<= TB_MAX_IT) iterations
// in one pass (temporal blocking), equal bit for bit to `it` launch_sweep
// calls; reads e (unless zero) and r once, writes en or adds into u once.
// A wave walks a band of `len` rows (0: tb_band's choice).  Short bands
// re-read more halo rows (from L2) but put more waves in flight: tb_band
// returns the longest band (64, 32, 16 or 8 rows) that still gives
// TB_MIN_WAVES waves, else 4 (measured on MI355X, FP64: the pass beats the
// single-iteration kernels from 129^2 up, 1.4-2.8x; on the small lattices
// of a 4097^2 solve, 4-row bands took 10 -> 7.6 us per pass at 257^2).
constexpr int TB_MAX_IT = 4;
constexpr int TB_MIN_WAVES = 4096;
__host__ __device__ inline int tb_waves(int n, int it, int len) {
  const int valid = 64 - 2 * it;
  return ((n - 2 + valid - 1) / valid) * ((n - 2 + len - 1) / len);
}
// Workgroups of a pass: each takes one column tile on four consecutive bands
// (one wave per band), so its four waves write different rows.
__host__ __device__ inline int tb_blocks(int n, int it, int len) {
  const int valid = 64 - 2 * it;
  return ((n - 2 + valid - 1) / valid) * ((n - 2 + 4 * len - 1) / (4 * len));
}
int tb_band(int n, int it);
// A coarse level's final compact state (layout cl, side (n-1)/2+1 for a
// pass over side n): x_it in cur and x_{it-1} in prev (unread when
// zero_old: x_{it-1} = 0).  A pass given one -- level 0 after level 1, or
// the compact lattice of level m after level m + 1, which sits in it the
// same way -- takes its input iterate from it: lattice nodes of the
// coarser level x_it, every other interior node the multilinear
// interpolant of x_{it-1}, exactly as the coarser level's whole-grid write
// (or hand-over) would have stored them, instead of reading eo.
struct L1State {
  const void* prev = nullptr;
  const void* cur = nullptr;
  Lay cl;
  bool zero_old = false;
};
hipError_t launch_sweep_2d_l0_tb(int prec, int n, int it, double omega, const void* eo, void* en,
                                 const Lay& el, const void* rm, const Lay& rl, double* u,
                                 const Lay& ul, bool zero, bool accum, const int* done, hipStream_t s,
                                 int len = 0, const L1State* l1 = nullptr);
// 3D lattice of side n (Laplacian, damped Jacobi): it (<= LT_MAX_IT)
// iterations in one launch, blocks of 8^3 owned nodes iterating with a halo
// of `it` nodes in LDS.  x_0: 0 (zero), the array xo, or the next coarser
// level's state (l1); x_it into xn and, if given, x_{it-1} into xprev (layout
// cl; none may alias another), or -- u given, xn and xprev null, the last
// pass of level 0 -- x_it, unrounded, added into u (layout ul).
// lattice_3d_tiled_lds: its LDS bytes.
constexpr int LT_MAX_IT = 4;
constexpr int LT_MAX_SIDE = 65;  // the solver uses it on lattices up to this side
size_t lattice_3d_tiled_lds(int prec, int it);
hipError_t launch_lattice_3d_tiled(int prec, int n, int it, double omega, const void* xo, void* xn, void* xprev,
                                   const Lay& cl, const void* rm, const Lay& rl, bool zero, const L1State* l1,
                                   const int* done, hipStream_t s, double* u = nullptr, const Lay& ul = Lay());
// The same on a 2D lattice (blocks of 24^2 owned nodes); a: the lattice's
// nodal coefficient (layout al), or null for the Laplacian.
constexpr int LT2_MAX_SIDE = 513;  // the solver uses it on Laplacian lattices up to this side,
constexpr int LT2_MAX_L0 = 257;    // on level 0 up to this one, and with a coefficient on all
hipError_t launch_lattice_2d_tiled(int prec, int n, int it, double omega, const void* xo, void* xn, void* xprev,
                                   const Lay& cl, const void* rm, const Lay& rl, bool zero, const L1State* l1,
                                   const int* done, hipStream_t s, double* u = nullptr, const Lay& ul = Lay(),
                                   const double* a = nullptr, const Lay& al = Lay());
// The same on the compact lattice of a coarse level (side nm): x_it into en
// and, when eprev is not null, x_{it-1} into eprev (layout cl); l1: x_0
// from the next coarser level's state.
hipError_t launch_lattice_2d_tb(int prec, int nm, int it, double omega, const void* eo, void* en,
                                void* eprev, const Lay& cl, const void* rm, const Lay& rl, bool zero,
                                const int* done, hipStream_t s, int len = 0, const L1State* l1 = nullptr);
// 3D (7-point Laplacian) counterpart: `it` (<= TB3_MAX_IT) iterations in one
// pass over the level-0 grid or (compact) a coarse level's lattice of side
// n (layout el for eo, en, eprev; r in rl); accum (level 0 only): add x_it
// into u (dense FP64, ul) instead of storing it; eprev (compact only): also
// store x_{it-1}; l1: the input iterate from the next coarser level's
// state (not with zero).  A block walks
// `len` planes (0: tb3_band's choice: the longest of 32, 16, 8 planes that
// still gives TB3_MIN_BLOCKS blocks, else 4; at 257^3 that is 16 planes in
// 1760 blocks, measured 5% faster per pass than 32 planes in 880 -- 119
// against 126 us for the pass that adds into u -- and at 513^3 level 0
// keeps 32 planes).
constexpr int TB3_MAX_IT = 2;
constexpr int TB3_MIN_BLOCKS = 1536;
int tb3_blocks(int n, int it, int len);
int tb3_band(int n, int it);
hipError_t launch_tb_3d(int prec, int n, int it, double omega, const void* eo, void* en, void* eprev,
                        const Lay& el, const void* rm, const Lay& rl, double* u, const Lay& ul,
                        bool zero, bool accum, bool compact, const int* done, hipStream_t s, int len = 0,
                        const L1State* l1 = nullptr);
// Convert between a dense FP64 array and an internal array of `prec`.
hipError_t launch_pack(int prec, int d, const double* src, const Lay& sl, void* dst,
                       const Lay& dl, hipStream_t s);
hipError_t launch_unpack(int prec, int d, const void* src, const Lay& sl, double* dst,
                         const Lay& dl, hipStream_t s);
// Copy an FP64 array between layouts, sampling every `stride`-th node of the
// source (stride 1: plain copy; stride l: the level-l lattice).
hipError_t launch_sample(int d, const double* src, const Lay& sl, int stride, double* dst,
                         const Lay& dl, hipStream_t s);

// Level-blocked path (same results as one launch per iteration):
// x_0 = the whole grid sampled on the level-l lattice (all compact nodes).
hipError_t launch_gather(int prec, int d, const void* src, const Lay& sl, int l, void* dst,
                         const Lay& dl, const int* done, hipStream_t s);
// LDS bytes the single-workgroup lattice kernel needs for a compact side nm.
size_t lattice_small_lds(int prec, int d, int nm, bool var);
// All `it` iterations of a level on a compact lattice of side nm held by one
// workgroup; x_0 gathered from e (layout el, stride l) unless zero; writes
// x_{it-1} to xprev and x_it to xcur (compact layout cl).
hipError_t launch_lattice_small(int prec, int d, int nm, int l, int it, double omega, bool zero,
                                const void* e, const Lay& el, const void* rm, const Lay& rl,
                                const double* am, const Lay& al, void* xprev, void* xcur,
                                const Lay& cl, const int* done, hipStream_t s);
// One-workgroup kernels (chained execution, damped Jacobi): levels ms .. ms +
// nlev - 1 of a schedule that starts at the coarsest of them and descends
// one level at a time, its[k] iterations of level ms + k, on a finest side
// of at most tail_max_side(d) (its nodes in registers, four per lane).
// coarse_tail_lds: the LDS bytes.  top64 (FP32/BF16 cycles): the coarsest
// level in FP64 (its restriction, iterates and arithmetic), rounded to the
// storage type only for the hand-over.  faces (2D, or null): the factors of
// level ms and the coarser levels behind it, as launch_faces leaves them.
//
// launch_coarse_tail: restricts r_ms (side nms, layout rl) and leaves level
// ms's final x_it and x_{it-1} in scur and sprev (layout sl, interior nodes)
// for a next pass that interpolates them itself or the hand-over kernel.
// Does nothing if st->done; given partials, it first records the relative
// residual of `cycle` from them, as launch_finalize, and stops there if that
// ends the solve.
// launch_small_solve: cycles c0 .. c1 of a solve of A u = f on a grid of side
// n (f, u dense) from the residual to the update of u, with the residual
// norms in hist and hhist and the final state in st and hst; c0 = 0 starts
// the state.  rr: the norms summed as launch_residual_restrict_2d's, else as
// launch_residual's.
constexpr int tail_max_side(int d) { return d == 2 ? 65 : 17; }
// launch_faces: per level k < levels (sides at most tail_max_side(2), one half
// of the one before) of a variable coefficient three arrays of side^2 values,
// one level after the other: the face coefficients west and south of each node
// and omega / the sum of its four, in the cycle's arithmetic (wide_last: the
// last level's in FP64).
hipError_t launch_faces(int prec, int levels, const double* const* a, const Lay* al, bool wide_last, double omega,
                        double* out, hipStream_t s);
size_t coarse_tail_lds(int prec, int d, int nms, int nlev, bool top64, bool var, bool solve);
hipError_t launch_coarse_tail(int prec, int d, int nms, int nlev, const int* its, double omega,
                              const double* faces, const void* rms, const Lay& rl, void* sprev, void* scur, const Lay& sl,
                              bool top64, DevState* st, double* hist, const double* partials, int count, int cycle,
                              hipStream_t s);
hipError_t launch_small_solve(int prec, int d, int n, int nlev, const int* its, double omega,
                              const double* faces, const double* f, double* u, bool top64, bool rr, int c0, int c1,
                              double tol, int stop, DevState* st, double* hist, DevState* hst, double* hhist,
                              hipStream_t s);
// FP64 coarsest level of a reduced-precision cycle: the restriction to it
// (input in the storage type of prec, widened exactly, FP64 sums and
// output); the exact widening of the level-l lattice of an array in the
// storage type into an FP64 compact array (every node of dl.side); and the
// rounding of an FP64 compact array to the storage type (to FP32, then BF16).
hipError_t launch_restrict_to_f64(int prec, int d, const void* rf, const Lay& fl, double* rc,
                                  const Lay& cl, const int* done, hipStream_t s);
hipError_t launch_widen(int prec, int d, const void* src, const Lay& sl, int l, double* dst,
                        const Lay& dl, const int* done, hipStream_t s);
hipError_t launch_narrow(int prec, int d, const double* src, const Lay& sl, void* dst, const Lay& dl,
                         const int* done, hipStream_t s);
// LDS bytes of the whole-grid pass of level m.
size_t level_write_lds(int prec, int d, int n, int m);
// Whole-grid pass of level m from compact x_{it-1} (xprev) and x_it (xcur):
// mode SW_ZERO_OLD = x_{it-1} is 0, SW_ACCUM = add into u instead of storing.
hipError_t launch_level_write(int prec, int d, int n, int m, const void* xprev, const void* xcur,
                              const Lay& cl, void* en, const Lay& el, double* u, const Lay& ul,
                              int mode, const int* done, hipStream_t s);
// Chained path: the state the level-m write would produce, sampled at the
// interior nodes of the level-mt lattice into that level's compact array
// (layout tl); zero_old: x_{it-1} = 0.
hipError_t launch_level_transfer(int prec, int d, int m, const void* xprev, const void* xcur,
                                 const Lay& cl, int mt, void* dst, const Lay& tl, bool zero_old,
                                 const int* done, hipStream_t s);
// ---- power-of-two grids (Sec. 3; 2D Laplacian, FP64), N = 2^k nodes per side
// One level of the four restriction families (q = 2 sy + sx): level 1 from the
// whole-grid r_0, or (r0 null) level j from level j - 1 (compact, side
// 2 * cl.side).
hipError_t launch_p2_restrict(const double* r0, const Lay& rl, const double* const* F, const Lay& fl, int N,
                              double* const* Cc, const Lay& cl, const int* done, hipStream_t s);
// Compact form (the same bits as the whole-grid iterations): the marks of
// level m, four quadrants of (h + 2)^2 values, h = N / 2^(m+1) = layout side,
// quadrant to quadrant `plane` apart.
//   launch_p2_iter: one iteration; the final pair of a level is the state
//     before and after its last one;
//   launch_p2_tile: the first it <= P2T_IT iterations of a level in one
//     launch.  They start from 0 (from < 0), the whole grid e (from = 0) or
//     the final pair sprev, scur of level `from` (layout sl); leaves x_{it-1}
//     in prev and x_it with its ghosts in cur;
//   launch_p2_write: the whole grid after a level, into en or (u given)
//     added into u;
//   launch_p2_tail: levels ms + nlev - 1 .. ms from 0 in one workgroup
//     (p2_tail_fits), with the norm of the residual of `cycle` reduced first
//     as launch_coarse_tail does.
Lay p2_mark_layout(int N, int m);
constexpr int P2T_IT = 4;
hipError_t launch_p2_tile(int N, int m, int it, double omega, int from, const double* sprev, const double* scur,
                          const Lay& sl, const double* e, const Lay& el, double* prev, double* cur, const Lay& ml,
                          const double* const* fam, const Lay& fl, const int* done, hipStream_t s);
hipError_t launch_p2_iter(int N, int m, double omega, const double* in, double* out, const Lay& ml,
                          const double* const* fam, const Lay& fl, const int* done, hipStream_t s);
hipError_t launch_p2_write(int N, int m, const double* prev, const double* cur, const Lay& ml, double* en,
                           const Lay& el, double* u, const Lay& ul, const int* done, hipStream_t s);
// it <= TB_MAX_IT iterations of level 0 whose first iterate is level 1's final
// pair, into en or (u given) added into u (homg_kernels.hip).
hipError_t launch_p2_l0(int N, int it, double omega, const double* prev, const double* cur, const Lay& ml, double* en,
                        const Lay& el, const double* r, const Lay& rl, double* u, const Lay& ul, const int* done,
                        hipStream_t s);
bool p2_tail_fits(int N, int ms);
hipError_t launch_p2_tail(int N, int ms, int nlev, const int* its, double omega, const double* const* fam,
                          const Lay& fl, double* prev, double* cur, const Lay& ml, DevState* st, double* hist,
                          const double* partials, int count, int cycle, hipStream_t s);
// One whole-grid iteration at level m >= 1; fam[q] (q = 2 sy + sx) is the
// level-m family array of quadrant q (layout fl, side N >> m); mode: SW_ZERO_OLD
// / SW_ACCUM (add into u, layout ul, instead of storing en).
hipError_t launch_p2_sweep(int N, int m, double omega, const double* eo, double* en, const Lay& el,
                           const double* const* fam, const Lay& fl, double* u, const Lay& ul, int mode,
                           const int* done, hipStream_t s);

constexpr int BATCH_MAX_LEVELS = 16;

// ---- batched solver (2D, constant coefficient): one launch per stage for
// all problems.  Every launch takes a list of {descriptor, block} pairs, one
// per workgroup; st, f, u, hist are indexed by the problem.
struct BatchResidual {  // residual + first restriction (n >= 5)
  void* r;
  void* rc;
  int64_t rp, cp;
  double* partials;  // `count` sums of r^2 and of f^2
  double* fpart;
  double inv_h2;
  int prob, n, len, count;
};
struct BatchRestrict {  // one restriction to side nc
  const void* rf;
  void* rc;
  int64_t fp, cp;
  int prob, nc, len, pad;
};
struct BatchPass {  // iterations of one lattice (or level 0) of one problem
  const void* xo;   // input iterate, or the coarser level's state in l1_*
  void* xn;
  void* xp;
  const void* r;
  const void* l1_prev;
  const void* l1_cur;
  int64_t cp, rp, l1_pitch;
  double hl2;
  int prob, n, len, accum;  // len: blocks per axis (tiled), rows per band (walking)
};
struct BatchState {  // what the host reads of a problem
  int done, cycles;
  double rel, prev;  // relative residual after the last two cycles
};
int default_walk_len(int d, int n);
int batch_residual_waves(int n, int len);
int batch_tiled_side(int n);
int batch_restrict_tiles(int nc, int len);
size_t batch_multi_bytes();
// Fills a multi-level restriction descriptor (see launch_restrict_multi);
// returns its number of blocks.
int batch_multi_fill(int prec, void* dst, int prob, int P, int B, void* const* r, const Lay* l);
hipError_t launch_batch_residual(int prec, const BatchResidual* res, const int2* tiles, int count, bool norm,
                                 const double* const* f, double* const* u, const DevState* st, hipStream_t s);
hipError_t launch_batch_restrict(int prec, const BatchRestrict* rs, const int2* tiles, int count, const DevState* st,
                                 hipStream_t s);
hipError_t launch_batch_restrict_multi(int prec, const void* ms, const int2* tiles, int count, size_t lds,
                                       const DevState* st, hipStream_t s);
// it iterations: lat, from the coarser level's state; kind: BATCH_TILED
// (into u by BatchPass), or a walking pass that stores x_it, adds it into u,
// or stores x_it and x_{it-1}.
enum { BATCH_TILED = -1, BATCH_WALK = 0, BATCH_WALK_ACCUM = 1, BATCH_WALK_PREV = 2 };
hipError_t launch_batch_pass(int prec, const BatchPass* ps, const int2* tiles, int count, int it, bool lat, int kind,
                             double omega, const DevState* st, double* const* u, hipStream_t s);
hipError_t launch_batch_finalize(const BatchResidual* res, int count, DevState* st, double* const* hist, int cycle,
                                 bool first, double tol, hipStream_t s);
hipError_t launch_batch_publish(int P, const DevState* st, const double* const* hist, BatchState* out, hipStream_t s);
// One-workgroup problems and coarse tails (homg_tail.hip): descriptors
// filled on the host, one workgroup each.  Tails reduce the norm of the
// residual of `cycle` first (cycle >= 0); whole solves run cycles c0 .. c1.
// All descriptors of a launch share top64; lds: the largest of theirs.
size_t batch_tail_bytes(int prec);
void batch_tail_fill(int prec, void* dst, int n_level, int nlev, const int* its, double omega, const void* r,
                     int64_t rp, void* sprev, void* scur, int64_t sp, bool top64, DevState* st, double* hist,
                     const double* partials, int count);
void batch_small_fill(int prec, void* dst, int n, int nlev, const int* its, double omega, bool top64, bool rr, int prob,
                      DevState* st, double* hist);
hipError_t launch_batch_tails(int prec, bool top64, const void* args, int count, size_t lds, int cycle, hipStream_t s);
hipError_t launch_batch_small(int prec, bool top64, const void* args, int count, size_t lds, const double* const* f,
                              double* const* u, double tol, int c0, int c1, hipStream_t s);

// ---- learned lattice smoother (2D)
constexpr int HID = 16;                 // hidden channels
constexpr int NW1 = HID * 3 * 9;        // first layer: 16 x 3 channels x 3x3 taps
constexpr int NW = NW1 + HID * 9;       // + second layer: 16 x 3x3 taps = 576 weights
constexpr int TRAIN_MAX_ROWS = 1024;    // workgroups (partial-sum rows) of one backward launch
constexpr int ENERGY_MAX_PARTS = 1024;  // workgroups of one energy launch

// One learned relaxation of every interior node of a compact lattice of
// side nm and spacing hl: xo = xi + y.  Layouts: xl for xi/xo, rl for r,
// al for the FP64 nodal coefficient a (null: constant coefficient); mode
// SW_ZERO_OLD (xi = 0, not read) / SW_ACCUM (u += xi + y instead of the store).
// w: the 576 weights as FP32 values.
// Lattices of side <= LEARNED_SMALL_NM: all `it` learned relaxations in one
// workgroup (x_0 from e with stride l, or 0 when zero); writes x_{it-1} to
// xprev and x_it to xcur.
constexpr int LEARNED_SMALL_NM = 16;
hipError_t launch_learned_small(int prec, int nm, int l, int it, double hl, bool zero, const void* e,
                                const Lay& el, const void* r, const Lay& rl, const double* a,
                                const Lay& al, void* xprev, void* xcur, const Lay& cl,
                                const float* w, const int* done, hipStream_t s);
hipError_t launch_learned_iter(int prec, int nm, double hl, const void* xi, const Lay& xl,
                               void* xo, const void* r, const Lay& rl, const double* a,
                               const Lay& al, double* u, const Lay& ul, const float* w, int mode,
                               const int* done, hipStream_t s);
// Chained execution (homg_learned_tiles.hip).  Up to LEARNED_TILE_IT
// relaxations of a lattice of side n in one launch: x_0 is 0, the array xo, or
// the next coarser level's state l1; x_it into xn and x_{it-1} into xp
// (nullable; layout cl, none may alias xo), or u += x_it.
constexpr int LEARNED_TILE_IT = 4;
constexpr int LEARNED_DEEP_SIDE = 129;  // largest side that takes so many (two above)
hipError_t launch_learned_tiles(int prec, int n, int it, double hl, const void* xo, void* xn, void* xp, const Lay& cl,
                                const void* r, const Lay& rl, const double* a, const Lay& al, double* u, const Lay& ul,
                                const L1State* l1, const float* w, const int* done, hipStream_t s);
// The leading coarse levels of the schedule, the finest of side n <=
// LEARNED_TAIL_SIDE, in one workgroup (as launch_coarse_tail: restrictions
// from r, its[k] iterations of the level 2^k times coarser, the finest level's
// final pair into sprev and scur, the previous cycle's norm first).
constexpr int LEARNED_TAIL_SIDE = 33;
hipError_t launch_learned_tail(int prec, int n, int nlev, const int* its, const double* a, const Lay& al, const void* r,
                               const Lay& rl, void* sprev, void* scur, const Lay& sl, const float* w, DevState* st,
                               double* hist, const double* partials, int count, int cycle, hipStream_t s);
size_t learned_tiles_lds(int prec);
// Training on dense FP32 compact arrays of side nm.  fwd: z = delta - y (y if
// delta is null).  bwd: per-workgroup partial sums of dL/dw (576) and E(z)
// into part[j * pstride + row], rows = train_bwd_rows(nm); e0 = &E(delta).
hipError_t launch_train_fwd(int nm, float hl2, const float* x, const float* r, const float* a,
                            const float* delta, float* z, const float* w, hipStream_t s);
int train_bwd_rows(int nm);
hipError_t launch_train_bwd(int nm, float hl2, const float* x, const float* r, const float* a,
                            const float* z, const double* e0, const float* w, float* part,
                            int64_t pstride, hipStream_t s);
// out[j] = sum of part[j][0..rows) (FP64, fixed order), j = 0..NW; given
// energy, the last of them there too.
hipError_t launch_train_reduce(const float* part, int64_t pstride, int rows, double* out,
                               hipStream_t s, double* energy = nullptr);
hipError_t launch_train_adam(const double* sums, int batch, const double* e0s, const int* idx,
                             float* theta, float* m1, float* m2, uint16_t* wbf, float* w32,
                             int step, double lr, double beta1, double beta2, double eps,
                             double* loss, hipStream_t s);
// *out = E(v) = v^T A v over interior nodes (part: ENERGY_MAX_PARTS doubles).
hipError_t launch_energy(const float* v, const float* a, int nm, double* part, double* out,
                         hipStream_t s);
hipError_t launch_round_weights(const float* src, uint16_t* wbf, float* w32, hipStream_t s);
// dst (dense FP32, side nm) = src on the l-lattice, or sub - src when sub != null.
hipError_t launch_lattice_f32(const double* src, int64_t sp, int l, const double* sub, int64_t bp,
                              int nm, float* dst, hipStream_t s);

hipError_t launch_add_dense(double* v, const double* e, int64_t count, hipStream_t s);

// What the trainer needs to know about a solver handle.
struct CtxView {
  int d = 0, n = 0, levels = 0, stencil = 0, prec = 0, has_coef = 0, smoother = 0, pow2 = 0;
  double fallback_ratio = 1.0;
  std::vector<int> sched;  // (level, iterations) pairs
};
void ctx_view(const homg_ctx* h, CtxView* v);
// The handle's level-m nodal coefficient as a dense FP64 array (side (n-1)/2^m + 1).
hipError_t ctx_level_coefficient(const homg_ctx* h, int m, double* dense, hipStream_t s);

// Record the text of the calling thread's last error (homg_last_error(NULL)).
void set_last_error(const char* msg);

// Start/stop events stamped on the next launch of this thread (null: none).
void set_launch_events(hipEvent_t start, hipEvent_t stop);
void current_launch_events(hipEvent_t* start, hipEvent_t* stop);

}  // namespace homg
