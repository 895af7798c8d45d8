// homg_batch.cpp -- batched HOMG solver: C ABI, workspace, stage lists.
//
// Many independent 2D problems of uneven size advance together, cycle by
// cycle of their own MFMG sequence (Sec. 2 of arXiv:1108.2045): one launch
// per stage of the cycle for all problems that have it -- residual with the
// first restriction, the rest of the restriction chain, the coarse tails
// (one workgroup per problem), the iterations of each lattice level, level 0
// -- each workgroup taking its {problem, block} from a list made once per
// handle (again when a tile shape or pass depth changes).  The stages are
// the single-problem solver's, block for block.  Problems of side up to
// tail_max_side are solved whole by one workgroup each, in one launch.
// Convergence is decided on the device; a problem that is done returns at
// the start of every later launch.  The host reads the states after a few
// cycles and sizes the next batch of cycles from the slowest problem.
// Aligned at their ends the sequences of problems of different depth share
// their launches: side 65 .. 1025 takes 9 launches a cycle (three
// restrictions, the tails, three lattice levels, level 0, the residual).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/homg.h"
#include "homg_internal.h"

using namespace homg;

namespace {

// One launch of the iteration stages.
struct PassGroup {
  int it, kind;
  bool lat;
  int desc;          // its first descriptor (the tiles count from it)
  int first, count;  // its workgroups in the tile list
};
struct TileRange {
  int first = 0, count = 0;
};

// One problem's workspace (solved in stages: side > tail_max_side).
struct Problem {
  int n = 0, levels = 0, ms = 0;  // ms: finest level of the coarse tail
  Lay el, rl[BATCH_MAX_LEVELS];
  char* r[BATCH_MAX_LEVELS] = {};  // right-hand sides of levels 0 .. ms (arrays as allocated)
  char* x[BATCH_MAX_LEVELS][3] = {};  // levels 1 .. ms: iterate pair; below ms also x_{it-1}
  char* e[2] = {nullptr, nullptr};    // level 0's iterates, if it may take several passes
  double* partials = nullptr;
};

}  // namespace

struct homg_batch_ctx {
  int count = 0, prec = 0, max_i = 4, max_cycles = 200;
  double omega = 0.8;
  int def_rows = 16;              // default rows per tile (default_rows)
  std::vector<int> sides;
  std::map<int, int> tile_rows;   // side -> rows per tile (absent: default)
  std::map<int, int> pass_iters;  // side -> iterations per level-0 pass (absent: TB_MAX_IT)
  std::vector<Problem> probs;
  std::vector<int> big, small[2];  // problems solved in stages; by one workgroup (small[1]: FP64 coarsest level)
  // stage lists; dirty: to be made (again) before the next solve, on whose
  // stream they go up from lists (kept while the copy may be in flight)
  bool dirty = true;
  std::vector<char> lists;
  std::vector<PassGroup> passes;   // in launch order
  std::vector<TileRange> restricts;  // restriction a -> a + 1 at [a]
  TileRange residual, multi;
  size_t multi_lds = 0, tail_lds = 0, small_lds[2] = {0, 0};
  size_t o_res = 0, o_rs = 0, o_multi = 0, o_pass = 0, o_tail = 0, o_small[2] = {0, 0}, o_tiles = 0;  // in plan
  char* plan = nullptr;
  size_t plan_bytes = 0;  // enough for any tile rows and pass iterations (plan_bound)
  // per-call inputs and results
  void** h_ptrs = nullptr;  // f, then u (pinned), and their device copy
  void** d_ptrs = nullptr;
  BatchState* h_state = nullptr;  // pinned
  DevState* d_st = nullptr;
  double** d_hist = nullptr;      // per problem
  std::vector<double*> hist;
  void* arena = nullptr;
  int device = 0;
  std::string err;
};

namespace {

homg_status bfail(homg_batch_ctx* b, homg_status s, const std::string& msg) {
  set_last_error(msg.c_str());
  if (b) b->err = msg;
  return s;
}

#define BHIP(b, call)                                                                     \
  do {                                                                                    \
    hipError_t e_ = (call);                                                               \
    if (e_ != hipSuccess)                                                                 \
      return bfail(b, HOMG_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_));   \
  } while (0)

int side_k(int64_t n) {
  if (n < 3) return -1;
  int k = 0;
  while ((int64_t(1) << (k + 1)) + 1 <= n) ++k;
  return ((int64_t(1) << k) + 1 == n) ? k : -1;
}

void free_batch(homg_batch_ctx* b) {
  if (!b) return;
  (void)hipFree(b->arena);
  (void)hipFree(b->plan);
  (void)hipFree(b->d_ptrs);
  (void)hipFree(b->d_st);
  (void)hipFree(b->d_hist);
  if (b->h_ptrs) (void)hipHostFree(b->h_ptrs);
  if (b->h_state) (void)hipHostFree(b->h_state);
  delete b;
}

int level_iters(const homg_batch_ctx* b, int levels, int m) {
  return std::min(1 << std::min(levels - m, 30), b->max_i);
}

// Default rows per tile: 16, halved while the batch's residual pass has
// fewer than 8192 waves (the card's wave slots) and tiles more than 4 rows.
// Longer tiles load fewer halo rows, shorter ones keep a small batch from
// being a few serial chains.  Solves with 4, 8, 16, 32 and 64 rows (FP32; the
// default's in brackets): 512 problems of side 65 .. 1025 24.7, [23.9] with 8
// or 16, 24.5, 26.1 ms; 64 of side 1025 12.0, 11.8, [11.9], 12.2, 13.0 ms; 8 of
// side 1025 2.05, 2.08, [2.12], 2.02, 2.34 ms; 8 of side 129 [0.35], 0.37, 0.41,
// 0.49, 0.71 ms; 2 of side 1025 [1.23], 1.22, 1.27, 1.48, 1.87 ms.
int default_rows(const homg_batch_ctx* b) {
  int rows = 16;
  for (; rows > 4; rows /= 2) {
    int64_t waves = 0;
    for (int i : b->big) waves += batch_residual_waves(b->sides[i], rows);
    if (waves >= 8192) break;
  }
  return rows;
}

int rows_for(const homg_batch_ctx* b, int side) {
  auto it = b->tile_rows.find(side);
  if (it != b->tile_rows.end() && it->second > 0) return std::min(it->second, side - 2);
  return std::min(b->def_rows, side - 2);
}

int depth_for(const homg_batch_ctx* b, int side) {
  auto it = b->pass_iters.find(side);
  return (it != b->pass_iters.end() && it->second > 0) ? std::min(it->second, TB_MAX_IT) : TB_MAX_IT;
}

// Up to this many nodes in all, a batch is bound by latency: its passes run
// on tiles (1.8 times the work, but every load in one round trip; above, the
// walking waves) and the end of the restriction chain in one launch (above,
// one launch per step).  512 problems of side 65 .. 1025, 143e6 nodes: the
// lattice passes took 570 us a cycle on tiles, the chain 476 us in one launch.
// Whole solves, time of the one form over the other's by total nodes: side 129
// 0.25e6 0.89, 1.0e6 1.06, 2.1e6 1.22; 257 0.5e6 0.87, 1.0e6 0.97, 2.0e6 1.18;
// 513 0.8e6 0.87, 1.8e6 1.13, 3.9e6 1.47; 1025, whose level 0 walks in either
// form, 1.1e6 0.74, 3.2e6 0.87, 7.4e6 1.05, 16e6 1.21.  The line lies between
// the two groups: one problem of side 1025 is to be on tiles, and batches of
// small sides give away up to a fifth just below it.
constexpr int64_t BATCH_TILED_NODES = 1 << 21;

// Rows per band of a walking lattice pass, and level 0's least.  Solves with 8,
// 16 and 32 (FP32): 512 problems of side 65 .. 1025 24.19, 24.05, 24.16 ms, 64 of
// side 1025 11.94, 11.90, 11.96 ms; few problems, where bands are short of
// waves, gain from 8 what those lose: 8 of side 1025 2.06, 2.12, 2.28 ms.
constexpr int LATTICE_ROWS = 16;

constexpr int MULTI_B = 4, MULTI_P = 4;  // the multi-level restriction: owned nodes per axis, levels at most

bool latency_bound(const homg_batch_ctx* b) {
  int64_t nodes = 0;
  for (int i : b->big) nodes += int64_t(b->sides[i]) * b->sides[i];
  return nodes <= BATCH_TILED_NODES;
}
// Restriction steps of a problem that run as one multi-level launch.
int multi_steps(const Problem& p, bool small_batch) {
  return small_batch && p.ms - 1 >= 2 ? std::min(p.ms - 1, MULTI_P) : 0;
}
bool walks(bool small_batch, int side) { return !(small_batch && side <= LT2_MAX_SIDE); }

// Bytes that build_plan's lists take at most, whatever the tile rows and pass
// iterations.  Of the pass lists there is one set for each run of launches
// that differ in their iterates alone (two sets of descriptors, the iterates
// alternate).  A run ends where the problems of some side go over to their next
// kind of launch: a level's first, a further or its last one.
size_t plan_bound(const homg_batch_ctx* b) {
  const bool small_batch = latency_bound(b);
  int64_t runs = 1;
  int last = 0;  // (big is sorted by side)
  for (int i : b->big) {
    if (b->sides[i] != last) runs += 3 * b->probs[i].ms + 1;
    last = b->sides[i];
  }
  int64_t tiles = 0, rs = 0, multi = 0, descs = 0;
  for (int i : b->big) {
    const Problem& p = b->probs[i];
    tiles += (batch_residual_waves(p.n, 2) + 3) / 4;
    const int P = multi_steps(p, small_batch);
    for (int a = 1; a < p.ms - P; ++a, ++rs) {
      const int nc = (p.n - 1) / (2 << a) + 1;
      tiles += batch_restrict_tiles(nc, default_walk_len(2, nc));
    }
    if (P) {
      const int nb = (p.rl[p.ms].side - 1 + MULTI_B - 1) / MULTI_B;
      tiles += int64_t(nb) * nb;
      ++multi;
    }
    for (int m = 0; m < p.ms; ++m) {
      const int nm = (p.n - 1) / (1 << m) + 1, it = level_iters(b, p.levels, m);
      const int64_t launches = m ? (it + LT_MAX_IT - 1) / LT_MAX_IT : it;
      const int64_t ts = batch_tiled_side(nm);
      tiles += std::min(launches, runs) * (walks(small_batch, nm) ? tb_blocks(nm, TB_MAX_IT, LATTICE_ROWS) : ts * ts);
      descs += std::min(launches, 2 * runs);
    }
  }
  const size_t ta = batch_tail_bytes(b->prec);
  return sizeof(BatchResidual) * b->big.size() + sizeof(BatchRestrict) * rs + batch_multi_bytes() * multi +
         ta * (b->big.size() + b->small[0].size() + b->small[1].size()) + sizeof(BatchPass) * descs +
         sizeof(int2) * tiles + 8 * 256;  // each of the eight lists starts at a multiple of 256 bytes
}

// The stage lists of the current tile shapes and pass depths, on the host
// alone: what a solve needs on the device is there since the handle was made.
homg_status build_plan(homg_batch_ctx* b) try {
  const int eb = prec_bytes(b->prec);
  const bool red = b->prec != PREC_F64;
  auto node = [&](char* p, const Lay& l) -> char* { return p ? p + size_t(l.off) * eb : nullptr; };
  const bool small_batch = latency_bound(b);

  std::vector<int2> tiles;
  auto add_tiles = [&](int desc, int n) {
    for (int t = 0; t < n; ++t) tiles.push_back(make_int2(desc, t));
  };
  auto close = [&](int first) { return TileRange{first, int(tiles.size()) - first}; };
  // residual + restriction to level 1
  std::vector<BatchResidual> res;
  for (int i : b->big) {
    Problem& p = b->probs[i];
    const int len = std::max(2, (rows_for(b, p.n) + 1) / 2 * 2);  // whole level-1 rows
    const int waves = batch_residual_waves(p.n, len);
    const double h = 1.0 / double(p.n - 1);
    res.push_back(BatchResidual{node(p.r[0], p.rl[0]), node(p.r[1], p.rl[1]), p.rl[0].pitch, p.rl[1].pitch, p.partials,
                                p.partials + batch_residual_waves(p.n, 2), 1.0 / (h * h), i, p.n, len, waves});
    add_tiles(int(res.size()) - 1, (waves + 3) / 4);
  }
  b->residual = close(0);
  // the chain 1 -> ms: single steps, then the last P as one launch
  std::vector<BatchRestrict> rs;
  std::vector<char> multi;
  b->multi_lds = 0;
  int deepest = 0;
  for (int i : b->big) deepest = std::max(deepest, b->probs[i].ms);
  b->restricts.assign(deepest + 1, TileRange{});
  for (int a = 1; a <= deepest; ++a) {
    const int first = int(tiles.size());
    for (int i : b->big) {
      const Problem& p = b->probs[i];
      if (a >= p.ms - multi_steps(p, small_batch)) continue;
      const int nc = (p.n - 1) / (2 << a) + 1, len = default_walk_len(2, nc);
      rs.push_back(BatchRestrict{node(p.r[a], p.rl[a]), node(p.r[a + 1], p.rl[a + 1]), p.rl[a].pitch,
                                 p.rl[a + 1].pitch, i, nc, len, 0});
      add_tiles(int(rs.size()) - 1, batch_restrict_tiles(nc, len));
    }
    b->restricts[a] = close(first);
  }
  {
    const int first = int(tiles.size());
    int k = 0;
    for (int i : b->big) {
      Problem& p = b->probs[i];
      const int P = multi_steps(p, small_batch);
      if (!P) continue;
      void* r[MR_MAX + 1];
      Lay l[MR_MAX + 1];
      for (int j = 0; j <= P; ++j) {
        r[j] = p.r[p.ms - P + j];
        l[j] = p.rl[p.ms - P + j];
      }
      multi.resize(multi.size() + batch_multi_bytes());
      const int blocks = batch_multi_fill(b->prec, multi.data() + multi.size() - batch_multi_bytes(), i, P, MULTI_B, r, l);
      b->multi_lds = std::max(b->multi_lds, restrict_multi_lds(b->prec, 2, P, MULTI_B));
      add_tiles(k++, blocks);
    }
    b->multi = close(first);
  }
  // coarse tails
  const size_t ta = batch_tail_bytes(b->prec);
  std::vector<char> tails(ta * b->big.size());
  b->tail_lds = 0;
  for (size_t k = 0; k < b->big.size(); ++k) {
    Problem& p = b->probs[b->big[k]];
    const int nlev = p.levels - p.ms, nms = (p.n - 1) / (1 << p.ms) + 1;
    int its[BATCH_MAX_LEVELS];
    for (int j = 0; j < nlev; ++j) its[j] = level_iters(b, p.levels, p.ms + j);
    batch_tail_fill(b->prec, tails.data() + ta * k, nms, nlev, its, b->omega, node(p.r[p.ms], p.rl[p.ms]),
                    p.rl[p.ms].pitch, node(p.x[p.ms][0], p.rl[p.ms]), node(p.x[p.ms][1], p.rl[p.ms]),
                    p.rl[p.ms].pitch, red, b->d_st + b->big[k], b->hist[b->big[k]], p.partials, res[k].count);
    b->tail_lds = std::max(b->tail_lds, coarse_tail_lds(b->prec, 2, nms, nlev, red, false, false));
  }
  // one-workgroup problems
  std::vector<char> smalls[2];
  for (int t = 0; t < 2; ++t) {
    smalls[t].resize(ta * b->small[t].size());
    b->small_lds[t] = 0;
    for (size_t k = 0; k < b->small[t].size(); ++k) {
      const int i = b->small[t][k], n = b->sides[i], L = side_k(n);
      int its[BATCH_MAX_LEVELS];
      for (int j = 0; j < L; ++j) its[j] = level_iters(b, L, j);
      const bool rr = n >= 5 && L >= 2 && !(t == 1 && L == 2);  // as a single solve's residual
      batch_small_fill(b->prec, smalls[t].data() + ta * k, n, L, its, b->omega, t == 1, rr, i, b->d_st + i, b->hist[i]);
      b->small_lds[t] = std::max(b->small_lds[t], coarse_tail_lds(b->prec, 2, n, L, t == 1, false, true));
    }
  }
  // iteration passes: every problem's sequence, aligned at its end
  std::vector<std::vector<std::pair<PassGroup, BatchPass>>> seq;  // [position from the end]
  for (int i : b->big) {
    Problem& p = b->probs[i];
    std::vector<std::pair<PassGroup, BatchPass>> mine;
    const char* prev = p.x[p.ms][0];  // the state level m starts from
    const char* cur = p.x[p.ms][1];
    for (int m = p.ms - 1; m >= 0; --m) {
      const int nm = (p.n - 1) / (1 << m) + 1, it = level_iters(b, p.levels, m);
      const int step = m ? LT_MAX_IT : depth_for(b, p.n);
      const Lay& cl = m ? p.rl[m] : p.el;
      const double h = 1.0 / double(nm - 1);
      const bool walk = walks(small_batch, nm);
      int src = 1;
      for (int t0 = 0; t0 < it; t0 += step) {
        const int g = std::min(step, it - t0);
        const bool lat = t0 == 0, accum = m == 0 && t0 + g == it;
        const int kind = !walk ? BATCH_TILED : m ? BATCH_WALK_PREV : accum ? BATCH_WALK_ACCUM : BATCH_WALK;
        char* from = m ? p.x[m][src] : p.e[src];
        char* to = m ? p.x[m][1 - src] : p.e[1 - src];
        BatchPass q{};
        q.xo = lat ? nullptr : node(from, cl);
        q.xn = accum ? nullptr : node(to, cl);
        q.xp = m ? node(p.x[m][2], cl) : nullptr;
        q.r = node(p.r[m], p.rl[m]);
        if (lat) {
          q.l1_prev = node(const_cast<char*>(prev), p.rl[m + 1]);
          q.l1_cur = node(const_cast<char*>(cur), p.rl[m + 1]);
          q.l1_pitch = p.rl[m + 1].pitch;
        }
        q.cp = cl.pitch;
        q.rp = p.rl[m].pitch;
        q.hl2 = h * h;
        q.prob = i;
        q.n = nm;
        q.len = walk ? (m ? LATTICE_ROWS : std::max(LATTICE_ROWS, rows_for(b, p.n))) : batch_tiled_side(nm);
        q.accum = accum ? 1 : 0;
        mine.push_back({PassGroup{g, kind, lat, 0, 0, 0}, q});
        src = 1 - src;
      }
      if (m) {
        cur = p.x[m][src];
        prev = p.x[m][2];
      }
    }
    for (size_t k = 0; k < mine.size(); ++k) {
      const size_t pos = mine.size() - 1 - k;
      if (seq.size() <= pos) seq.resize(pos + 1);
      seq[pos].push_back(mine[k]);
    }
  }
  // (Levels of many iterations repeat the same launch, the two iterates
  // alternating: a launch takes its tiles from the one before it and its
  // descriptors from the one before that where they are the same.  With lists of
  // their own 32768 iterations of level 0 at 32769^2 were 2.5e9 tiles.)
  std::vector<BatchPass> passes;
  b->passes.clear();
  using Key = std::tuple<int, int, bool>;
  struct Made {
    std::vector<BatchPass> q;
    int desc, first, count;
  };
  std::map<Key, Made> made[2];  // of the last position and the one before
  for (size_t pos = seq.size(); pos-- > 0;) {
    std::map<Key, Made> now;  // the largest problems stay first
    for (auto& e : seq[pos]) now[Key(e.first.it, e.first.kind, e.first.lat)].q.push_back(e.second);
    for (auto& kv : now) {
      const int it = std::get<0>(kv.first), kind = std::get<1>(kv.first);
      Made& m = kv.second;
      auto same = [&](const std::map<Key, Made>& from, auto&& eq) -> const Made* {
        const auto f = from.find(kv.first);
        if (f == from.end() || f->second.q.size() != m.q.size()) return nullptr;
        return std::equal(m.q.begin(), m.q.end(), f->second.q.begin(), eq) ? &f->second : nullptr;
      };
      if (const Made* o = same(made[1], [](const BatchPass& a, const BatchPass& c) { return !std::memcmp(&a, &c, sizeof a); })) {
        m.desc = o->desc;
      } else {
        m.desc = int(passes.size());
        passes.insert(passes.end(), m.q.begin(), m.q.end());
      }
      if (const Made* o = same(made[0], [](const BatchPass& a, const BatchPass& c) { return a.n == c.n && a.len == c.len; })) {
        m.first = o->first;
        m.count = o->count;
      } else {
        m.first = int(tiles.size());
        for (size_t k = 0; k < m.q.size(); ++k)
          add_tiles(int(k), kind == BATCH_TILED ? m.q[k].len * m.q[k].len : tb_blocks(m.q[k].n, it, m.q[k].len));
        m.count = int(tiles.size()) - m.first;
      }
      b->passes.push_back(PassGroup{it, kind, std::get<2>(kv.first), m.desc, m.first, m.count});
    }
    made[1] = std::move(made[0]);
    made[0] = std::move(now);
  }
  // one allocation for all lists
  std::vector<char> host;
  auto put = [&](const void* p, size_t bytes) {
    const size_t at = (host.size() + 255) & ~size_t(255);
    host.resize(at + bytes);
    if (bytes) std::memcpy(host.data() + at, p, bytes);
    return at;
  };
  b->o_res = put(res.data(), sizeof(BatchResidual) * res.size());
  b->o_rs = put(rs.data(), sizeof(BatchRestrict) * rs.size());
  b->o_multi = put(multi.data(), multi.size());
  b->o_tail = put(tails.data(), tails.size());
  for (int t = 0; t < 2; ++t) b->o_small[t] = put(smalls[t].data(), smalls[t].size());
  b->o_pass = put(passes.data(), sizeof(BatchPass) * passes.size());
  b->o_tiles = put(tiles.data(), sizeof(int2) * tiles.size());
  if (host.size() > b->plan_bytes)
    return bfail(b, HOMG_ERR_WORKSPACE, "the stage lists exceed their allocation");
  b->lists = std::move(host);
  return HOMG_OK;
} catch (const std::bad_alloc&) {
  return bfail(b, HOMG_ERR_OOM, "host allocation of the stage lists failed");
}

// The lists on the device, on stream s.
homg_status ready_plan(homg_batch_ctx* b, hipStream_t s) {
  if (!b->dirty) return HOMG_OK;
  if (homg_status e = build_plan(b)) return e;
  BHIP(b, hipMemcpyAsync(b->plan, b->lists.data(), b->lists.size(), hipMemcpyHostToDevice, s));
  b->dirty = false;
  return HOMG_OK;
}

// One cycle of every problem solved in stages; pending: the cycle whose
// residual norm the tails reduce first (-1: none).
homg_status enqueue_cycle(homg_batch_ctx* b, int pending, hipStream_t s) {
  const bool red = b->prec != PREC_F64;
  const int2* tiles = reinterpret_cast<const int2*>(b->plan + b->o_tiles);
  const BatchRestrict* rs = reinterpret_cast<const BatchRestrict*>(b->plan + b->o_rs);
  const BatchPass* ps = reinterpret_cast<const BatchPass*>(b->plan + b->o_pass);
  const double* const* f = reinterpret_cast<const double* const*>(b->d_ptrs);
  double* const* u = reinterpret_cast<double* const*>(b->d_ptrs + b->count);
  for (const TileRange& t : b->restricts)
    if (t.count) BHIP(b, launch_batch_restrict(b->prec, rs, tiles + t.first, t.count, b->d_st, s));
  if (b->multi.count)
    BHIP(b, launch_batch_restrict_multi(b->prec, b->plan + b->o_multi, tiles + b->multi.first, b->multi.count,
                                        b->multi_lds, b->d_st, s));
  BHIP(b, launch_batch_tails(b->prec, red, b->plan + b->o_tail, int(b->big.size()), b->tail_lds, pending, s));
  for (const PassGroup& g : b->passes)
    BHIP(b, launch_batch_pass(b->prec, ps + g.desc, tiles + g.first, g.count, g.it, g.lat, g.kind, b->omega, b->d_st, u, s));
  BHIP(b, launch_batch_residual(b->prec, reinterpret_cast<const BatchResidual*>(b->plan + b->o_res),
                                tiles + b->residual.first, b->residual.count, false, f, u, b->d_st, s));
  return HOMG_OK;
}

constexpr int SMALL_CYCLES = 64;  // cycles per launch of the one-workgroup problems (at most 126 iterations each)

homg_status run_once(homg_batch_ctx* b, const double* const* f, double* const* u, double tol,
                     hipStream_t s) {
  for (int i = 0; i < b->count; ++i) {
    if (!f[i] || !u[i]) return bfail(b, HOMG_ERR_INVALID_ARG, "null f or u pointer");
    b->h_ptrs[i] = const_cast<double*>(f[i]);
    b->h_ptrs[b->count + i] = u[i];
  }
  if (homg_status e = ready_plan(b, s)) return e;
  BHIP(b, hipMemcpyAsync(b->d_ptrs, b->h_ptrs, 2 * sizeof(void*) * b->count, hipMemcpyHostToDevice, s));
  const double* const* df = reinterpret_cast<const double* const*>(b->d_ptrs);
  double* const* du = reinterpret_cast<double* const*>(b->d_ptrs + b->count);
  const BatchResidual* res = reinterpret_cast<const BatchResidual*>(b->plan + b->o_res);
  const int2* tiles = reinterpret_cast<const int2*>(b->plan + b->o_tiles);
  const int nbig = int(b->big.size());
  int small_c0 = 0;  // the one-workgroup problems' next cycles
  auto launch_small = [&]() -> homg_status {
    const int c1 = std::min(b->max_cycles, small_c0 + SMALL_CYCLES);
    for (int t = 0; t < 2; ++t)
      if (!b->small[t].empty())
        BHIP(b, launch_batch_small(b->prec, t == 1, b->plan + b->o_small[t], int(b->small[t].size()), b->small_lds[t],
                                   df, du, tol, small_c0, c1, s));
    small_c0 = c1;
    return HOMG_OK;
  };
  if (homg_status e = launch_small()) return e;
  if (nbig) {
    BHIP(b, launch_batch_residual(b->prec, res, tiles + b->residual.first, b->residual.count, true, df, du, b->d_st, s));
    BHIP(b, launch_batch_finalize(res, nbig, b->d_st, b->d_hist, 0, true, tol, s));
  }
  int enqueued = 0, batch = 2;
  for (;;) {
    const int upto = nbig ? std::min(b->max_cycles, enqueued + batch) : enqueued;
    for (int c = enqueued + 1; c <= upto; ++c)
      if (homg_status e = enqueue_cycle(b, c > enqueued + 1 ? c - 1 : -1, s)) return e;
    if (upto > enqueued) BHIP(b, launch_batch_finalize(res, nbig, b->d_st, b->d_hist, upto, false, tol, s));
    enqueued = upto;
    BHIP(b, launch_batch_publish(b->count, b->d_st, b->d_hist, b->h_state, s));
    BHIP(b, hipStreamSynchronize(s));
    // the next batch of cycles from the slowest problem still running
    bool run_big = false, run_small = false;
    double need = 1.0;
    for (int i : b->big) {
      const BatchState& v = b->h_state[i];
      if (v.done) continue;
      run_big = true;
      double q = 0.5;
      if (v.cycles >= 2 && v.prev > 0) q = v.rel / v.prev;
      q = std::min(std::max(q, 1e-3), 0.95);
      need = std::max(need, std::log(tol / v.rel) / std::log(q));
    }
    for (int t = 0; t < 2; ++t)
      for (int i : b->small[t]) run_small = run_small || !b->h_state[i].done;
    run_big = run_big && enqueued < b->max_cycles;
    run_small = run_small && small_c0 < b->max_cycles;
    if (!run_big && !run_small) break;
    batch = run_big ? int(std::ceil(std::min(need, 16.0))) : 0;
    if (run_small)
      if (homg_status e = launch_small()) return e;
  }
  return HOMG_OK;
}

}  // namespace

extern "C" {

homg_status homg_batch_create(homg_batch* out, int count, const int64_t* sides, const homg_options* opt) {
  if (!out) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "null output handle");
  *out = nullptr;
  if (count < 1 || count > 16000) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "count must be in [1, 16000]");
  if (!sides) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "null sides");
  homg_options o;
  homg_options_init(&o);
  if (opt) {
    if (opt->struct_size != sizeof(homg_options))
      return bfail(nullptr, HOMG_ERR_INVALID_ARG, "homg_options.struct_size mismatch");
    o = *opt;
    if (o.grid_layout != HOMG_GRID_NESTED || o.restriction != HOMG_RESTRICT_PYRAMID)
      return bfail(nullptr, HOMG_ERR_UNSUPPORTED,
                   "the batched solver runs nested grids with the restriction pyramid only");
  }
  for (int i = 0; i < count; ++i) {
    const int k = side_k(sides[i]);
    if (k < 1 || k > 15) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "every side must be 2^k + 1, 1 <= k <= 15");
  }
  const double omega = o.omega > 0 ? o.omega : 0.8;
  if (!(omega > 0.0 && omega <= 1.0)) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "omega must be in (0, 1]");
  if (o.precision < HOMG_FP64 || o.precision > HOMG_BF16_IR)
    return bfail(nullptr, HOMG_ERR_INVALID_ARG, "unknown precision");
  homg_batch_ctx* b = new (std::nothrow) homg_batch_ctx;
  if (!b) return bfail(nullptr, HOMG_ERR_OOM, "host allocation failed");
  b->count = count;
  b->prec = o.precision;
  b->omega = omega;
  b->max_i = o.max_i > 0 ? o.max_i : 4;
  b->max_cycles = o.max_cycles > 0 ? o.max_cycles : 200;
  if (hipGetDevice(&b->device) != hipSuccess) {
    delete b;
    return bfail(nullptr, HOMG_ERR_HIP, "hipGetDevice failed");
  }
  const int eb = prec_bytes(b->prec);
  // one arena: what must start at 0 (boundaries) first, then sums and histories
  size_t total = 0, zeroed = 0;
  auto take = [&](size_t bytes) {
    const size_t o2 = total;
    total += (bytes + 255) & ~size_t(255);
    return o2;
  };
  b->probs.resize(count);
  std::vector<std::vector<size_t>> at(count);
  for (int i = 0; i < count; ++i) {
    const int n = int(sides[i]), L = side_k(n);
    b->sides.push_back(n);
    Problem& p = b->probs[i];
    p.n = n;
    p.levels = L;
    if (n <= tail_max_side(2)) {
      b->small[b->prec != PREC_F64 && L >= 2 ? 1 : 0].push_back(i);
      continue;
    }
    b->big.push_back(i);
    p.el = padded_layout(2, n, eb);
    while (((n - 1) >> p.ms) + 1 > tail_max_side(2)) ++p.ms;
    for (int m = 0; m <= p.ms; ++m) {
      p.rl[m] = padded_layout(2, (n - 1) / (1 << m) + 1, eb);
      const size_t bytes = size_t(p.rl[m].alloc) * eb;
      at[i].push_back(take(bytes));
      for (int c = 0; m && c < (m < p.ms ? 3 : 2); ++c) at[i].push_back(take(bytes));
    }
    if (level_iters(b, L, 0) > 1)  // level 0's iterates (passes may be of one iteration)
      for (int c = 0; c < 2; ++c) at[i].push_back(take(size_t(p.el.alloc) * eb));
  }
  zeroed = total;
  b->def_rows = default_rows(b);
  // the largest problems first in every list: a launch does not end on them
  std::stable_sort(b->big.begin(), b->big.end(), [&](int x, int y) { return b->sides[x] > b->sides[y]; });
  std::vector<size_t> part(count), hist(count);
  for (int i = 0; i < count; ++i) {
    if (b->sides[i] > tail_max_side(2)) part[i] = take(2 * sizeof(double) * size_t(batch_residual_waves(b->sides[i], 2)));
    hist[i] = take(sizeof(double) * size_t(b->max_cycles + 1));
  }
  if (hipMalloc(&b->arena, total) != hipSuccess) {
    (void)hipGetLastError();
    free_batch(b);
    return bfail(nullptr, HOMG_ERR_OOM, "batch arena allocation of " + std::to_string(total) + " bytes failed");
  }
  bool ok = !zeroed || hipMemset(b->arena, 0, zeroed) == hipSuccess;
  ok = ok && hipMalloc(reinterpret_cast<void**>(&b->d_ptrs), 2 * sizeof(void*) * count) == hipSuccess;
  ok = ok && hipMalloc(reinterpret_cast<void**>(&b->d_st), sizeof(DevState) * count) == hipSuccess;
  ok = ok && hipMalloc(reinterpret_cast<void**>(&b->d_hist), sizeof(double*) * count) == hipSuccess;
  ok = ok && hipHostMalloc(reinterpret_cast<void**>(&b->h_ptrs), 2 * sizeof(void*) * count, hipHostMallocDefault) == hipSuccess;
  ok = ok && hipHostMalloc(reinterpret_cast<void**>(&b->h_state), sizeof(BatchState) * count, hipHostMallocDefault) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    free_batch(b);
    return bfail(nullptr, HOMG_ERR_OOM, "batch workspace allocation failed");
  }
  char* base = static_cast<char*>(b->arena);
  for (int i = 0; i < count; ++i) {
    b->hist.push_back(reinterpret_cast<double*>(base + hist[i]));
    Problem& p = b->probs[i];
    if (at[i].empty()) continue;
    p.partials = reinterpret_cast<double*>(base + part[i]);
    size_t k = 0;
    for (int m = 0; m <= p.ms; ++m) {
      p.r[m] = base + at[i][k++];
      for (int c = 0; m && c < (m < p.ms ? 3 : 2); ++c) p.x[m][c] = base + at[i][k++];
    }
    for (int c = 0; c < 2 && k < at[i].size(); ++c) p.e[c] = base + at[i][k++];
  }
  if (hipMemcpy(b->d_hist, b->hist.data(), sizeof(double*) * count, hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipGetLastError();
    free_batch(b);
    return bfail(nullptr, HOMG_ERR_HIP, "batch initialisation failed");
  }
  b->plan_bytes = plan_bound(b);
  if (hipMalloc(reinterpret_cast<void**>(&b->plan), b->plan_bytes) != hipSuccess) {
    (void)hipGetLastError();
    const size_t bytes = b->plan_bytes;
    free_batch(b);
    return bfail(nullptr, HOMG_ERR_OOM, "stage list allocation of " + std::to_string(bytes) + " bytes failed");
  }
  if (homg_status e = ready_plan(b, nullptr)) {
    const std::string msg = b->err;
    free_batch(b);
    return bfail(nullptr, e, msg);
  }
  if (hipDeviceSynchronize() != hipSuccess) {
    free_batch(b);
    return bfail(nullptr, HOMG_ERR_HIP, "batch initialisation failed");
  }
  *out = b;
  return HOMG_OK;
}

homg_status homg_batch_destroy(homg_batch b) {
  if (!b) return HOMG_OK;
  (void)hipDeviceSynchronize();
  free_batch(b);
  return HOMG_OK;
}

homg_status homg_batch_set_tile_rows(homg_batch b, int64_t side, int rows) {
  if (!b) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "null batch handle");
  if (rows < 0 || rows > 4096) return bfail(b, HOMG_ERR_INVALID_ARG, "rows must be in [0, 4096]");
  if (rows == 0) b->tile_rows.erase(int(side));
  else b->tile_rows[int(side)] = rows;
  b->dirty = true;
  return HOMG_OK;
}

homg_status homg_batch_set_pass_iters(homg_batch b, int64_t side, int iters) {
  if (!b) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "null batch handle");
  if (iters < 0 || iters > TB_MAX_IT) return bfail(b, HOMG_ERR_INVALID_ARG, "iters must be in [0, 4]");
  if (iters == 0) b->pass_iters.erase(int(side));
  else b->pass_iters[int(side)] = iters;
  b->dirty = true;
  return HOMG_OK;
}

homg_status homg_batch_solve(homg_batch b, const double* const* f, double* const* u, double tol,
                             void* stream, double* relres_out, int* cycles_out, int* status_out) {
  if (!b) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "null batch handle");
  if (!f || !u) return bfail(b, HOMG_ERR_INVALID_ARG, "null f or u array");
  if (!(tol > 0.0)) return bfail(b, HOMG_ERR_INVALID_ARG, "tol must be > 0");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (homg_status e = run_once(b, f, u, tol, s)) return e;
  homg_status worst = HOMG_OK;
  for (int i = 0; i < b->count; ++i) {
    const int dn = b->h_state[i].done;
    homg_status si = dn == 1 ? HOMG_OK : (dn == 2 ? HOMG_ERR_NUMERICAL : HOMG_ERR_NOT_CONVERGED);
    if (relres_out) relres_out[i] = b->h_state[i].rel;
    if (cycles_out) cycles_out[i] = b->h_state[i].cycles;
    if (status_out) status_out[i] = si;
    if (si == HOMG_ERR_NUMERICAL) worst = si;
    else if (si != HOMG_OK && worst == HOMG_OK) worst = si;
  }
  if (worst != HOMG_OK) return bfail(b, worst, "some problems did not converge");
  return HOMG_OK;
}

homg_status homg_batch_tune(homg_batch b, const double* const* f, double* const* u, double tol,
                            void* stream, const char* cache_path) {
  if (!b) return bfail(nullptr, HOMG_ERR_INVALID_ARG, "null batch handle");
  if (!f || !u) return bfail(b, HOMG_ERR_INVALID_ARG, "null f or u array");
  if (!(tol > 0.0)) return bfail(b, HOMG_ERR_INVALID_ARG, "tol must be > 0");
  for (int i = 0; i < b->count; ++i)
    if (!f[i] || !u[i]) return bfail(b, HOMG_ERR_INVALID_ARG, "null f or u pointer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  std::vector<int> distinct = b->sides;
  std::sort(distinct.begin(), distinct.end());
  distinct.erase(std::unique(distinct.begin(), distinct.end()), distinct.end());
  const char* pname = b->prec == PREC_F64 ? "fp64" : (b->prec == PREC_F32 ? "fp32" : "bf16");
  int cus = 0;
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b->device);
  // the sides solved in stages: the others read neither setting
  const std::vector<int> staged(std::upper_bound(distinct.begin(), distinct.end(), tail_max_side(2)), distinct.end());
  // what the best settings depend on beside the side: the passes' kernels
  // (latency_bound) and the number of waves in flight (default_rows), both of the
  // whole batch
  char key[128];
  std::snprintf(key, sizeof key, "gfx950/cu%d/%s/maxi%d/%s%d", cus, pname, b->max_i,
                latency_bound(b) ? "tiles" : "bands", b->def_rows);
  // cache: lines of the form   <key> <side> <rows> <iterations per level-0 pass>
  if (cache_path) {
    if (FILE* fp = std::fopen(cache_path, "r")) {
      char line[256], k2[128];
      int side = 0, rows = 0, its = 0, hits = 0;
      while (std::fgets(line, sizeof line, fp))
        if (std::sscanf(line, "%127s %d %d %d", k2, &side, &rows, &its) == 4 && std::strcmp(k2, key) == 0 &&
            std::find(staged.begin(), staged.end(), side) != staged.end() && rows > 0 && its > 0 &&
            its <= TB_MAX_IT) {
          b->tile_rows[side] = rows;
          b->pass_iters[side] = its;
          b->dirty = true;
          ++hits;
        }
      std::fclose(fp);
      if (hits >= int(staged.size())) return HOMG_OK;
    }
  }
  // Every candidate starts from the caller's initial guesses: they are saved
  // here and restored (outside the timed region) before each run, and
  // restored once more at the end, so u is left as given.
  std::vector<size_t> uoff(b->count + 1, 0);
  for (int i = 0; i < b->count; ++i) uoff[i + 1] = uoff[i] + size_t(b->sides[i]) * b->sides[i];
  double* saved = nullptr;
  if (hipMalloc(reinterpret_cast<void**>(&saved), sizeof(double) * uoff[b->count]) != hipSuccess) {
    (void)hipGetLastError();
    return bfail(b, HOMG_ERR_OOM, "tuner copy of the initial guesses could not be allocated");
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  homg_status st = HOMG_OK;
  auto hip_ok = [&](hipError_t e, const char* what) {
    if (e != hipSuccess && st == HOMG_OK) st = bfail(b, HOMG_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
    return st == HOMG_OK;
  };
  auto copy_u = [&](bool save) {
    for (int i = 0; i < b->count && st == HOMG_OK; ++i) {
      const size_t bytes = sizeof(double) * (uoff[i + 1] - uoff[i]);
      hip_ok(save ? hipMemcpyAsync(saved + uoff[i], u[i], bytes, hipMemcpyDeviceToDevice, s)
                  : hipMemcpyAsync(u[i], saved + uoff[i], bytes, hipMemcpyDeviceToDevice, s),
             "hipMemcpyAsync");
    }
  };
  // one run of the current tiles: restore u, time the solve, check that it
  // did work (a run whose problems all meet tol at cycle 0 times nothing)
  auto once = [&](float* ms) {
    copy_u(false);
    if (homg_status e = ready_plan(b, s)) {
      st = e;
      return false;
    }
    if (!hip_ok(hipEventRecord(e0, s), "hipEventRecord")) return false;
    if (homg_status e = run_once(b, f, u, tol, s)) {
      st = e;
      return false;
    }
    if (!hip_ok(hipEventRecord(e1, s), "hipEventRecord") || !hip_ok(hipEventSynchronize(e1), "hipEventSynchronize") ||
        !hip_ok(hipEventElapsedTime(ms, e0, e1), "hipEventElapsedTime"))
      return false;
    int most = 0;
    for (int i = 0; i < b->count; ++i) most = std::max(most, b->h_state[i].cycles);
    if (most < 1) {
      st = bfail(b, HOMG_ERR_INVALID_ARG, "the initial guesses already meet tol: no cycle to time");
      return false;
    }
    return true;
  };
  // a candidate's time: the median of three runs
  auto timed = [&](float* ms) {
    float t[3];
    for (int r = 0; r < 3; ++r)
      if (!once(&t[r])) return false;
    std::sort(t, t + 3);
    *ms = t[1];
    return true;
  };
  hip_ok(hipEventCreate(&e0), "hipEventCreate");
  hip_ok(hipEventCreate(&e1), "hipEventCreate");
  copy_u(true);
  float best = 0.f, warm = 0.f;
  bool ok = st == HOMG_OK && once(&warm) && timed(&best);
  // coordinate descent over the sides, largest first: tile rows, then the
  // iterations per level-0 pass
  for (auto it = staged.rbegin(); ok && it != staged.rend(); ++it) {
    const int side = *it;
    const int keep = rows_for(b, side);
    int best_rows = keep;
    for (int rows : {4, 8, 16, 32, 64, 128}) {
      if (rows == keep || rows > side - 2) continue;
      b->tile_rows[side] = rows;
      b->dirty = true;
      float ms = 0.f;
      if (!(ok = timed(&ms))) break;
      if (ms < best) {
        best = ms;
        best_rows = rows;
      }
    }
    b->tile_rows[side] = best_rows;
    b->dirty = true;
    const int keep_it = depth_for(b, side);
    int best_it = keep_it;
    for (int its = 1; ok && its <= TB_MAX_IT; ++its) {
      if (its == keep_it) continue;
      b->pass_iters[side] = its;
      b->dirty = true;
      float ms = 0.f;
      if (!(ok = timed(&ms))) break;
      if (ms < best) {
        best = ms;
        best_it = its;
      }
    }
    b->pass_iters[side] = best_it;
    b->dirty = true;
  }
  copy_u(false);
  hip_ok(hipStreamSynchronize(s), "hipStreamSynchronize");
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(saved);
  if (st != HOMG_OK) return st;
  if (cache_path) {
    if (FILE* fp = std::fopen(cache_path, "a")) {
      for (int side : distinct) std::fprintf(fp, "%s %d %d %d\n", key, side, rows_for(b, side), depth_for(b, side));
      std::fclose(fp);
    }
  }
  return HOMG_OK;
}

}  // extern "C"
