// C boundary of libcompactor: argument checks, output layout, workspace carving and the
// stream-ordered launch sequence.  Declarations and their contracts: include/compactor.h.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>

#include "common.h"

using namespace cmp;

namespace {

constexpr long long DEFAULT_GROUP_BYTES = 1ll << 40;   // one group unless the caller asks
constexpr size_t WS_ALIGN = 256;

inline size_t align_up(size_t x) { return (x + WS_ALIGN - 1) / WS_ALIGN * WS_ALIGN; }
inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

enum Need { NEED_SCORE = 1, NEED_PACK = 2 };

int check_params(const compactor_params_t *p, bool scoring) {
  if (!p) return COMPACTOR_EINVAL;
  if (p->layers < 1 || p->kv_heads < 1) return COMPACTOR_EINVAL;
  if ((long long)p->layers * p->kv_heads > (1 << 20)) return COMPACTOR_EINVAL;
  if (p->head_dim != D) return COMPACTOR_EUNSUPPORTED;
  const int ks = p->sketch_dim;
  if (!(ks == 0 || ks == 16 || ks == 32 || ks == 48 || ks == 64)) return COMPACTOR_EUNSUPPORTED;
  if (scoring) {
    if (ks > 0 && !p->phi) return COMPACTOR_EINVAL;
    if (ks > 0 && !aligned16(p->phi)) return COMPACTOR_EALIGN;
    if (!(p->ridge_rel >= 0.f) || !isfinite(p->ridge_rel)) return COMPACTOR_EINVAL;
    if (!isfinite(p->lambda_blend)) return COMPACTOR_EINVAL;
  }
  if (p->group_bytes < 0 || p->gram_wgs < 0 || p->score_tokens < 0)
    return COMPACTOR_EINVAL;
  if (p->select_scope != COMPACTOR_SCOPE_HEAD && p->select_scope != COMPACTOR_SCOPE_LAYER)
    return COMPACTOR_EINVAL;
  return COMPACTOR_OK;
}

// Layer scope pools H heads: their tokens and their budget are counted in 32-bit integers.
int check_scope(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq) {
  if (p->select_scope != COMPACTOR_SCOPE_LAYER) return COMPACTOR_OK;
  for (int b = 0; b < nreq; ++b)
    if ((long long)reqs[b].n * p->kv_heads > 0x7fffffffll - 64) return COMPACTOR_EINVAL;
  return COMPACTOR_OK;
}

int check_requests(const compactor_request_t *reqs, int32_t nreq, int need) {
  if (!reqs || nreq < 1 || nreq > (1 << 20)) return COMPACTOR_EINVAL;
  for (int b = 0; b < nreq; ++b) {
    const compactor_request_t &r = reqs[b];
    if (r.n < 1 || r.n > 0x7fffffff - 64) return COMPACTOR_EINVAL;
    if (!(r.ratio > 0.f && r.ratio <= 1.f)) return COMPACTOR_EINVAL;
    if (need) {
      if ((need & NEED_SCORE) && !r.k_score) return COMPACTOR_EINVAL;
      if ((need & NEED_PACK) && (!r.v_cache || (!r.k_cache && !r.k_score))) return COMPACTOR_EINVAL;
      if (r.stride_t < D || r.stride_l < 0 || r.stride_h < 0) return COMPACTOR_EINVAL;
      if ((r.stride_t & 7) || (r.stride_l & 7) || (r.stride_h & 7)) return COMPACTOR_EALIGN;
      if (!aligned16(r.k_score) || !aligned16(r.k_cache) || !aligned16(r.v_cache) ||
          (reinterpret_cast<uintptr_t>(r.attn) & 3u))
        return COMPACTOR_EALIGN;
    }
  }
  return COMPACTOR_OK;
}

int compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
    n = 256;
  return n;
}

// Gram: a persistent launch, each workgroup taking an equal run of 64-row tiles.  Every (workgroup, head) partial costs
// the factorisation 40 KB, so there is one workgroup a compute unit as long as its run stays short; long ones stream a little
// faster with two.
// Where that one workgroup sums its run as it goes on and where tile by tile (GRAM_FOLD, see gram_kernel) goes by precision: as it
// goes on up to 4 tiles, and up to 24 (17 to 32 heads: 16; exact mode: 32) with few heads and 8 tiles a unit or more; a call of other
// sizes would else sum twice the rows in one accumulator that it used to.
// compactor_score on MI355X, keys not in the last-level cache, us with one workgroup a unit / folding / two, tiles a unit in
// brackets.  k_s = 48: 8 heads of 8192 (4) 30.4 / 31.3 / 32.4, 16384 (8) 36.7 / 38.1 / 39.5, 32768 (16) 45.9 / 47.0 / 51.3, 48000 (23)
// 55.3 / 56.7 / 60.6, 65536 (32) 64.4 / 65.5 / 70.0, 131072 (64) 101 / 103 / 106, 147000 (72) 118 / 118 / 120; 16 of 32768 (32) 63.3 /
// 64.7 / 68.5; 32 of 8000 (16) 45.9 / 47.7 / 49.7, 32768 (64) 102 / 103 / 105, 47000 (92) 141 / 143.5 / 144.5; 64 of 2048 (8) 39.8 / 40.6 /
// 41.8, 4096 (16) 48.9 / 49.7 / 52.0; 128 of 4096 (32) 69.5 / 70.5 / 72.7, 16384 (128) 188 / 195 / 192; 192 of 8192 (96) 159 / 157 / 160;
// 256 of 1024 (16) 48.3 / 49.1 / 55.7, 2048 (32) 66.7 / 67.8 / 74.2, 4096 (64) 104 / 105 / 111, 8192 (128) 187 / 194 / 191.  Exact mode: 8
// of 65536 (32) 83.2 / 84.6 / 86.7, 131072 (64) 122 / 125 / 125; 32 of 18000 (35) 92.3 / 93.0 / 94.8, 57000 (111) 186 / 189 / 189; 256 of
// 4096 (64) 125 / 128 / 128, 8192 (128) 209 / 214 / 210.
// Heads for every unit that end inside runs: one workgroup waits for every partial but two of its run to leave, where two take turns, so
// two it is unless they leave more.  us with one / two, k_s = 16: 304 of 500 (partials 487 / 304) 41.6 / 33.9, 768 of 200 (768 / 768)
// 48.7 / 46.8, 1024 of 1000 (1024 / 1024) 129 / 120, 512 of 2048 (512 / 512) 108 / 102; 512 of 300 (512 / 768) 41.5 / 43.7, 256 of 1000
// (256 / 512) 37.9 / 44.5, 384 of 4096 (638 / 512) 151 / 151, k_s = 48 182 / 183.  Up to 8 tiles a unit they are the same
// workgroups, 400 of 300 38.4 / 40.0, 1024 of 64 36.1 / 36.5.
// half_wgs: not 0 where two workgroups may share a run of 8 tiles, and how many there are then.
struct GramPlan { int nwg, tiles_per_wg; GramKind kind; int half_wgs; };
// Tiles a workgroup: even shares, not below 8 (512 rows), since every partial costs a 40 KB round trip.
int run_of(long long total, int wgs) { return (int)std::max((total + wgs - 1) / wgs, 2ll * GRAM_HALF_RUN); }

// Partials that workgroups of `run` tiles leave: one for every head and every workgroup, less where both begin with the same tile.
long long partials_left(const SegTable &T, int run) {
  const long long total = total_tiles(T);
  long long pieces = T.nheads + (total + run - 1) / run, first = 0;
  for (int i = 0; i < T.nseg; ++i) {
    const int tph = tiles_of(T.s[i].n), heads = T.s[i].head_count, step = tph % run;
    int at = (int)(first % run), cycle = 0, rest = 0;      // the place in a run where a head begins comes again after `run` heads
    for (int h = 0; h < std::min(heads, run); ++h) {
      cycle += at == 0;
      rest += at == 0 && h < heads % run;
      at = at + step < run ? at + step : at + step - run;
    }
    pieces -= (long long)(heads / run) * cycle + rest;
    first += (long long)tph * heads;
  }
  return pieces;
}

GramPlan gram_plan(const compactor_params_t *p, const SegTable &T, int cus) {
  const long long total = total_tiles(T);
  const bool exact = p->sketch_dim == 0;
  const int plain_most = T.nheads <= 16 ? (exact ? 32 : 24) : T.nheads <= 32 ? (exact ? 32 : 16) : 0;
  const bool plain = total >= 8ll * cus && total < (long long)plain_most * cus;
  bool one = total < 112ll * cus;
  if (one && T.nheads >= cus && total > 8ll * cus && p->gram_wgs <= 0)
    one = partials_left(T, run_of(total, 2 * cus)) > partials_left(T, run_of(total, cus));
  GramPlan g;
  long long want = p->gram_wgs > 0 ? p->gram_wgs : (one ? 1ll : 2ll) * cus;
  if (want > total) want = total;
  if (want < 1) want = 1;
  g.tiles_per_wg = (int)((total + want - 1) / want);
  // Not below 8 tiles (512 rows) a workgroup: every partial costs a 40 KB round trip; in small calls 4, where the run is what
  // takes longest, if the workspace has room for the partials.  compactor_score, us with 4 / 8 tiles: one head of 2048 24.7 / 26.9,
  // 4096 25.6 / 27.6, 8192 27.1 / 28.3, 8 of 1024 25.0 / 27.3, 2048 26.3 / 27.7, 4096 (512 tiles) 28.1 / 28.8, 64 of 512 30.7 / 31.9, 136 of
  // 128 31.6 / 35.5, 256 of 64 34.0 / 39.8; beyond 512 tiles the partials cost more, 8 of 8192 32.8 / 31.7, 64 of 1024 36.0 / 35.4, as in
  // exact mode, 8 of 4096 46.5 / 45.6.
  if (g.tiles_per_wg < 2 * GRAM_HALF_RUN && p->gram_wgs <= 0) g.tiles_per_wg = 2 * GRAM_HALF_RUN;
  const bool halves = !exact && p->gram_wgs <= 0 && total <= 2ll * cus;
  g.kind = !one ? GRAM_TWO : plain || g.tiles_per_wg <= 4 ? GRAM_ONE : halves ? GRAM_HALVES : GRAM_FOLD;
  g.nwg = (int)((total + g.tiles_per_wg - 1) / g.tiles_per_wg);
  g.half_wgs = halves ? (int)((total + GRAM_HALF_RUN - 1) / GRAM_HALF_RUN) : 0;
  return g;
}

long long key_rows(const SegTable &T) {
  long long rows = 0;
  for (int i = 0; i < T.nseg; ++i) rows += (long long)T.s[i].n * T.s[i].head_count;
  return rows;
}

// Sketched mode, few heads: one workgroup per unit, which then factors its head itself (score_solves), as long as
// no run is much longer than the even share of a unit; not below 256 tokens, where half the run changes nothing any
// more.  compactor_score on MI355X, us with runs of 128 / 256 / 384 / 512 / 768 / 1024 tokens, k_s = 48: one head of 8192
// 30.2 / 31.4 / 32.8 / 33.4 / 35.8 / 38.0, 8 heads of 4096 32.3 / 32.7 / 33.8 / 34.5 / 36.6 / 38.4, 8192 37.9 / 36.3 / 36.6 /
// 37.5 / 39.5 / 41.1, 16384 48.1 / 45.0 / 47.3 / 42.3 / 44.7 / 46.4, 32768 63.4 / 60.2 / 62.5 / 55.7 / 57.7 / 53.4.  Against
// the search of score_tokens_for, whose workgroups get W^T from a kernel of its own, with k_s = 16, 48 and 64: 8 heads of 40007
// 50.3 / 54.7, 60.0 / 65.0, 69.6 / 74.5, 65536 65.3 / 67.5, 76.0 / 79.1, 87.9 / 87.5, 100000 89.6 / 92.4, 99.3 / 102.3, 112.3 / 112.3,
// 32 heads of 30000 99.6 / 99.2, 111.0 / 110.7, 125.4 / 119.5.
// The same runs where the workspace has no room for the shares (the sums of a blend are parted as the runs are, and its
// scores are the same bits either way): the factorisation then costs 15 to 27 us more whatever the runs.  us without room with
// these runs / the best of 512 to 4096 tokens, k_s = 48: 8 heads of 8192 55.7 / 57.2, 16384 68.8 / 68.8, 32768 79.6 / 79.5,
// 40007 86.6 / 86.4, 65536 99.8 / 99.7, 100000 125.4 / 126.5, 32 of 8192 70.4 / 70.4, 30000 128.8 / 128.2, 128 of 4096 90.7 /
// 90.4.
// 0: no such runs.
int unit_run(const compactor_params_t *p, const SegTable &T, int cus) {
  if (p->sketch_dim == 0 || T.nheads > cus) return 0;
  const int most = p->sketch_dim <= 48 ? SCORE_BURST : 1536;
  const long long rows = key_rows(T), even = (rows + cus - 1) / cus;
  int run = even > most ? most + 1 : (int)(even + SCORE_STEP - 1) / SCORE_STEP * SCORE_STEP;
  if (run < 256) run = 256;
  while (run <= most && total_blocks(T, run, SCORE_STEP, false) > cus) run += SCORE_STEP;
  return run <= most && (run == 256 || (run - 256ll) * cus <= rows) ? run : 0;
}

// Score: workgroups of equal token runs inside a head, 2 (exact mode: 3) per compute unit at a time.  A launch
// of W workgroups takes ceil(W / slots) rounds; the run length is chosen to keep the last
// round full and the per-workgroup fixed cost (staging W^T, about 32 KB) small.
int score_tokens_for(const compactor_params_t *p, const SegTable &T, int cus) {
  if (p->score_tokens > 0) {
    const int t = (p->score_tokens + SCORE_STEP - 1) / SCORE_STEP * SCORE_STEP;
    return t > SCORE_MAX_RUN ? SCORE_MAX_RUN : t;
  }
  // Sketched mode: one burst per workgroup (measured on MI355X: runs of two bursts are 2 to 9 %
  // slower, the barriers around a burst in mid-run cost more than the longer run saves, and many
  // short workgroups balance the CUs better).  Exact mode: three workgroups a unit, runs of up to 16384
  // tokens; compactor_score, us with runs of 512 / 1024 / 2048 / 4096 / 8192 tokens and those of the search below, 32
  // heads of 50001 196 / 194 / 202 / 200 / 233 and 189, 256 of 16384 415 / 405 / 397 / 414 / 408 and 397.
  const int cap = p->sketch_dim == 0 ? 16384 : SCORE_BURST;
  const int slots = (p->sketch_dim == 0 ? 3 : 2) * cus;
  const long long rows = key_rows(T);
  if (const int run = unit_run(p, T, cus)) return run;
  // A call of few heads that gives a compute unit less than 1024 tokens is all latency: one workgroup per
  // unit.  Whole call on MI355X, exact mode, us with runs of 128 / 256 / 512 / 768 / 1024 tokens, 8 heads of 8192
  // 80.0 / 79.8 / 82.1 / 86.5 / 90.3.
  if (T.nheads <= cus && rows < 1024ll * cus) {
    const int even = (int)((rows + cus - 1) / cus + SCORE_STEP - 1) / SCORE_STEP * SCORE_STEP;
    return even < 256 ? 256 : even;
  }
  int best = cap;
  double best_score = -1.0;
  for (int c = cap; c >= 1024; c -= SCORE_STEP) {
    const double w = (double)total_blocks(T, c, SCORE_STEP, false);
    const double rounds = ceil(w / slots);
    const double score = w / (rounds * slots) * (c * 256.0) / (c * 256.0 + 32768.0);
    if (score > best_score + 1e-9) { best_score = score; best = c; }
  }
  return best;
}

SolvePlan solve_plan_for(const compactor_params_t *p, const SegTable &T, const GramPlan &gp, int cus) {
  bool in_score = false;
  if (p->sketch_dim > 0 && T.nheads > DIRECT_HEADS && T.nheads <= cus)
    in_score = p->score_tokens > 0 ? score_solves(T, p->sketch_dim, score_tokens_for(p, T, cus), cus) : unit_run(p, T, cus) > 0;
  return solve_plan(T, p->sketch_dim, gp.tiles_per_wg, gp.half_wgs > 0, in_score, cus);
}

// What a group's launches are, and the bytes of workspace that they need.
struct GroupBytes {
  GramPlan gram;
  SolvePlan solve;
  size_t partials, wt, hist1, sel, bstat, scores;   // in this order in the workspace
  size_t shares, halves; // and, where the workspace has room for one or both, scratch that speeds up the factorisation, and
                         // partials of half runs (the results do not depend on them)
  size_t total() const { return partials + wt + hist1 + sel + bstat + scores; }
  size_t off_wt() const { return partials; }
  size_t off_hist1() const { return off_wt() + wt; }
  size_t off_sel() const { return off_hist1() + hist1; }
  size_t off_bstat() const { return off_sel() + sel; }
  size_t off_scores() const { return off_bstat() + bstat; }
  size_t off_shares() const { return total(); }
  size_t off_halves() const { return total() + shares; }
  size_t with_shares() const { return total() + shares; }
  size_t with_halves() const { return total() + shares + halves; }
};

size_t partial_bytes(const SegTable &T, long long wgs) {
  return align_up((size_t)(wgs + T.nheads) * GRAM_PARTIAL_FLOATS * sizeof(float));
}

// Heads up to which there are shares (see below).
int share_heads(int ks, int cus) { return ks > 0 ? cus : 3 * cus / 8; }

// demand: only what total() counts is wanted, no plan of the factorisation.
GroupBytes group_bytes_needed(const compactor_params_t *p, const SegTable &T, bool need_scores, bool demand = false) {
  const int ks = p->sketch_dim;
  const int m = ks > 0 ? ks : D;
  const int cus = compute_units();
  GroupBytes g;
  g.gram = gram_plan(p, T, cus);
  g.solve = demand ? SolvePlan{} : solve_plan_for(p, T, g.gram, cus);
  g.partials = partial_bytes(T, g.gram.nwg);
  // Many workgroups per head form S = Phi^T G Phi (exact mode: G) only where the heads alone do not fill
  // the chip.  Factorisation stage on MI355X, us with / without shares, n = 2048:
  //   heads         8           64          128         256         512         1024       2048       4096
  //   k_s = 16  12.7/18.9   14.6/19.6   16.4/20.2   18.0/18.4   21.7/20.0   33.2/32.2  60.0/56.2   110/105
  //   k_s = 48  22.8/37.6   27.5/39.3   30.9/39.5   36.9/38.9   54.9/51.5   95.3/94.0   176/182    336/358
  //   k_s = 64  30.4/52.0   36.6/54.0   43.8/54.0   54.4/52.6   85.8/76.4    157/142    309/277    596/534
  //   exact     37.7/38.9   40.0/40.2   43.4/41.4   46.4/38.4   81.9/69.6    156/135    303/271    600/532
  // and in exact mode 41.8/45.8 at 64 heads of 4096, 42.5/43.4 at 96, 42.9/41.2 at 128; k_s = 48, one head
  // of n = 131072, which brings 64 partials: 27 against 210.  At 2048 heads and more k_s = 32 and 48 would
  // be 4 to 9 % of this stage faster with shares, for 60 KB of scratch a head: the stage is 2 % of such calls.
  // (Figures of sketched mode from before sketch_direct_kernel, which takes most calls of more than 128 heads now, without shares.)
  g.shares = !demand && T.nheads <= share_heads(ks, cus) && !g.solve.direct ? align_up(g.solve.share_bytes) : 0;
  g.wt = align_up((size_t)T.nheads * W_TERMS * m * D * sizeof(uint16_t));
  g.hist1 = align_up((size_t)T.nheads * HIST1_BINS * sizeof(int));
  g.sel = select_needs_pools(T) ? align_up((size_t)select_scratch(T).ints() * sizeof(int)) : 0;
  // the blend's sums: four doubles per score workgroup
  g.bstat = 0;
  if (blend_wanted(T))
    g.bstat = align_up((size_t)total_blocks(T, score_tokens_for(p, T, compute_units()), SCORE_STEP, false) *
                       4 * sizeof(double));
  g.scores = need_scores ? align_up((size_t)key_rows(T) * sizeof(float)) : 0;
  g.halves = g.gram.half_wgs > 0 && (g.shares > 0 || g.solve.direct) ? partial_bytes(T, g.gram.half_wgs) : 0;
  return g;
}

// What compactor_workspace_size counts.  A workspace is often asked for at the greatest lengths and used for shorter ones, which
// may need more of something: runs are whole tiles (one head of 2048 tiles has 256 of them, of 2049 228), small calls have half runs,
// and the workgroups of a score launch change with the lengths.  So this holds any call of the same heads at lengths of the same
// proportions (and shares, where only other proportions lead to them).
size_t bytes_asked(const compactor_params_t *p, const SegTable &T, bool need_scores) {
  const GroupBytes g = group_bytes_needed(p, T, need_scores);
  const long long cus = compute_units(), total = total_tiles(T);
  const long long most_wgs = p->gram_wgs > 0 ? p->gram_wgs : total < 112 * cus && T.nheads < cus ? cus : 2 * cus;
  const int least_run = p->gram_wgs > 0 ? 1 : 2 * GRAM_HALF_RUN;
  auto runs = [&](int tiles, long long most) { return std::min((total + tiles - 1) / tiles, most); };
  auto shares = [&](long long wgs, bool halves) {
    if (T.nheads > share_heads(p->sketch_dim, (int)cus)) return (size_t)0;
    return align_up(share_bytes_most(T, p->sketch_dim, least_run, wgs, halves, (int)cus));
  };
  size_t rest = g.total() - g.partials;
  if (g.bstat > 0) {
    // runs are of 1024 tokens or more, or one a unit
    rest += std::max(g.bstat, align_up((size_t)(key_rows(T) / 1024 + cus + T.nheads) * 4 * sizeof(double))) - g.bstat;
  }
  size_t asked = std::max(g.with_halves(), rest + shares(most_wgs, false) + partial_bytes(T, runs(least_run, most_wgs)));
  if (p->sketch_dim > 0 && p->gram_wgs <= 0 && T.nheads <= 2 * cus)       // (more heads are more tiles)
    asked = std::max(asked, rest + shares(cus / 4, true) + partial_bytes(T, runs(2 * GRAM_HALF_RUN, cus / 4)) +
                                partial_bytes(T, runs(GRAM_HALF_RUN, cus / 2)));
  return asked;
}

// Walks the batch in head order and cuts it into launch groups of about group_rows key rows
// (at most MAX_SEG request pieces each).  fn(T, group_score_rows) is called per group; with
// local_scores the segments' score offsets address a group-local buffer.
template <class F>
int for_each_group(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                   long long group_rows, bool local_scores, F &&fn) {
  const int LH = p->layers * p->kv_heads;
  if ((long long)nreq * LH > 0x7fffffffll) return COMPACTOR_EINVAL;   // heads are numbered in int
  long long score_off = 0, kept_off = 0;
  int b = 0, h = 0;
  while (b < nreq) {
    SegTable T;
    memset(&T, 0, sizeof(T));
    T.layer_scope = p->select_scope == COMPACTOR_SCOPE_LAYER;
    const int unit = T.layer_scope ? p->kv_heads : 1;     // heads are taken in whole pools
    long long rows = 0, local_off = 0;
    while (b < nreq && T.nseg < MAX_SEG && rows < group_rows) {
      const compactor_request_t &r = reqs[b];
      const int kk = compactor_keep_count(r.n, r.ratio);
      long long can = (group_rows - rows + r.n - 1) / r.n;
      can = (can + unit - 1) / unit * unit;
      if (can < unit) can = unit;
      const int take = (int)(can < (long long)(LH - h) ? can : (long long)(LH - h));
      Seg &s = T.s[T.nseg++];
      s.k_score = static_cast<const uint16_t *>(r.k_score);
      s.k_cache = static_cast<const uint16_t *>(r.k_cache);
      s.v_cache = static_cast<const uint16_t *>(r.v_cache);
      s.attn = r.attn;
      s.stride_l = r.stride_l; s.stride_h = r.stride_h; s.stride_t = r.stride_t;
      s.score_off = local_scores ? local_off - (long long)h * r.n : score_off;
      s.kept_off = kept_off;
      s.n = r.n; s.k_keep = kk;
      s.head_begin = h; s.head_count = take;
      s.ghead0 = b * LH; s.lhead0 = T.nheads; s.H = p->kv_heads; s.req = b;
      T.nheads += take;
      rows += (long long)take * r.n;
      local_off += (long long)take * r.n;
      h += take;
      if (h == LH) {
        score_off += (long long)LH * r.n;
        kept_off += (long long)LH * kk;
        h = 0;
        ++b;
      }
    }
    index_chunks(T);
    const int rc = fn(T, rows);
    if (rc != COMPACTOR_OK) return rc;
  }
  return COMPACTOR_OK;
}

// Key rows per head group: an explicit group_bytes wins, otherwise the whole call is one group.
long long group_rows_of(const compactor_params_t *p) {
  if (p->group_bytes > 0) {
    const long long r = p->group_bytes / (D * 2);
    return r < 1 ? 1 : r;
  }
  return DEFAULT_GROUP_BYTES / (D * 2);
}

// Bytes of workspace a call needs: what its largest head group needs (groups run one after the
// other on the stream and reuse the workspace).  wanted: what compactor_workspace_size reports.
int workspace_need(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                   bool local_scores, bool wanted, size_t *bytes) {
  size_t need = 0;
  const int rc = for_each_group(p, reqs, nreq, group_rows_of(p), local_scores,
                                [&](const SegTable &T, long long) {
                                  const size_t t = wanted ? bytes_asked(p, T, local_scores)
                                                          : group_bytes_needed(p, T, local_scores, true).total();
                                  if (t > need) need = t;
                                  return COMPACTOR_OK;
                                });
  *bytes = need;
  return rc;
}

// The launchers report hipGetLastError(), which also returns an error that an earlier, unrelated
// HIP call left pending on this thread.  Every enqueueing entry point discards such a leftover
// first, so that COMPACTOR_EHIP always speaks of the library's own calls.
inline void drop_pending_error() { (void)hipGetLastError(); }

#define HIP_TRY(expr)                                \
  do {                                               \
    if ((expr) != hipSuccess) return COMPACTOR_EHIP; \
  } while (0)

// Optional profiling events (compactor_params_t.stage_events): mark(i) records event i.
struct Marks {
  void **ev;
  hipStream_t st;
  int mark(int i) const {
    if (ev && ev[i] && hipEventRecord(static_cast<hipEvent_t>(ev[i]), st) != hipSuccess)
      return COMPACTOR_EHIP;
    return COMPACTOR_OK;
  }
};
#define MARK(m, i)                       \
  do {                                   \
    const int rc_ = (m).mark(i);         \
    if (rc_ != COMPACTOR_OK) return rc_; \
  } while (0)

// score (+ blend) of one group; gb describes the workspace.  With want_hist1 the per-pool histogram of the top 12 key bits
// of the final scores is left at gb.off_hist1() of the workspace (for the selection).
int enqueue_score(const compactor_params_t *p, const SegTable &T, const GroupBytes &gb, float *scores,
                  int32_t *status, unsigned char *ws, size_t ws_bytes, hipStream_t st, bool want_hist1) {
  uint16_t *wt = reinterpret_cast<uint16_t *>(ws + gb.off_wt());
  int *hist1 = want_hist1 ? reinterpret_cast<int *>(ws + gb.off_hist1()) : nullptr;
  double *ostat = gb.bstat ? reinterpret_cast<double *>(ws + gb.off_bstat()) : nullptr;
  // the histogram is cleared on the way, by the factorisation kernel
  int *zero = hist1;
  const long long zero_ints = hist1 ? (long long)T.nheads * HIST1_BINS : 0;
  const int cus = compute_units();
  const GramPlan &gp = gb.gram;
  const SolvePlan &plan = gb.solve;
  const int rpw = gp.tiles_per_wg;
  const Marks m{p->stage_events, st};
  MARK(m, 0);
  double *shares =
      gb.shares > 0 && ws_bytes >= gb.with_shares() ? reinterpret_cast<double *>(ws + gb.off_shares()) : nullptr;
  const bool halves = gb.halves > 0 && ws_bytes >= gb.with_halves();
  float *partials = reinterpret_cast<float *>(halves ? ws + gb.off_halves() : ws);
  if (halves) {
    HIP_TRY(launch_gram(T, gp.half_wgs, GRAM_HALF_RUN, GRAM_HALF, partials, st));
  } else {
    HIP_TRY(launch_gram(T, gp.nwg, gp.tiles_per_wg, gp.kind, partials, st));
  }
  MARK(m, COMPACTOR_STAGE_GRAM + 1);
  MARK(m, COMPACTOR_STAGE_REDUCE + 1);       // the fp64 sum of the partials is part of the next kernel
  const int score_tokens = score_tokens_for(p, T, cus);
  const bool in_score = shares != nullptr && !plan.direct && score_solves(T, p->sketch_dim, score_tokens, cus);
  if (p->sketch_dim > 0) {
    HIP_TRY(launch_sketch_solve(T, p->sketch_dim, rpw, plan, partials, halves, shares, p->phi, p->ridge_rel,
                                in_score ? nullptr : wt, status, zero, zero_ints, st));
  } else {
    HIP_TRY(launch_exact_solve(T, rpw, partials, shares, p->ridge_rel, wt, status, zero, zero_ints, st));
  }
  MARK(m, COMPACTOR_STAGE_SOLVE + 1);
  const ScoreSolve solve{shares, plan.nshares, p->phi, p->ridge_rel};
  HIP_TRY(launch_score(T, p->sketch_dim, score_tokens, wt, in_score ? &solve : nullptr, scores, status, hist1, ostat,
                       st));
  MARK(m, COMPACTOR_STAGE_SCORE + 1);
  if (ostat != nullptr) {
    HIP_TRY(launch_blend(T, p->lambda_blend, score_tokens, scores, ostat, hist1, st));
  }
  MARK(m, COMPACTOR_STAGE_BLEND + 1);
  return COMPACTOR_OK;
}

// Scratch of compactor_compress_static: part of the device image, one copy per GPU.  In host
// code the array's name is only a handle for hipGetSymbolAddress; the device address it yields
// (per device) is what kernels, and everything else that touches the memory, are given.
constexpr size_t STATIC_SCRATCH_BYTES = COMPACTOR_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[MAX_DEVICES];      // device address of `scratch` on each GPU, once looked up

// Address of the current device's copy of `scratch` (looked up once per device).
int static_scratch(void **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return COMPACTOR_EHIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr)
      return COMPACTOR_EHIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return COMPACTOR_OK;
}

// Argument checks of the fused call (everything but the workspace).
int check_compress(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                   const int32_t *kept_idx, const int32_t *kept_cnt, const void *k_packed,
                   const void *v_packed, const int32_t *status) {
  int rc = check_params(p, true);
  if (rc) return rc;
  rc = check_requests(reqs, nreq, NEED_SCORE | NEED_PACK);
  if (rc) return rc;
  rc = check_scope(p, reqs, nreq);
  if (rc) return rc;
  if (!kept_idx || !kept_cnt || !k_packed || !v_packed || !status) return COMPACTOR_EINVAL;
  if (!aligned16(k_packed) || !aligned16(v_packed)) return COMPACTOR_EALIGN;
  return COMPACTOR_OK;
}

// score -> select -> gather of every head group on `st`, scratch in [workspace, +workspace_bytes).
int enqueue_compress(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                     float *scores, int32_t *kept_idx, int32_t *kept_cnt, void *k_packed,
                     void *v_packed, int32_t *status, void *workspace, size_t workspace_bytes,
                     hipStream_t st) {
  const bool local_scores = scores == nullptr;
  size_t need;
  const int rc = workspace_need(p, reqs, nreq, local_scores, false, &need);
  if (rc) return rc;
  if (!workspace || workspace_bytes < need) return COMPACTOR_EWORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & (WS_ALIGN - 1)) return COMPACTOR_EALIGN;
  drop_pending_error();
  unsigned char *ws = static_cast<unsigned char *>(workspace);
  return for_each_group(p, reqs, nreq, group_rows_of(p), local_scores,
                        [&](const SegTable &T, long long) {
    float *sc = scores;
    const GroupBytes gb = group_bytes_needed(p, T, local_scores);
    if (local_scores) sc = reinterpret_cast<float *>(ws + gb.off_scores());
    const int rc2 = enqueue_score(p, T, gb, sc, status, ws, workspace_bytes, st, true);
    if (rc2) return rc2;
    const Marks m{p->stage_events, st};
    int *hist1 = reinterpret_cast<int *>(ws + gb.off_hist1());
    if (select_needs_pools(T)) {
      int *sel = reinterpret_cast<int *>(ws + gb.off_sel());
      HIP_TRY(launch_select_pools(T, sc, hist1, nullptr, sel, kept_idx, kept_cnt, st));
    } else {
      HIP_TRY(launch_select(T, sc, hist1, kept_idx, kept_cnt, st));
    }
    MARK(m, COMPACTOR_STAGE_SELECT + 1);
    HIP_TRY(launch_gather(T, kept_idx, kept_cnt, static_cast<uint16_t *>(k_packed),
                          static_cast<uint16_t *>(v_packed), st));
    MARK(m, COMPACTOR_STAGE_GATHER + 1);
    return (int)COMPACTOR_OK;
  });
}

}  // namespace

extern "C" {
#pragma GCC visibility push(default)

void compactor_default_params(compactor_params_t *p, int32_t layers, int32_t kv_heads) {
  if (!p) return;
  memset(p, 0, sizeof(*p));
  p->layers = layers;
  p->kv_heads = kv_heads;
  p->head_dim = D;
  p->sketch_dim = 48;
  p->phi = nullptr;
  p->ridge_rel = 0.f;
  p->lambda_blend = 0.3f;
  p->group_bytes = 0;
  p->gram_wgs = 0;
  p->score_tokens = 0;
  p->select_scope = COMPACTOR_SCOPE_HEAD;
  p->stage_events = nullptr;
}

int32_t compactor_keep_count(int32_t n, float ratio) {
  if (n <= 0) return 0;
  const double x = ((double)ratio * (double)n) * (1.0 - 0x1p-23);
  double k = ceil(x);
  if (!(k >= 1.0)) k = 1.0;
  if (k > (double)n) k = (double)n;
  return (int32_t)k;
}

int compactor_layout(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                     int64_t *score_off, int64_t *kept_off, int32_t *k_keep) {
  int rc = check_params(p, false);
  if (rc) return rc;
  rc = check_requests(reqs, nreq, 0);
  if (rc) return rc;
  const long long LH = (long long)p->layers * p->kv_heads;
  long long so = 0, ko = 0;
  for (int b = 0; b < nreq; ++b) {
    const int kk = compactor_keep_count(reqs[b].n, reqs[b].ratio);
    if (score_off) score_off[b] = so;
    if (kept_off) kept_off[b] = ko;
    if (k_keep) k_keep[b] = kk;
    so += LH * reqs[b].n;
    ko += LH * kk;
  }
  if (score_off) score_off[nreq] = so;
  if (kept_off) kept_off[nreq] = ko;
  return COMPACTOR_OK;
}

int compactor_srht_phi(int32_t sketch_dim, const uint8_t *signs, const int32_t *cols, float *phi,
                       void *stream) {
  if (!(sketch_dim == 16 || sketch_dim == 32 || sketch_dim == 48 || sketch_dim == 64))
    return COMPACTOR_EUNSUPPORTED;
  if (!signs || !cols || !phi) return COMPACTOR_EINVAL;
  if (!aligned16(phi)) return COMPACTOR_EALIGN;
  bool seen[D] = {false};
  for (int j = 0; j < sketch_dim; ++j) {
    if (cols[j] < 0 || cols[j] >= D || seen[cols[j]]) return COMPACTOR_EINVAL;
    seen[cols[j]] = true;
  }
  drop_pending_error();
  HIP_TRY(launch_srht_phi(sketch_dim, signs, cols, phi, static_cast<hipStream_t>(stream)));
  return COMPACTOR_OK;
}

int compactor_workspace_size(const compactor_params_t *p, const compactor_request_t *reqs,
                             int32_t nreq, size_t *bytes) {
  if (!bytes) return COMPACTOR_EINVAL;
  int rc = check_params(p, false);
  if (rc) return rc;
  rc = check_requests(reqs, nreq, 0);
  if (rc) return rc;
  // sized for the fused call that keeps its scores in the workspace, the largest user
  return workspace_need(p, reqs, nreq, true, true, bytes);
}

int compactor_score(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                    float *scores, int32_t *status, void *workspace, size_t workspace_bytes,
                    void *stream) {
  int rc = check_params(p, true);
  if (rc) return rc;
  rc = check_requests(reqs, nreq, NEED_SCORE);
  if (rc) return rc;
  if (!scores || !status) return COMPACTOR_EINVAL;
  size_t need;
  rc = workspace_need(p, reqs, nreq, false, false, &need);
  if (rc) return rc;
  if (!workspace || workspace_bytes < need) return COMPACTOR_EWORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & (WS_ALIGN - 1)) return COMPACTOR_EALIGN;
  drop_pending_error();
  unsigned char *ws = static_cast<unsigned char *>(workspace);
  hipStream_t st = static_cast<hipStream_t>(stream);
  return for_each_group(p, reqs, nreq, group_rows_of(p), false,
                        [&](const SegTable &T, long long) {
                          return enqueue_score(p, T, group_bytes_needed(p, T, false), scores, status, ws,
                                               workspace_bytes, st, false);
                        });
}

int compactor_select(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                     const float *scores, int32_t *kept_idx, int32_t *kept_cnt,
                     void *workspace, size_t workspace_bytes, void *stream) {
  int rc = check_params(p, false);
  if (rc) return rc;
  rc = check_requests(reqs, nreq, 0);
  if (rc) return rc;
  rc = check_scope(p, reqs, nreq);
  if (rc) return rc;
  if (!scores || !kept_idx || !kept_cnt) return COMPACTOR_EINVAL;
  // only a pooled selection (long heads, layer scope) uses the workspace: for the tally where there is one, then its
  // lists, records and states
  const long long grows = group_rows_of(p);
  auto tally_bytes = [](const SegTable &T) {
    return select_by_tally(T) ? align_up((size_t)select_scratch(T).pools * HIST1_BINS * sizeof(int)) : 0;
  };
  size_t need = 0;
  rc = for_each_group(p, reqs, nreq, grows, false, [&](const SegTable &T, long long) {
    if (select_needs_pools(T)) {
      const size_t bytes = tally_bytes(T) + align_up((size_t)select_scratch(T).ints() * sizeof(int));
      if (bytes > need) need = bytes;
    }
    return COMPACTOR_OK;
  });
  if (rc) return rc;
  if (need > 0) {
    if (!workspace || workspace_bytes < need) return COMPACTOR_EWORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & (WS_ALIGN - 1)) return COMPACTOR_EALIGN;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  drop_pending_error();
  return for_each_group(p, reqs, nreq, grows, false, [&](const SegTable &T, long long) {
    if (select_needs_pools(T)) {
      const size_t tb = tally_bytes(T);
      int *tally = tb > 0 ? static_cast<int *>(workspace) : nullptr;
      int *sel = reinterpret_cast<int *>(static_cast<unsigned char *>(workspace) + tb);
      HIP_TRY(launch_select_pools(T, scores, nullptr, tally, sel, kept_idx, kept_cnt, st));
    } else {
      HIP_TRY(launch_select(T, scores, nullptr, kept_idx, kept_cnt, st));
    }
    return COMPACTOR_OK;
  });
}

int compactor_compact(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                      const int32_t *kept_idx, const int32_t *kept_cnt, void *k_packed,
                      void *v_packed, void *stream) {
  int rc = check_params(p, false);
  if (rc) return rc;
  rc = check_requests(reqs, nreq, NEED_PACK);
  if (rc) return rc;
  rc = check_scope(p, reqs, nreq);
  if (rc) return rc;
  if (!kept_idx || !kept_cnt || !k_packed || !v_packed) return COMPACTOR_EINVAL;
  if (!aligned16(k_packed) || !aligned16(v_packed)) return COMPACTOR_EALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  drop_pending_error();
  return for_each_group(p, reqs, nreq, 1ll << 60, false, [&](const SegTable &T, long long) {
    HIP_TRY(launch_gather(T, kept_idx, kept_cnt, static_cast<uint16_t *>(k_packed),
                          static_cast<uint16_t *>(v_packed), st));
    return COMPACTOR_OK;
  });
}

int compactor_compact_paged(const compactor_params_t *p, const compactor_request_t *reqs,
                            int32_t nreq, const int32_t *kept_idx, const int32_t *kept_cnt,
                            const compactor_page_pool_t *pool, const compactor_page_table_t *tables,
                            int32_t in_place, void *stream) {
  int rc = check_params(p, false);
  if (rc) return rc;
  rc = check_requests(reqs, nreq, in_place ? 0 : NEED_PACK);
  if (rc) return rc;
  rc = check_scope(p, reqs, nreq);
  if (rc) return rc;
  if (!kept_idx || !kept_cnt || !pool || !tables) return COMPACTOR_EINVAL;
  if (!pool->k_pages || !pool->v_pages || pool->page_size < 1 || pool->num_pages < 1)
    return COMPACTOR_EINVAL;
  if (pool->page_stride < 0 || pool->layer_stride < 0 || pool->head_stride < 0 ||
      pool->slot_stride < D)
    return COMPACTOR_EINVAL;
  if (!aligned16(pool->k_pages) || !aligned16(pool->v_pages) ||
      ((pool->page_stride | pool->layer_stride | pool->head_stride | pool->slot_stride) & 7))
    return COMPACTOR_EALIGN;
  for (int b = 0; b < nreq; ++b) {
    // logical pages a head can need: all its tokens when they are read from the pages, else
    // what it can retain (in layer scope one head may take the whole layer's budget)
    const long long kk = compactor_keep_count(reqs[b].n, reqs[b].ratio);
    long long rows = p->select_scope == COMPACTOR_SCOPE_LAYER ? kk * p->kv_heads : kk;
    if (rows > reqs[b].n || in_place) rows = reqs[b].n;
    if (!tables[b].pages || tables[b].len < (rows + pool->page_size - 1) / pool->page_size)
      return COMPACTOR_EINVAL;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  drop_pending_error();
  return for_each_group(p, reqs, nreq, 1ll << 60, false, [&](const SegTable &T, long long) {
    PagePool P;
    memset(&P, 0, sizeof(P));
    P.k = static_cast<uint16_t *>(pool->k_pages);
    P.v = static_cast<uint16_t *>(pool->v_pages);
    P.page_stride = pool->page_stride; P.layer_stride = pool->layer_stride;
    P.head_stride = pool->head_stride; P.slot_stride = pool->slot_stride;
    P.page_size = pool->page_size; P.num_pages = pool->num_pages;
    for (int i = 0; i < T.nseg; ++i) {
      P.t[i].pages = tables[T.s[i].req].pages;
      P.t[i].len = tables[T.s[i].req].len;
    }
    HIP_TRY(launch_gather_paged(T, P, kept_idx, kept_cnt, in_place != 0, st));
    return COMPACTOR_OK;
  });
}

int compactor_compress(const compactor_params_t *p, const compactor_request_t *reqs, int32_t nreq,
                       float *scores, int32_t *kept_idx, int32_t *kept_cnt, void *k_packed,
                       void *v_packed, int32_t *status, void *workspace, size_t workspace_bytes,
                       void *stream) {
  const int rc = check_compress(p, reqs, nreq, kept_idx, kept_cnt, k_packed, v_packed, status);
  if (rc) return rc;
  return enqueue_compress(p, reqs, nreq, scores, kept_idx, kept_cnt, k_packed, v_packed, status,
                          workspace, workspace_bytes, static_cast<hipStream_t>(stream));
}

int compactor_compress_static(const compactor_params_t *p, const compactor_request_t *reqs,
                              int32_t nreq, float *scores, int32_t *kept_idx, int32_t *kept_cnt,
                              void *k_packed, void *v_packed, int32_t *status, void *stream) {
  int rc = check_compress(p, reqs, nreq, kept_idx, kept_cnt, k_packed, v_packed, status);
  if (rc) return rc;
  size_t need;
  rc = workspace_need(p, reqs, nreq, scores == nullptr, false, &need);
  if (rc) return rc;
  if (need > STATIC_SCRATCH_BYTES) return COMPACTOR_EWORKSPACE;
  drop_pending_error();
  void *ptr = nullptr;
  rc = static_scratch(&ptr);
  if (rc) return rc;
  return enqueue_compress(p, reqs, nreq, scores, kept_idx, kept_cnt, k_packed, v_packed, status,
                          ptr, STATIC_SCRATCH_BYTES, static_cast<hipStream_t>(stream));
}

double compactor_calibrated_ratio(double nll, double alpha, double beta, double tau) {
  const double b = alpha * nll + beta;
  double r = (b == 0.0) ? tau : 1.0 + log(tau * (1.0 - exp(-b)) + exp(-b)) / b;
  if (!(r > 0.0)) r = 4.9406564584124654e-324;
  if (r > 1.0) r = 1.0;
  return r;
}

const char *compactor_error_string(int code) {
  switch (code) {
    case COMPACTOR_OK: return "ok";
    case COMPACTOR_EINVAL: return "invalid argument";
    case COMPACTOR_EUNSUPPORTED: return "unsupported shape (head_dim must be 128; sketch_dim 0, 16, 32, 48 or 64)";
    case COMPACTOR_EWORKSPACE: return "workspace missing or too small (or the batch needs more than the static scratch)";
    case COMPACTOR_EALIGN: return "pointer or stride not 16-byte aligned";
    case COMPACTOR_EHIP: return "HIP runtime error";
    default: return "unknown error";
  }
}

const char *compactor_version(void) { return "0.1"; }

#pragma GCC visibility pop
}  // extern "C"
