// Gather-compaction: the retained K/V rows of every head, in ascending token order, copied
// into a dense packed cache (paper Sec. 3: the compressed cache consists of the retained
// key/value pairs).  Pure copy, bit exact: 16 lanes move one 256-byte row with 16-byte
// accesses, four rows per wave instruction, K and V in the same pass.
//
// Small workgroups with few rows per lane do best on this read + write stream (measured on the
// benchmark's shape with random retained sets: 128 threads x 2 rows per 16-lane group 6.1 TB/s,
// 256 x 4 5.7 TB/s, 256 x 8 2.8 TB/s): a workgroup is 2 waves and moves GATHER_ROWS = 16 rows.
#include "common.h"

namespace cmp {

constexpr int GATHER_GROUPS = GATHER_THREADS / 16;        // 16-lane groups, one row each per pass
constexpr int GATHER_PASSES = GATHER_ROWS / GATHER_GROUPS;
static_assert(GATHER_ROWS % GATHER_GROUPS == 0, "whole passes");

// Workgroup -> (segment, head, tile of GATHER_ROWS retained rows).  The gather launches many small
// workgroups, so this avoids the 64-bit divisions of the general block locator.
__device__ __forceinline__ Where locate_rows(const SegTable &T, unsigned blk) {
  Where w{0, 0, 0, 0, GATHER_ROWS};
  unsigned base = 0;
  for (int i = 0; i < T.nseg; ++i) {
    const unsigned bph = ((unsigned)T.s[i].k_keep + GATHER_ROWS - 1) / GATHER_ROWS;
    const unsigned nb = bph * (unsigned)T.s[i].head_count;
    if (blk < base + nb || i == T.nseg - 1) {
      const unsigned local = blk - base, hh = local / bph;
      w.seg = i;
      w.head = T.s[i].head_begin + (int)hh;
      w.lhead = T.s[i].lhead0 + (int)hh;
      w.tile = (int)(local - hh * bph);
      return w;
    }
    base += nb;
  }
  return w;
}

__global__ __launch_bounds__(GATHER_THREADS) void gather_kernel(const SegTable T,
                                                     const int32_t *__restrict__ kept_idx,
                                                     uint16_t *__restrict__ k_packed,
                                                     uint16_t *__restrict__ v_packed) {
  const Where w = locate_rows(T, blockIdx.x);
  const Seg &s = T.s[w.seg];
  const int k = s.k_keep;
  const long long row0 = s.kept_off + (long long)w.head * k;      // first packed row of the head
  const int32_t *idx = kept_idx + row0;
  const uint16_t *ksrc = head_ptr(s.k_cache ? s.k_cache : s.k_score, s, w.head);
  const uint16_t *vsrc = head_ptr(s.v_cache, s, w.head);
  const int chunk = threadIdx.x & 15, sub = threadIdx.x >> 4;     // GATHER_GROUPS rows per pass

  uint4 kv[GATHER_PASSES], vv[GATHER_PASSES];
#pragma unroll
  for (int p = 0; p < GATHER_PASSES; ++p) {
    const int j = w.tile * GATHER_ROWS + p * GATHER_GROUPS + sub;
    kv[p] = make_uint4(0, 0, 0, 0);
    vv[p] = make_uint4(0, 0, 0, 0);
    if (j < k) {
      const int tok = idx[j];
      if (tok >= 0 && tok < s.n) {
        const long long off = (long long)tok * s.stride_t + chunk * 8;
        kv[p] = load_stream16(ksrc + off);
        vv[p] = load_stream16(vsrc + off);
      }
    }
  }
#pragma unroll
  for (int p = 0; p < GATHER_PASSES; ++p) {
    const int j = w.tile * GATHER_ROWS + p * GATHER_GROUPS + sub;
    if (j < k) {
      const long long off = (row0 + j) * D + chunk * 8;
      store_stream16(k_packed + off, kv[p]);
      store_stream16(v_packed + off, vv[p]);
    }
  }
}

// Layer scope: the retained rows of a layer's heads are packed one head after the other, head h
// holding kept_cnt[h] rows (ragged; the counts of a layer add up to H * k_keep).  A workgroup
// takes GATHER_ROWS rows of a layer's region and looks every row's head up in the counts.
__global__ __launch_bounds__(GATHER_THREADS) void gather_layer_kernel(const SegTable T,
                                                           const int32_t *__restrict__ kept_idx,
                                                           const int32_t *__restrict__ kept_cnt,
                                                           uint16_t *__restrict__ k_packed,
                                                           uint16_t *__restrict__ v_packed) {
  int seg = 0, layer = 0, tile = 0;
  {
    int base = 0;
    for (int i = 0; i < T.nseg; ++i) {
      const int bpl = (T.s[i].H * T.s[i].k_keep + GATHER_ROWS - 1) / GATHER_ROWS;
      const int nb = bpl * (T.s[i].head_count / T.s[i].H);
      if ((int)blockIdx.x < base + nb || i == T.nseg - 1) {
        const int local = blockIdx.x - base;
        seg = i;
        layer = local / bpl;
        tile = local - layer * bpl;
        break;
      }
      base += nb;
    }
  }
  const Seg &s = T.s[seg];
  const int head0 = s.head_begin + layer * s.H;                   // first head of the layer
  const int rows = s.H * s.k_keep;
  const long long row0 = s.kept_off + (long long)head0 * s.k_keep;
  const int32_t *idx = kept_idx + row0;
  const int32_t *cnt = kept_cnt + s.ghead0 + head0;
  const int chunk = threadIdx.x & 15, sub = threadIdx.x >> 4;

  uint4 kv[GATHER_PASSES], vv[GATHER_PASSES];
#pragma unroll
  for (int p = 0; p < GATHER_PASSES; ++p) {
    const int j = tile * GATHER_ROWS + p * GATHER_GROUPS + sub;
    kv[p] = make_uint4(0, 0, 0, 0);
    vv[p] = make_uint4(0, 0, 0, 0);
    if (j < rows) {
      int h = -1, run = 0;
      for (int hh = 0; hh < s.H; ++hh) {
        const int c = cnt[hh];
        if (j < run + c) { h = hh; break; }
        run += c;
      }
      const int tok = idx[j];
      if (h >= 0 && tok >= 0 && tok < s.n) {
        const long long off = (long long)tok * s.stride_t + chunk * 8;
        kv[p] = load_stream16(head_ptr(s.k_cache ? s.k_cache : s.k_score, s, head0 + h) + off);
        vv[p] = load_stream16(head_ptr(s.v_cache, s, head0 + h) + off);
      }
    }
  }
#pragma unroll
  for (int p = 0; p < GATHER_PASSES; ++p) {
    const int j = tile * GATHER_ROWS + p * GATHER_GROUPS + sub;
    if (j < rows) {
      const long long off = (row0 + j) * D + chunk * 8;
      store_stream16(k_packed + off, kv[p]);
      store_stream16(v_packed + off, vv[p]);
    }
  }
}

// ---- paged cache as the target (and, in place, the source) ----------------------------------
// Element offset of (logical slot j, layer l, head h) of a segment's request in the page pool,
// or -1 when the block table does not cover it or names a page outside the pool.
__device__ __forceinline__ long long page_slot(const PagePool &P, int seg, int l, int h, int j) {
  const int lp = j / P.page_size, slot = j - lp * P.page_size;
  if (lp >= P.t[seg].len) return -1;
  const int pg = P.t[seg].pages[lp];
  if (pg < 0 || pg >= P.num_pages) return -1;
  return (long long)pg * P.page_stride + (long long)l * P.layer_stride +
         (long long)h * P.head_stride + (long long)slot * P.slot_stride;
}

// Retained rows from the dense source tensors into pages: retained token j of a head goes to
// logical slot j of that head.  Workgroups are dealt as in the dense gathers.
// FROM_PAGES: the second part of a compaction in place, the rows whose tokens lie beyond all destinations of their
// head (see compact_inplace_kernel).
template <bool FROM_PAGES>
__global__ __launch_bounds__(GATHER_THREADS) void gather_paged_kernel(const SegTable T, const PagePool P,
                                                           const int32_t *__restrict__ kept_idx,
                                                           const int32_t *__restrict__ kept_cnt) {
  int seg = 0, head0 = 0, tile = 0, rows = 0;       // head0: the head, or the layer's first head
  if (T.layer_scope) {
    int base = 0;
    for (int i = 0; i < T.nseg; ++i) {
      const int bpl = (T.s[i].H * T.s[i].k_keep + GATHER_ROWS - 1) / GATHER_ROWS;
      const int nb = bpl * (T.s[i].head_count / T.s[i].H);
      if ((int)blockIdx.x < base + nb || i == T.nseg - 1) {
        const int local = blockIdx.x - base, layer = local / bpl;
        seg = i;
        head0 = T.s[i].head_begin + layer * T.s[i].H;
        tile = local - layer * bpl;
        rows = T.s[i].H * T.s[i].k_keep;
        break;
      }
      base += nb;
    }
  } else {
    const Where w = locate_rows(T, blockIdx.x);
    seg = w.seg; head0 = w.head; tile = w.tile; rows = T.s[w.seg].k_keep;
  }
  const Seg &s = T.s[seg];
  const int32_t *idx = kept_idx + (s.kept_off + (long long)head0 * s.k_keep);
  const int32_t *cnt = kept_cnt + s.ghead0 + head0;
  const int chunk = threadIdx.x & 15, sub = threadIdx.x >> 4;
  const int layer = head0 / s.H;

  uint4 kv[GATHER_PASSES], vv[GATHER_PASSES];
  long long dst[GATHER_PASSES], src[GATHER_PASSES];
#pragma unroll
  for (int p = 0; p < GATHER_PASSES; ++p) {
    const int j = tile * GATHER_ROWS + p * GATHER_GROUPS + sub;
    dst[p] = src[p] = -1;
    kv[p] = make_uint4(0, 0, 0, 0);
    vv[p] = make_uint4(0, 0, 0, 0);
    if (j < rows) {
      int head = head0, jh = j, held = rows;         // head of the row, its rank and the rows of that head
      if (T.layer_scope) {
        head = -1;
        int run = 0;
        for (int hh = 0; hh < s.H; ++hh) {
          const int c = cnt[hh];
          if (j < run + c) { head = head0 + hh; jh = j - run; held = c; break; }
          run += c;
        }
      }
      const int tok = idx[j];
      if (FROM_PAGES) {
        if (head >= 0 && inplace_late(tok, held) && inplace_moves(tok, jh, s.n)) {
          src[p] = page_slot(P, seg, layer, head - layer * s.H, tok);
          dst[p] = page_slot(P, seg, layer, head - layer * s.H, jh);
          if (src[p] < 0) dst[p] = -1;
        }
      } else if (head >= 0 && tok >= 0 && tok < s.n) {
        const long long off = (long long)tok * s.stride_t + chunk * 8;
        kv[p] = load_stream16(head_ptr(s.k_cache ? s.k_cache : s.k_score, s, head) + off);
        vv[p] = load_stream16(head_ptr(s.v_cache, s, head) + off);
        dst[p] = page_slot(P, seg, layer, head - layer * s.H, jh);
      }
    }
  }
  if (FROM_PAGES) {
#pragma unroll
    for (int p = 0; p < GATHER_PASSES; ++p)
      if (dst[p] >= 0) {
        kv[p] = load_stream16(P.k + src[p] + chunk * 8);
        vv[p] = load_stream16(P.v + src[p] + chunk * 8);
      }
  }
#pragma unroll
  for (int p = 0; p < GATHER_PASSES; ++p) {
    if (dst[p] >= 0) {
      store_stream16(P.k + dst[p] + chunk * 8, kv[p]);
      store_stream16(P.v + dst[p] + chunk * 8, vv[p]);
    }
  }
}

// In place: a head's tokens already live in the pages (token t at logical slot t) and its
// retained rows move to the front.  A workgroup walks the retained list of one head in ascending
// runs: all rows of a run are read, the workgroup meets, the run is written.  A run's sources lie
// at or behind its own destinations and strictly behind those of earlier runs (kept[j] >= j,
// ascending), so nothing is overwritten before it has been read; for the same reason the next
// run's rows can be fetched while this run is being written (its sources lie behind every slot
// written so far), which keeps loads in flight across the barrier.
//
// The order binds a head's rows but not its columns: K and V, and column slices of LANES * 16 bytes
// within a row, move independently, each by a workgroup of its own.  What bounds a workgroup is the
// latency of scattered row reads, about 7 ns a row and compute unit whether 64, 128 or 256 bytes of
// it are taken and with 256 to 1024 threads alike (without the reads a pass takes a quarter of the
// time), so few heads gain from narrow slices, and many heads, which fill the chip as they are, from
// whole rows.  us on MI355X with slices of 64 / 128 / 256 bytes, n = 16384 and 30 % retained unless
// said otherwise, against one workgroup per head for both tensors: 8 heads of 131072 (20 %)
// 175 / 197 / 254 (799), 16 heads of 40007 101 / 108 / 137 (376), 32 heads 55 / 55 / 68 (158; with
// part of the pool in the last-level cache 40 / 43 / 46), 64 heads 102 / 77 / 82, 96 heads of 30000
// (50 %) 448 / 377 / 319, 128 heads 194 / 153 / 137 (211), 256 heads of 32768 708 / 588 / 527 (536).
//
// A head that keeps k rows writes its slots 0 .. k - 1 only.  Rows whose tokens lie behind those (late rows: of n
// tokens, 1 - k/n of the list, and its end) are overwritten by nothing, so where there are enough of them they move
// by a launch of their own that deals them out like a dense gather, once the early rows have been moved in order.
constexpr int INPLACE_THREADS = 512;
template <int LANES>
struct Inplace {
  static constexpr int PASSES = 8;                      // rows in flight per lane
  static constexpr int ROWS = INPLACE_THREADS / LANES;  // rows per pass
  static constexpr int RUN = ROWS * PASSES;             // rows per run
  // rows whose addresses a thread works out
  static constexpr int OWN = (RUN + INPLACE_THREADS - 1) / INPLACE_THREADS;
  static constexpr int SLICES = 16 / LANES;             // column slices of a row
};

// Elements between the starts of the K and the V row of a slot that lie inside one another's row (0: the
// same memory), or -1: K and V rows of a slot are apart, as they nearly always are.  A pool may hold both
// in one row (V a part of what K is read from); slices of K and of V would then move the shared columns
// each at its own pace, so the row from the start of the first to the end of the second moves as one.
__host__ __device__ __forceinline__ int shared_row_shift(const PagePool &P) {
  const intptr_t d = (reinterpret_cast<intptr_t>(P.v) - reinterpret_cast<intptr_t>(P.k)) / (intptr_t)sizeof(uint16_t);
  const intptr_t a = d < 0 ? -d : d;
  return a < D ? (int)a : -1;
}

// Pages of the rows j (destination) and tok (source), -1 where the row does not move.
struct RowPages { int src, dst, src_slot, dst_slot; };

// SHARED: K and V lie in one row of `pieces` 16-byte pieces from the lower of their addresses.
// EARLY: only rows whose tokens lie below the head's row count, which are those that destinations can overwrite
// and the first of the list; all others are left to gather_paged_kernel<true>.
template <int LANES, bool SHARED, bool EARLY>
__global__ __launch_bounds__(INPLACE_THREADS) void compact_inplace_kernel(
    const SegTable T, const PagePool P, int page_shift, int pieces, const int32_t *__restrict__ kept_idx,
    const int32_t *__restrict__ kept_cnt) {
  typedef Inplace<LANES> I;
  __shared__ long long src_l[3][I::RUN], dst_l[3][I::RUN];   // element offsets; -1: does not move
  __shared__ int more_l[3];                                  // EARLY: the run has rows to move
  // blocks b, b + 8, b + 16, .. (one XCD, hence one L2) hold the slices of one head
  const int parts = SHARED ? (pieces + LANES - 1) / LANES : 2 * I::SLICES;
  const int part = (blockIdx.x >> 3) % parts, oct = (blockIdx.x >> 3) / parts;
  const int hb = 8 * oct + (blockIdx.x & 7);
  if (hb >= T.nheads) return;
  const Where w = locate_block(T, hb, 0, 1, false);      // heads in launch order
  const Seg &s = T.s[w.seg];
  const int layer = w.head / s.H, h = w.head - layer * s.H;
  int rows = s.k_keep;
  long long first = s.kept_off + (long long)w.head * s.k_keep;
  if (T.layer_scope) {                  // ragged: this head's rows follow those of heads 0..h-1
    const int32_t *cnt = kept_cnt + s.ghead0 + layer * s.H;
    first = s.kept_off + (long long)layer * s.H * s.k_keep;
    for (int hh = 0; hh < h; ++hh) first += cnt[hh];
    rows = cnt[h];
  }
  const int32_t *idx = kept_idx + first;
  const int32_t *table = P.t[w.seg].pages;
  const int tlen = P.t[w.seg].len;
  const int tid = threadIdx.x;
  const int lane = tid & (LANES - 1), sub = tid / LANES;
  const int slice = SHARED ? part : part >> 1;
  uint16_t *base = (SHARED ? (P.v < P.k ? P.v : P.k) : part & 1 ? P.v : P.k) +
                   ((long long)layer * P.layer_stride + (long long)h * P.head_stride) + slice * (LANES * 8) + lane * 8;
  const bool have = !SHARED || slice * LANES + lane < pieces;

  // The address of a row takes three dependent loads (its index, two table entries); they are
  // spread over the runs before: indices three runs ahead, table entries two.  Each thread does
  // this for rows of its own and leaves the offsets in LDS for the lanes that move them.
  auto fetch_idx = [&](int run, int (&tok)[I::OWN]) {
#pragma unroll
    for (int o = 0; o < I::OWN; ++o) {
      const int jr = o * INPLACE_THREADS + tid;
      const long long j = inplace_row(run, I::RUN, jr);
      tok[o] = -1;
      if (jr < I::RUN && j < rows) {
        tok[o] = idx[j];
        if (EARLY && inplace_late(tok[o], rows)) tok[o] = INPLACE_LATE;
      }
    }
  };
  auto split = [&](int j, int &lp, int &slot) {
    if (page_shift >= 0) { lp = j >> page_shift; slot = j & (P.page_size - 1); }
    else { lp = (int)((unsigned)j / (unsigned)P.page_size); slot = j - lp * P.page_size; }
  };
  auto fetch_pages = [&](int run, const int (&tok)[I::OWN], RowPages (&pg)[I::OWN]) {
#pragma unroll
    for (int o = 0; o < I::OWN; ++o) {
      const long long j = inplace_row(run, I::RUN, o * INPLACE_THREADS + tid);
      pg[o] = RowPages{-1, -1, 0, 0};
      if (inplace_moves(tok[o], j, s.n)) {
        int lp;
        split(tok[o], lp, pg[o].src_slot);
        if (lp < tlen) pg[o].src = table[lp];
        split((int)j, lp, pg[o].dst_slot);
        if (lp < tlen) pg[o].dst = table[lp];
      }
    }
  };
  // `more`: the first row of the run is not late, so that the run may have early rows.  What a list says of that row
  // decides, not whether it moves: entries below their own rank, negative ones among them, are skipped and do not end
  // the list.  (Tokens ascend: behind a late row all are.)
  auto put_moves = [&](int slot, const RowPages (&pg)[I::OWN], bool more) {
    if (EARLY && tid == 0) more_l[slot] = more;
#pragma unroll
    for (int o = 0; o < I::OWN; ++o) {
      const int jr = o * INPLACE_THREADS + tid;
      if (jr < I::RUN) {
        const bool ok = pg[o].src >= 0 && pg[o].src < P.num_pages && pg[o].dst >= 0 && pg[o].dst < P.num_pages;
        src_l[slot][jr] = ok ? (long long)pg[o].src * P.page_stride + (long long)pg[o].src_slot * P.slot_stride : -1;
        dst_l[slot][jr] = ok ? (long long)pg[o].dst * P.page_stride + (long long)pg[o].dst_slot * P.slot_stride : -1;
      }
    }
  };
  auto load_rows = [&](int slot, uint4 (&r)[I::PASSES]) {
    long long src[I::PASSES];
#pragma unroll
    for (int p = 0; p < I::PASSES; ++p) src[p] = src_l[slot][p * I::ROWS + sub];
#pragma unroll
    for (int p = 0; p < I::PASSES; ++p) {
      r[p] = make_uint4(0, 0, 0, 0);
      if (src[p] >= 0 && have)     // whole rows are read once; a 128-byte line shared by slices may be cached
        r[p] = LANES == 16 ? load_stream16(base + src[p]) : *reinterpret_cast<const uint4 *>(base + src[p]);
    }
  };
  auto store_rows = [&](int slot, const uint4 (&r)[I::PASSES]) {
    long long dst[I::PASSES];
#pragma unroll
    for (int p = 0; p < I::PASSES; ++p) dst[p] = dst_l[slot][p * I::ROWS + sub];
#pragma unroll
    for (int p = 0; p < I::PASSES; ++p)
      if (dst[p] >= 0 && have) store_stream16(base + dst[p], r[p]);
  };

  int tok[I::OWN];
  RowPages pg[I::OWN];
  uint4 a[I::PASSES], b[I::PASSES];
  const int runs = inplace_runs(rows, I::RUN);
  fetch_idx(0, tok);
  fetch_pages(0, tok, pg);
  bool more = tok[0] != INPLACE_LATE;    // of the run whose pages pg holds (thread 0: its first row)
  fetch_idx(1, tok);
  put_moves(0, pg, more);
  fetch_pages(1, tok, pg);
  more = tok[0] != INPLACE_LATE;
  fetch_idx(2, tok);
  __syncthreads();
  load_rows(0, a);
  // on entry of step r: the rows of run r are being read, pg holds run r + 1, tok run r + 2
  auto step = [&](int r, uint4 (&cur)[I::PASSES], uint4 (&next)[I::PASSES]) {
    put_moves((r + 1) % 3, pg, more);
    // every wave waits for its own rows of run r before it meets the others (a barrier by itself
    // does not wait for loads): behind the barrier all of them have been read
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    fetch_pages(r + 2, tok, pg);
    more = tok[0] != INPLACE_LATE;
    fetch_idx(r + 3, tok);
    load_rows((r + 1) % 3, next);
    store_rows(r % 3, cur);
    return r + 1 < runs && (!EARLY || more_l[(r + 1) % 3]);        // uniform, behind the barrier
  };
  for (int r = 0; r < runs; r += 2) {
    if (!step(r, a, b)) break;
    if (!step(r + 1, b, a)) break;
  }
}

template <int LANES, bool SHARED, bool EARLY>
static hipError_t launch_inplace(const SegTable &T, const PagePool &P, const int32_t *kept_idx,
                                 const int32_t *kept_cnt, hipStream_t st, int pieces) {
  const int parts = SHARED ? (pieces + LANES - 1) / LANES : 2 * Inplace<LANES>::SLICES;
  const long long nb = ((long long)T.nheads + 7) / 8 * 8 * parts;
  if (nb > 0x7fffffffll) return hipErrorInvalidValue;
  const int shift = (P.page_size & (P.page_size - 1)) == 0 ? __builtin_ctz((unsigned)P.page_size) : -1;
  hipLaunchKernelGGL((compact_inplace_kernel<LANES, SHARED, EARLY>), dim3((unsigned)nb), dim3(INPLACE_THREADS), 0, st, T, P,
                     shift, pieces, kept_idx, kept_cnt);
  return hipGetLastError();
}

// Whether a compaction in place is cut in two (see compact_inplace_kernel): by the rows of a head that are late if
// the retained ones are spread evenly, k (1 - k / n).  The second launch costs 3 to 6 us and lets every compute
// unit take part, which is worth most to few heads and nothing around 64, where the slices of one launch are a workgroup
// for every unit as it is; more heads take several rounds of workgroups, and two launches fill the last of them better.
// MI355X, pages of 16, time in two launches over time in one, pool in memory / in the last-level cache, by late rows a head:
//   8 heads   1721 1.13 / 1.02, 3441 0.74 / 1.13, 4096 0.70 / 1.06, 5040 0.65 / 0.90, 6882 0.63 / 0.80, 15729 0.61 / 0.73
//   16        1721 0.94 / 1.15, 3441 0.79 / 0.96, 4096 0.79 / 0.96, 5040 0.73 / 0.86, 8192 0.77 / 0.88
//   24        3441 0.86 / 0.94, 5040 0.81 / 0.91, 6882 0.81 / 0.90, 8400 0.76 / 0.90
//   32        1476 1.35 / 1.06, 3441 0.92 / 1.01, 4096 0.90 / 1.00, 6000 0.87 / 0.96, 6882 0.80 / 0.95, 8192 0.87 / 0.92
//   48        6000 0.93 / 0.97, 8192 0.97 / 0.97
//   64        3441 1.04 / 1.26, 5899 1.03 / 1.04, 6882 1.04 / 1.04, 8192 0.96 / 0.96, 13763 0.92 / 0.92
//   65        2880 1.10, 3441 1.07 / 1.07;  72  3441 0.95 / 0.96, 7200 0.97;  96  2880 0.98, 3441 0.97 / 0.97, 7200 0.99
//   128       2400 1.01, 2880 1.00 / 1.00, 3441 0.99 / 0.99, 4096 1.01 / 1.01;  256  2880 0.98, 4096 0.99
// The more is retained, the less the late rows weigh: 8 heads of 65536, 60, 65 and 70 % 0.70, 0.74, 0.78, 16 of 40007, 60 and
// 70 % 0.81, 0.87 (80 % 0.99), 64 of 32768, 65 % 0.98, 128 of 16384, 65 % 1.02, 8 of 32768, 80 % 1.09, 96 of 30000, 60 and
// 80 % 0.99, 1.05.
static bool inplace_in_two(const SegTable &T) {
  long long late = 0, kept = 0, rows = 0;
  for (int i = 0; i < T.nseg; ++i) {
    const Seg &s = T.s[i];
    late += s.head_count * ((long long)s.k_keep * (s.n - s.k_keep) / s.n);
    kept += (long long)s.head_count * s.k_keep;
    rows += (long long)s.head_count * s.n;
  }
  const int least = T.nheads <= 48 ? 4800 : T.nheads <= 64 ? 8192 : 3400;
  return late >= (long long)least * T.nheads && 8 * kept <= 5 * rows;
}

hipError_t launch_gather_paged(const SegTable &T, const PagePool &P, const int32_t *kept_idx,
                               const int32_t *kept_cnt, bool in_place, hipStream_t st) {
  if (T.nheads <= 0) return hipSuccess;
  if (in_place) {
    const int shift = shared_row_shift(P);
    if (shift >= 0) return launch_inplace<16, true, false>(T, P, kept_idx, kept_cnt, st, (D + shift) / 8);
    // slices by the number of heads (see compact_inplace_kernel for the times on both sides)
    const bool two = inplace_in_two(T);
    const auto launch = T.nheads <= 16   ? (two ? launch_inplace<4, false, true> : launch_inplace<4, false, false>)
                        : T.nheads <= 64 ? (two ? launch_inplace<8, false, true> : launch_inplace<8, false, false>)
                                         : (two ? launch_inplace<16, false, true> : launch_inplace<16, false, false>);
    const hipError_t rc = launch(T, P, kept_idx, kept_cnt, st, 0);
    if (rc != hipSuccess || !two) return rc;
  }
  long long nb = 0;
  if (T.layer_scope) {
    for (int i = 0; i < T.nseg; ++i)
      nb += (long long)((T.s[i].H * (long long)T.s[i].k_keep + GATHER_ROWS - 1) / GATHER_ROWS) *
            (T.s[i].head_count / T.s[i].H);
  } else {
    nb = total_blocks(T, GATHER_ROWS, GATHER_ROWS, true);
  }
  if (nb <= 0) return hipSuccess;
  if (nb > 0x7fffffffll) return hipErrorInvalidValue;
  hipLaunchKernelGGL(in_place ? gather_paged_kernel<true> : gather_paged_kernel<false>, dim3((unsigned)nb),
                     dim3(GATHER_THREADS), 0, st, T, P, kept_idx, kept_cnt);
  return hipGetLastError();
}

hipError_t launch_gather(const SegTable &T, const int32_t *kept_idx, const int32_t *kept_cnt,
                         uint16_t *k_packed, uint16_t *v_packed, hipStream_t st) {
  if (T.layer_scope) {
    long long nb = 0;
    for (int i = 0; i < T.nseg; ++i)
      nb += (long long)((T.s[i].H * (long long)T.s[i].k_keep + GATHER_ROWS - 1) / GATHER_ROWS) *
            (T.s[i].head_count / T.s[i].H);
    if (nb <= 0) return hipSuccess;
    if (nb > 0x7fffffffll) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gather_layer_kernel, dim3((unsigned)nb), dim3(GATHER_THREADS), 0, st, T, kept_idx,
                       kept_cnt, k_packed, v_packed);
    return hipGetLastError();
  }
  const long long nb = total_blocks(T, GATHER_ROWS, GATHER_ROWS, true);
  if (nb <= 0) return hipSuccess;
  if (nb > 0x7fffffffll) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gather_kernel, dim3((unsigned)nb), dim3(GATHER_THREADS), 0, st, T, kept_idx, k_packed,
                     v_packed);
  return hipGetLastError();
}

}  // namespace cmp
