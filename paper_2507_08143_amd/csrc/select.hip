// Per-head top-k selection (paper Sec. 3.3: retain the top ceil(r N) tokens by score, within a
// single head) and the score blend of Eq. "scoring".
//
// Selection is an exact radix select on an order-preserving 32-bit key of the fp32 score (a bin of
// 17 to 23 key bits, then 12 bits and the 5 to 11 left; LDS histograms), followed by an ordered emit: tokens above the threshold
// key, plus the lowest-indexed tokens equal to it until k_keep is reached, written in
// ascending token order.  Ties therefore go to the lower index, deterministically.
// Heads of up to 32768 tokens get one workgroup of 1024 threads each, which reads the scores
// once and holds them in registers; longer heads, and selection
// across the heads of a layer, are shared by several workgroups (second half of this file).
#include "common.h"

namespace cmp {

// Inclusive prefix sum over the lanes of a wave, by moves within and across the 16-lane rows: a move costs
// a vector instruction, where a shuffle is an LDS round trip.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  constexpr int ROW_SHR = 0x110, ROW_BCAST15 = 0x142, ROW_BCAST31 = 0x143;
  v += __builtin_amdgcn_update_dpp(0, v, ROW_SHR + 1, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, ROW_SHR + 2, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, ROW_SHR + 4, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, ROW_SHR + 8, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, ROW_BCAST15, 0xa, 0xf, false);   // lane 15 to row 1, 47 to row 3
  v += __builtin_amdgcn_update_dpp(0, v, ROW_BCAST31, 0xc, 0xf, false);   // lane 31 to rows 2 and 3
  return v;
}

// Exclusive prefix sum of one int per thread over a workgroup of NT threads; *total gets the
// workgroup sum.  wsum is NT / 64 ints of LDS.
template <int NT = SELECT_THREADS>
__device__ __forceinline__ int block_exclusive_scan(int v, int *wsum, int *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = wave_inclusive_scan(v);
  __syncthreads();                       // wsum may still be read from a previous call
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    const int x = wsum[i];
    if (i < wave) base += x;
    tot += x;
  }
  *total = tot;
  return base + inc - v;
}

constexpr int WHOLE_HEAD = 32768;  // heads up to this many tokens are selected by one workgroup

// Finds, in a histogram of `nb` digits, the digit where the descending cumulative count reaches
// `need`; returns the digit and leaves in *need the count still wanted inside that digit.
// Thread t owns the PER digits first, first - 1, .. (descending, those of thread t + 1 below), so that an ascending scan
// over threads is a descending scan over digits; c[] are their counts.
template <int NT, int PER>
__device__ __forceinline__ int find_counted(const int (&c)[PER], int first, int *need, int *wsum, int *found) {
  int sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) sum += c[q];
  int total;
  int before = block_exclusive_scan<NT>(sum, wsum, &total);   // keys in higher digits
  const int want = *need;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (before < want && want <= before + c[q]) {          // exactly one (thread, q) matches
      found[0] = first - q;
      found[1] = want - before;
    }
    before += c[q];
  }
  __syncthreads();
  *need = found[1];
  return found[0];
}
template <int NT = SELECT_THREADS>
__device__ __forceinline__ int find_digit(const int *hist, int nb, int *need, int *wsum, int *found) {
  constexpr int PER = 4096 / NT;     // digits per thread (nb <= 4096)
  const int first = nb - 1 - PER * (int)threadIdx.x;
  int c[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) c[q] = first - q >= 0 ? hist[first - q] : 0;
  return find_counted<NT>(c, first, need, wsum, found);
}

// The scores of tokens [begin, end) of a head, 4 consecutive tokens per thread of NT and round (token of f[r][e]:
// begin + 4 * ((r0 + r) * NT + tid) + e); bit 4r+e of the result says that the token exists.  The loads are only issued here: whoever calls this first and converts to keys later
// has the latency of everything in between for free.
// One 16-byte load per 4 tokens also where a head's scores start off a 16-byte boundary (odd n): global memory
// takes vector loads at any 4-byte address.  No branch around a single load: each would wait for the one
// before it (112 heads of 131072 tokens, candidates 17 us with and 13 without; blend of 4 layers of 8 x 16383
// 10.3 and 7.4).  Four tokens that reach past a chunk's end are read from its last four on
// and moved into place by place_scores, after which the loads are waited for.
template <int NT, int R>
__device__ __forceinline__ void load_scores(const float *__restrict__ sp, int begin, int end, int r0,
                                            float (&f)[R][4]) {
  typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  const int at = 4 * (r0 * NT + (int)threadIdx.x), tokens = end - begin;
  if (end >= 4) {                        // uniform
    const char *base = reinterpret_cast<const char *>(sp + quad_base(begin, tokens));        // uniform
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const f32x4_any v = *reinterpret_cast<const f32x4_any *>(base + 4u * (unsigned)quad_from_base(at + 4 * r * NT, tokens));
      f[r][0] = v.x; f[r][1] = v.y; f[r][2] = v.z; f[r][3] = v.w;
    }
  } else {                               // a head of up to three tokens
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) f[r][e] = r == 0 && at + e < tokens ? sp[e] : 0.f;
  }
}
// Returns the bits of the tokens that exist; what f holds of others is any number.
template <int NT, int R>
__device__ __forceinline__ unsigned place_scores(int begin, int end, int r0, float (&f)[R][4]) {
  unsigned valid = 0xffffffffu >> (32 - 4 * R);
  const int tokens = end - begin;
  if (4 * (r0 + R) * NT > tokens) {      // uniform: some do not exist
    valid = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int have = tokens - 4 * ((r0 + r) * NT + (int)threadIdx.x);
      valid |= ((1u << min(max(have, 0), 4)) - 1u) << (4 * r);
      if (have > 0 && have < 4 && end >= 4) {
        if (have < 3) { f[r][0] = f[r][2]; f[r][1] = f[r][3]; }
        if (have != 2) { f[r][0] = f[r][1]; f[r][1] = f[r][2]; f[r][2] = f[r][3]; }
      }
    }
  }
  return valid;
}

// The float of a key (score_key's inverse; -0.0 has no key of its own).
__device__ __forceinline__ float key_score(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key);
}

// Classification of scores against a key interval [lo, hi]: bits of the tokens of f (see load_scores)
// above it and inside it; f becomes the keys' distances from lo (of those inside).  Keys of one sign are the
// float's bits with the sign set, or their complement; what lies outside wraps round to a distance beyond the
// interval.  Float comparison gives the order of the keys everywhere but at NaN (key 0, below every number)
// and just below zero (-0.0 is +0.0 but compares equal to it), and those have the general path.
template <int R, class ABOVE, class DIST>
__device__ __forceinline__ void classify_by(float (&f)[R][4], uint32_t span, unsigned &above, unsigned &in,
                                            ABOVE &&is_above, DIST &&distance) {
  above = in = 0;
#pragma unroll
  for (int r = R - 1; r >= 0; --r)
#pragma unroll
    for (int e = 3; e >= 0; --e) {
      above = above + above + (is_above(f[r][e]) ? 1u : 0u);
      const uint32_t v = distance(f[r][e]);
      in = in + in + (v <= span ? 1u : 0u);
      f[r][e] = __uint_as_float(v);
    }
}
template <int R>
__device__ __forceinline__ void classify(float (&f)[R][4], unsigned valid, uint32_t lo, uint32_t hi,
                                         unsigned &above, unsigned &in) {
  const bool positive = lo > 0x80000000u && hi <= 0xff800000u, negative = lo >= 0x007fffffu && hi < 0x7fffffffu;
  if (positive || negative) {
    const float fhi = key_score(hi);
    const uint32_t flip = positive ? 0x80000000u : 0xffffffffu;
    classify_by(f, hi - lo, above, in, [&](float x) { return x > fhi; },
                [&](float x) { return (__float_as_uint(x) ^ flip) - lo; });
  } else {
    classify_by(f, hi - lo, above, in, [&](float x) { return score_key(x) > hi; },
                [&](float x) { return score_key(x) - lo; });
  }
  above &= valid;
  in &= valid;
}

// The bits of rounds 0 .. R - 1 (4 tokens each, low nibbles of R bytes) in one word.
template <int R>
__device__ __forceinline__ unsigned nibbles(const unsigned char *by, int shift) {
  unsigned w = 0;
#pragma unroll
  for (int i = 0; i < R; ++i) w |= ((unsigned)by[i] >> shift & 0xfu) << (4 * i);
  return w;
}

// Positions and tokens of what a workgroup of NT retains of the tokens from `base` on.  keep: this thread's tokens above
// the threshold, of 32 at most that begin `first` tokens behind base; ties: those equal to it, of which the workgroup
// keeps `allow`, the first ones.  Threads hold their tokens in order.  The retained tokens are consecutive in the
// output: they are gathered in LDS (16 bits each, as many as the workgroup has tokens) and written out as one run of at
// most `limit`.
template <int NT>
__device__ __forceinline__ void emit_ordered(unsigned keep, unsigned ties, int allow, int base, int first, int limit,
                                             int *wsum, uint16_t *stage, int32_t *__restrict__ out) {
  int all_packed;                        // (above | equal << 16), at most 32768 each
  const unsigned before = (unsigned)block_exclusive_scan<NT>(__popc(keep) | (int)((unsigned)__popc(ties) << 16), wsum,
                                                             &all_packed);
  const unsigned all = (unsigned)all_packed;
  const int ties_before = (int)(before >> 16);
  for (int left = allow - ties_before; ties && left > 0; --left) {
    keep |= ties & (0u - ties);
    ties &= ties - 1;
  }
  int at = (int)(before & 0xffffu) + min(ties_before, allow);
  while (keep) {
    stage[at++] = (uint16_t)(first + __ffs(keep) - 1);
    keep &= keep - 1;
  }
  __syncthreads();
  const int total = min((int)(all & 0xffffu) + min((int)(all >> 16), allow), limit);
  for (int j = threadIdx.x; j < total; j += NT) out[j] = base + stage[j];
}

// One workgroup per head of up to 4096 R tokens, which hold their scores in registers.  HIST1: the first digit's
// histogram has come with the scores (top 12 key bits), otherwise it is tallied here by score_bin.  The keys above the
// threshold's bin and inside it become bits of two words per thread, those inside it their distance from its lowest key;
// the next digits are tallied from the latter, and a round's 4 tokens of a thread pass through LDS as a byte so that a
// thread then holds 4 R consecutive tokens and one scan gives every position.
// Bound: a chain of barriers (three for a digit) for few heads, vector issue for long ones.  Against keys in LDS, read
// again for every digit, which left room for one workgroup on a compute unit: behind the score kernel, one head of 4096
// tokens 9.6 us before and 7.0 now, 256 heads of 32768 27.1 and 23.6; on given scores, 256 heads of 32768 24.0 / 21.6,
// 512 45.9 / 43.9, 1024 of 8192 42.4 / 24.3, 2048 of 4096 67.5 / 35.2.
template <int R, bool HIST1>
__global__ __launch_bounds__(SELECT_THREADS) void select_kernel(const SegTable T,
                                                                const float *__restrict__ scores,
                                                                const int *__restrict__ hist1,
                                                                int32_t *__restrict__ kept_idx,
                                                                int32_t *__restrict__ kept_cnt) {
  constexpr int NT = SELECT_THREADS;
  union Big {
    int first[HIST1 ? 4 : HIST1_BINS];
    uint16_t stage[4 * R * NT];
  };
  union Second {
    int hist[4096];
    unsigned char quad[R * NT];
  };
  __shared__ __attribute__((aligned(16))) Big big;
  __shared__ __attribute__((aligned(16))) Second second;
  __shared__ __attribute__((aligned(16))) int third[2048];
  __shared__ int wsum[NT / 64];
  __shared__ int found[2];

  const Where w = locate_block(T, blockIdx.x, 0, 1, false);
  const Seg &s = T.s[w.seg];
  const int n = s.n, k = s.k_keep;
  const float *sp = scores + s.score_off + (long long)w.head * n;
  const int tid = threadIdx.x;
  float f[R][4];
  load_scores<NT, R>(sp, 0, n, 0, f);    // in flight while the first digit is found
  const int4 h1 = HIST1 ? *reinterpret_cast<const int4 *>(hist1 + (size_t)w.lhead * HIST1_BINS + hist_at(4092 - 4 * tid))
                        : make_int4(0, 0, 0, 0);
  if (tid == 0) kept_cnt[s.ghead0 + w.head] = k;
  *reinterpret_cast<int4 *>(&second.hist[4 * tid]) = make_int4(0, 0, 0, 0);
  *reinterpret_cast<int2 *>(&third[2 * tid]) = make_int2(0, 0);
  int need = k;
  unsigned valid;
  int bin;
  if constexpr (HIST1) {
    const int c[4] = {h1.w, h1.z, h1.y, h1.x};
    bin = find_counted<NT>(c, 4095 - 4 * tid, &need, wsum, found);
    valid = place_scores<NT, R>(0, n, 0, f);
  } else {
    *reinterpret_cast<int4 *>(&big.first[4 * tid]) = make_int4(0, 0, 0, 0);
    __syncthreads();
    valid = place_scores<NT, R>(0, n, 0, f);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (valid >> (4 * r + e) & 1) atomicAdd(&big.first[score_bin(score_key(f[r][e]))], 1);
    __syncthreads();
    bin = find_digit<NT>(big.first, HIST1_BINS, &need, wsum, found);
  }
  const BinKeys bk = bin_keys(bin, !HIST1);
  const int rest = bk.bits - 12;
  unsigned above, in;
  classify<R>(f, valid, bk.lo, bk.lo | ((1u << bk.bits) - 1u), above, in);
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (in >> (4 * r + e) & 1) atomicAdd(&second.hist[__float_as_uint(f[r][e]) >> rest], 1);
  __syncthreads();
  const uint32_t d2 = (uint32_t)find_digit<NT>(second.hist, 4096, &need, wsum, found);
  // Above the second digit, and from it on; few waves have a token inside it, and only they have more to look at.
  const uint32_t low = (1u << rest) - 1u, base2 = d2 << rest, top2 = base2 | low;
  unsigned gt = 0, eq = 0;
#pragma unroll
  for (int r = R - 1; r >= 0; --r)
#pragma unroll
    for (int e = 3; e >= 0; --e) {
      const uint32_t v = __float_as_uint(f[r][e]);
      gt = gt + gt + (v > top2 ? 1u : 0u);
      eq = eq + eq + (v >= base2 ? 1u : 0u);
    }
  gt &= in;
  unsigned at2 = eq & in & ~gt;
  const bool look = __any(at2 != 0);
  if (look) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (at2 >> (4 * r + e) & 1) atomicAdd(&third[__float_as_uint(f[r][e]) & low], 1);
  }
  __syncthreads();
  const uint32_t thr = base2 | (uint32_t)find_digit<NT>(third, 1 << rest, &need, wsum, found);
  eq = 0;
  if (look) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t v = __float_as_uint(f[r][e]);
        const unsigned bit = at2 & (1u << (4 * r + e));
        gt |= v > thr ? bit : 0u;
        eq |= v == thr ? bit : 0u;
      }
  }
  gt |= above;
#pragma unroll
  for (int r = 0; r < R; ++r)
    second.quad[r * NT + tid] = (unsigned char)((gt >> (4 * r) & 0xfu) | (eq >> (4 * r) & 0xfu) << 4);
  __syncthreads();
  unsigned char by[R];
#pragma unroll
  for (int i = 0; i < R; ++i) by[i] = second.quad[R * tid + i];
  emit_ordered<NT>(nibbles<R>(by, 0), nibbles<R>(by, 4), need, 0, 4 * R * tid, k, wsum, big.stage,
                   kept_idx + (s.kept_off + (long long)w.head * k));
}

// ---- selection by several workgroups per pool ------------------------------------------------
// Used when a head has more scores than one workgroup holds in registers, and for head-adaptive selection, where
// the pool is the H kv heads of a layer that share one budget of H * k_keep tokens (paper Sec. 3.3:
// the top scores "across all heads"; scoring stays per head).  The same radix select and ordered
// emit as above, with the scores read once or twice in all.  A pool (head or layer) is cut into chunks of
// up to 8192 tokens of one head, one workgroup each; three launches:
//   cand   a range of keys that holds the threshold: a bin of the pool's histogram (made by the score
//          kernel or the blend), or, for scores that come without one, a bin of a tally of all of them
//          (msel_hist1_kernel) or a bracket from a sample (msel_sample_kernel).  Keys above the range are retained for sure and only marked and
//          counted; the keys inside it (the candidates: 2 to 25 % of the pool unless the
//          scores are heavily tied) are marked and leave their distance from its lower end in a
//          per-chunk list
//   thr    one workgroup per pool finds the remaining bits of the threshold among the
//          candidates and derives, chunk by chunk in (head, token) order, every chunk's output
//          position and its allowance of threshold ties
//   emit   ordered emit of every chunk, from the marks and the candidates' scores
// Everything is integer work on exact counts, so the result does not depend on the order in which
// candidates are listed.  A chunk workgroup's chain (locate, load, classify, write) is latency
// bound, so the chunk kernels are small workgroups of 256 threads held to 64 or 72 registers: seven or
// eight of them share a CU and overlap each other's waits (1024-thread workgroups on 32768-token chunks
// moved 2.4 TB/s).  What is left is vector issue, hence float comparisons and marks instead of keys: emit
// 28.7 us before and 11.8 now for 112 heads of 131072 tokens,
// 11.3 and 5.4 for 8 heads; cand 22.9 and 17.9, 9.8 and 7.4 (5, 6, 7 and 8 workgroups a CU: 19.1, 19.3,
// 17.9, 21.1; at 8 it spills).
constexpr int CHUNK_THREADS = 256;
constexpr int SEL_ROUNDS = SEL_CHUNK / (4 * CHUNK_THREADS);    // 4-token groups per thread
constexpr int SEL_STATE = 8;             // ints of state per pool:
// A chunk's pair of ints in the records and in the offsets.  They stand behind a candidate list of one int
// per token, so a launch with an odd number of tokens leaves them on 4-byte boundaries only.
typedef int i32x2_any __attribute__((ext_vector_type(2), aligned(4)));
// the keys [ST_LO, ST_HI] hold the threshold, which becomes ST_THR; ST_FULL: they did not
enum { ST_LO = 0, ST_HI, ST_THR, ST_FULL };
static_assert(SEL_ROUNDS >= 1 && SEL_ROUNDS <= 8, "one validity bit per token in 32 bits");

struct SelWhere {
  int seg;
  int head;        // l*H + h inside the request
  int lhead;       // launch-local head index
  int tile;        // chunk inside the head
  int pool;        // launch-local pool index
  int tok_begin, tok_end;
};
// Every wave of every chunk workgroup runs this, and it is scalar work that the waves of a CU
// queue up for: the per-segment numbers come precomputed in the table (index_chunks), so that
// one division remains.
__device__ __forceinline__ SelWhere sel_locate(const SegTable &T, int blk) {
  SelWhere q;
  int seg = 0;
  for (int i = 1; i < T.nseg; ++i) seg += blk >= T.s[i].sel_blk0;
  const Seg &s = T.s[seg];
  const int local = blk - s.sel_blk0;
  const int hh = (int)((unsigned)local / (unsigned)s.sel_bph);
  q.seg = seg;
  q.head = s.head_begin + hh;
  q.lhead = s.lhead0 + hh;
  q.tile = local - hh * s.sel_bph;
  q.pool = T.layer_scope ? s.pool0 + hh / s.H : s.pool0 + hh;
  q.tok_begin = q.tile * s.sel_chunk;
  q.tok_end = q.tok_begin + chunk_tokens(q.tok_begin, s.sel_chunk, s.n);
  return q;
}

// Position of a chunk's first token in the launch's token sequence (segments, heads and tokens in
// order): where its candidate list starts.
__device__ __forceinline__ long long chunk_token_base(const SegTable &T, const SelWhere &q) {
  const Seg &s = T.s[q.seg];
  return s.tok0 + (long long)(q.head - s.head_begin) * s.n + q.tok_begin;
}

// Room for the marks of a chunk of `tokens` tokens: where each wave's candidates begin in the list, then a pair
// of words (above the range, inside it) per thread that has tokens.  They stand at the end of the chunk's part
// of the candidate list, where the candidates leave that much room (otherwise the emit reads the scores again).
__device__ __forceinline__ int mark_ints(int tokens) {
  return CHUNK_THREADS / 64 + 2 * min(CHUNK_THREADS, (tokens + 3) >> 2);
}

// find_digit on the 4096-digit histogram of a pool in global memory (16-byte aligned), by a
// workgroup of CHUNK_THREADS.
__device__ __forceinline__ int find_digit_global(const int *__restrict__ g, int *need, int *wsum,
                                                 int *found) {
  constexpr int NB = 4096, PER = NB / CHUNK_THREADS;
  const int t0 = PER * threadIdx.x;      // digits NB-1-t0 .. NB-PER-t0, descending
  int c[PER], sum = 0;
#pragma unroll
  for (int u = 0; u < PER / 4; ++u) {
    const int4 v = *reinterpret_cast<const int4 *>(g + hist_at(NB - 4 - t0 - 4 * u));
    c[4 * u] = v.w; c[4 * u + 1] = v.z; c[4 * u + 2] = v.y; c[4 * u + 3] = v.x;
    sum += v.x + v.y + v.z + v.w;
  }
  int total;
  int before = block_exclusive_scan<CHUNK_THREADS>(sum, wsum, &total);
  const int want = *need;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (before < want && want <= before + c[q]) {
      found[0] = NB - 1 - (t0 + q);
      found[1] = want - before;
    }
    before += c[q];
  }
  __syncthreads();
  *need = found[1];
  return found[0];
}

template <int NT>
__device__ __forceinline__ void flush_hist(const int *hist, int nb, int *__restrict__ g) {
  for (int i = threadIdx.x; i < nb; i += NT) {
    const int c = hist[i];
    if (c) atomicAdd(&g[hist_at(i)], c);
  }
}

// ---- scores that came without a histogram: one by a tally, or a bracket of the threshold from a sample ----
// The threshold is the K-th largest of a pool's N scores (contiguous in memory: a pool is whole heads).
// One workgroup per pool reads a sample of m scores, half a 128-byte line at a hashed place in each of
// equal stretches, and takes the order statistics of the sample `margin` places on either side of
// rank K m / N.  margin is 4.5 standard deviations of the number of sampled scores above the threshold,
// estimated from the half lines themselves (their counts above either end of the threshold's bin), since
// neighbouring scores may be alike: half a line then says no more than one score.  A bracket that misses all
// the same costs time and not exactness: msel_thr_kernel counts what lies above and inside it, and looks at
// all scores of a pool where the threshold is in neither.  Pools of up to SAMPLE_WHOLE scores are read whole.
// Half lines, because a compute unit takes about 7 ns a line from memory however much of it is used (112 heads
// of 131072 tokens: 15 us for this kernel with 2048 groups of four, 8192 scores either way, against 11).
// Against a tally of all scores (msel_hist1_kernel), which is another pass over them, as long as the candidates', with a
// launch to clear the histogram, and 16 KB that every chunk searches.  Whole selection on MI355X (graph replay), us
// sampled / tallied, leverage scores, then averaged over 63 neighbours: 128 heads of 40003 32.3 / 36.4, 38.4 / 43.3, 128 layers of
// 8 x 8192 36.1 / 41.3, 43.3 / 48.9, 256 of 8 x 4096 40.7 / 48.6, 45.5 / 54.3.  Few long pools are tallied all the
// same: select_by_tally.
constexpr int SAMPLE_THREADS = 1024, SAMPLE_ROUNDS = 2, SAMPLE_WAVES = SAMPLE_THREADS / 64;
static_assert(SAMPLE_ROUNDS * SAMPLE_THREADS * 4 == SAMPLE_WHOLE, "a whole pool fits the registers");

// Like find_digit on 4096 digits, for two ranks at once.
__device__ __forceinline__ void find_two(const int *hist, const int (&want)[2], int *wsum, int *found, int (&digit)[2],
                                         int (&need)[2]) {
  constexpr int PER = 4096 / SAMPLE_THREADS;
  static_assert(PER == 4, "one 16-byte read");
  const int t0 = PER * (int)threadIdx.x;                 // digits 4095 - t0 .. , descending
  const int4 v = *reinterpret_cast<const int4 *>(&hist[4096 - PER - t0]);
  const int c[PER] = {v.w, v.z, v.y, v.x};
  int total;
  int before = block_exclusive_scan<SAMPLE_THREADS>(v.x + v.y + v.z + v.w, wsum, &total);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (before < want[i] && want[i] <= before + c[q]) {        // exactly one (thread, q) matches
        found[2 * i] = 4095 - (t0 + q);
        found[2 * i + 1] = want[i] - before;
      }
    before += c[q];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) { digit[i] = found[2 * i]; need[i] = found[2 * i + 1]; }
}

__global__ __launch_bounds__(SAMPLE_THREADS) void msel_sample_kernel(const SegTable T,
                                                                     const float *__restrict__ scores,
                                                                     int *__restrict__ state) {
  __shared__ __attribute__((aligned(16))) int hist[HIST1_BINS], sub[2][4096];
  __shared__ int wsum[SAMPLE_WAVES], sums[SAMPLE_WAVES][4];
  __shared__ int found[4];
  const int pool = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int seg = 0;
  for (int i = 1; i < T.nseg; ++i) seg += pool >= T.s[i].pool0;
  const Seg &s = T.s[seg];
  const int ph = pool_heads(T, s);
  const int n = ph * s.n, k = ph * s.k_keep;             // of the pool; below 2^31 - 64
  const float *sp = scores + s.score_off + (long long)(s.head_begin + (pool - s.pool0) * ph) * s.n;
  const bool whole = n <= SAMPLE_WHOLE;
  float f[SAMPLE_ROUNDS][4];
  unsigned valid = 0;
  if (!whole) {
    const int first = (int)(-(reinterpret_cast<uintptr_t>(sp) >> 2) & 15u), lines = (n - first) >> 4;
#pragma unroll
    for (int r = 0; r < SAMPLE_ROUNDS; ++r) {
      const int at = first + 16 * sample_line(r * (SAMPLE_THREADS / 4) + (tid >> 2), lines) + 4 * (tid & 3);
      const float4 v = *reinterpret_cast<const float4 *>(sp + at);
      f[r][0] = v.x; f[r][1] = v.y; f[r][2] = v.z; f[r][3] = v.w;
    }
    valid = (1u << (4 * SAMPLE_ROUNDS)) - 1u;
  } else {
#pragma unroll
    for (int r = 0; r < SAMPLE_ROUNDS; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int at = (4 * r + e) * SAMPLE_THREADS + tid;
        f[r][e] = 0.f;
        if (at < n) {
          f[r][e] = sp[at];
          valid |= 1u << (4 * r + e);
        }
      }
  }
  const int m = min(n, SAMPLE_WHOLE);
  for (int i = 4 * tid; i < HIST1_BINS; i += 4 * SAMPLE_THREADS)
    *reinterpret_cast<int4 *>(&hist[i]) = *reinterpret_cast<int4 *>(&sub[0][i]) =
        *reinterpret_cast<int4 *>(&sub[1][i]) = make_int4(0, 0, 0, 0);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < SAMPLE_ROUNDS; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (valid >> (4 * r + e) & 1) atomicAdd(&hist[score_bin(score_key(f[r][e]))], 1);
  __syncthreads();
  // descending ranks (1 .. m) of the two ends of the bracket
  int rank[2] = {k, k};
  if (!whole) {
    const double mid = (double)k * m / n;
    int need = max(1, min(m, (int)(mid + 0.5)));
    const BinKeys bk = bin_keys(find_digit<SAMPLE_THREADS>(hist, HIST1_BINS, &need, wsum, found), true);
    const uint32_t last = bk.lo | ((1u << bk.bits) - 1u);
    // per line the scores above the bin, and those from its lower end on in the upper half of the word;
    // then sums (at most 2^13) and sums of squares (at most 2^17) of both over the lines
    int ab = 0, q0 = 0, q1 = 0;
#pragma unroll
    for (int r = 0; r < SAMPLE_ROUNDS; ++r) {
      int c = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t key = score_key(f[r][e]);
        c += (key > last ? 1 : 0) + (key >= bk.lo ? 0x10000 : 0);
      }
      constexpr int XOR1 = 0xb1, XOR2 = 0x4e;
      c += __builtin_amdgcn_update_dpp(0, c, XOR1, 0xf, 0xf, false);
      c += __builtin_amdgcn_update_dpp(0, c, XOR2, 0xf, 0xf, false);
      if ((lane & 3) == 0) {
        ab += c;
        q0 += (c & 0xffff) * (c & 0xffff);
        q1 += (c >> 16) * (c >> 16);
      }
    }
    ab = wave_inclusive_scan(ab);
    q0 = wave_inclusive_scan(q0);
    q1 = wave_inclusive_scan(q1);
    if (lane == 63) { sums[wave][0] = ab; sums[wave][1] = q0; sums[wave][2] = q1; }
    __syncthreads();
    ab = q0 = q1 = 0;
#pragma unroll
    for (int w = 0; w < SAMPLE_WAVES; ++w) { ab += sums[w][0]; q0 += sums[w][1]; q1 += sums[w][2]; }
    constexpr float per_line = 1.f / (float)SAMPLE_LINES;
    const float s0 = (float)(ab & 0xffff), s1 = (float)(ab >> 16);
    const float var = fmaxf((float)q0 - s0 * s0 * per_line, (float)q1 - s1 * s1 * per_line);
    const int margin = (int)(4.5f * sqrtf(fmaxf(var, 0.f))) + 3;
    rank[0] = (int)mid - margin;
    rank[1] = (int)mid + 1 + margin;
  }
  // Either end: its bin, then the 12 bits below the bin's.  No end above rank 1 or below rank m.
  const bool has_hi = rank[0] >= 1, has_lo = rank[1] <= m;
  const int want[2] = {max(1, rank[0]), min(m, rank[1])};
  int bin[2], need[2], dig[2];           // dig: below the bin's
  find_two(hist, want, wsum, found, bin, need);
  const BinKeys bh = bin_keys(bin[0], true), bl = bin_keys(bin[1], true);
#pragma unroll
  for (int r = 0; r < SAMPLE_ROUNDS; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (valid >> (4 * r + e) & 1) {
        const uint32_t key = score_key(f[r][e]);
        if (key >> bh.bits == bh.lo >> bh.bits) atomicAdd(&sub[0][key >> (bh.bits - 12) & 0xfffu], 1);
        if (key >> bl.bits == bl.lo >> bl.bits) atomicAdd(&sub[1][key >> (bl.bits - 12) & 0xfffu], 1);
      }
  __syncthreads();
  {
    // both digits by one scan: half of the threads have eight digits each of sub[0], the others of sub[1]
    const int half = wave / (SAMPLE_WAVES / 2), t0 = 8 * (tid & (SAMPLE_THREADS / 2 - 1));
    const int4 a = *reinterpret_cast<const int4 *>(&sub[half][4092 - t0]);
    const int4 b = *reinterpret_cast<const int4 *>(&sub[half][4088 - t0]);
    const int c[8] = {a.w, a.z, a.y, a.x, b.w, b.z, b.y, b.x};
    int total;
    int before = block_exclusive_scan<SAMPLE_THREADS>(a.x + a.y + a.z + a.w + b.x + b.y + b.z + b.w, wsum, &total);
    if (half)
#pragma unroll
      for (int w = 0; w < SAMPLE_WAVES / 2; ++w) before -= wsum[w];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (before < need[half] && need[half] <= before + c[q]) found[half] = 4095 - (t0 + q);
      before += c[q];
    }
    __syncthreads();
    dig[0] = found[0];
    dig[1] = found[1];
  }
  if (tid == 0) {
    int *st = state + pool * SEL_STATE;
    const int rh = bh.bits - 12, rl = bl.bits - 12;
    st[ST_LO] = has_lo ? (int)(bl.lo | (uint32_t)dig[1] << rl) : 0;
    st[ST_HI] = has_hi ? (int)(bh.lo | (uint32_t)dig[0] << rh | ((1u << rh) - 1u)) : (int)0xff800000u;      // +inf
  }
}

// First digit by a tally of all scores, into the pool's histogram (zero on entry).
__global__ __launch_bounds__(CHUNK_THREADS, 8) void msel_hist1_kernel(const SegTable T,
                                                                    const float *__restrict__ scores,
                                                                    int *__restrict__ hist1) {
  __shared__ int hist[HIST1_BINS];
  const SelWhere q = sel_locate(T, blockIdx.x);
  const Seg &s = T.s[q.seg];
  const float *sp = scores + s.score_off + (long long)q.head * s.n;
  float f[SEL_ROUNDS][4];
  load_scores<CHUNK_THREADS, SEL_ROUNDS>(sp, q.tok_begin, q.tok_end, 0, f);
  for (int i = threadIdx.x; i < HIST1_BINS; i += CHUNK_THREADS) hist[i] = 0;
  __syncthreads();
  const unsigned valid = place_scores<CHUNK_THREADS, SEL_ROUNDS>(q.tok_begin, q.tok_end, 0, f);
#pragma unroll
  for (int r = 0; r < SEL_ROUNDS; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (valid >> (4 * r + e) & 1) atomicAdd(&hist[score_bin(score_key(f[r][e]))], 1);
  __syncthreads();
  flush_hist<CHUNK_THREADS>(hist, HIST1_BINS, hist1 + (size_t)q.pool * HIST1_BINS);
}

// (a small kernel, not a memset: callers may capture the call into a graph)
__global__ __launch_bounds__(256) void fill_zero_kernel(int *__restrict__ z, long long count) {
  zero_slice(z, count);
}

// Where a pool's range of candidates comes from: the histogram that came with the scores (top 12 key bits), one made by
// msel_hist1_kernel (score_bin), or msel_sample_kernel.
enum Range { CAME, TALLIED, SAMPLED_RANGE };

// Candidates of a chunk: counts the keys above the range that holds the threshold and lists the
// keys inside it, less its lowest (cand, at the chunk's position in the launch's token sequence, so a list can
// never outgrow its room), and marks both kinds for the emit.  rec[chunk] = (keys above, candidates listed).
template <Range RANGE>
__global__ __launch_bounds__(CHUNK_THREADS, 7) void msel_cand_kernel(const SegTable T,
                                                                  const float *__restrict__ scores,
                                                                  const int *__restrict__ hist1,
                                                                  uint32_t *__restrict__ cand,
                                                                  int *__restrict__ rec,
                                                                  int *__restrict__ state) {
  __shared__ int wsum[CHUNK_THREADS / 64];
  __shared__ int found[2];
  __shared__ int above_s, ncand_s;
  constexpr bool SAMPLED = RANGE == SAMPLED_RANGE;
  constexpr int CAND_STAGE = 768;        // of at most 2048 a wave
  __shared__ __attribute__((aligned(16))) uint32_t stage[CHUNK_THREADS / 64][CAND_STAGE];
  const SelWhere q = sel_locate(T, blockIdx.x);
  const Seg &s = T.s[q.seg];
  const float *sp = scores + s.score_off + (long long)q.head * s.n;
  float f[SEL_ROUNDS][4];
  load_scores<CHUNK_THREADS, SEL_ROUNDS>(sp, q.tok_begin, q.tok_end, 0, f);             // in flight while the digit is found
  if (threadIdx.x == 0) { above_s = 0; ncand_s = 0; }
  uint32_t lo, hi;
  if constexpr (SAMPLED) {
    __syncthreads();                     // the counters are zero
    lo = (uint32_t)state[q.pool * SEL_STATE + ST_LO];
    hi = (uint32_t)state[q.pool * SEL_STATE + ST_HI];
  } else {
    const int ph = pool_heads(T, s);
    int need = ph * s.k_keep;
    const BinKeys bk = bin_keys(find_digit_global(hist1 + (size_t)q.pool * HIST1_BINS, &need, wsum, found), RANGE == TALLIED);
    lo = bk.lo;
    hi = bk.lo | ((1u << bk.bits) - 1u);
    if (q.tile == 0 && q.lhead % ph == 0 && threadIdx.x == 0) {   // the pool's first chunk
      state[q.pool * SEL_STATE + ST_LO] = (int)lo;
      state[q.pool * SEL_STATE + ST_HI] = (int)hi;
    }
  }
  unsigned above, in;
  const unsigned valid = place_scores<CHUNK_THREADS, SEL_ROUNDS>(q.tok_begin, q.tok_end, 0, f);
  classify<SEL_ROUNDS>(f, valid, lo, hi, above, in);
  uint32_t *list = cand + chunk_token_base(T, q);
  const int lane = threadIdx.x & 63;
  // A wave's candidates stand in thread order, a thread's in consecutive slots, so that the emit finds them
  // again by the same sums of the marks; the order in which waves claim their share of the list does not
  // matter.  Counts are packed with those above (at most 2048 each).
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int both = __popc(in) | (__popc(above) << 16);
  const int inc = wave_inclusive_scan(both);
  const int mine = __builtin_amdgcn_readlane(inc, 63) & 0xffff;          // of the wave
  int base = 0;
  if (lane == 63) {
    if (mine) base = atomicAdd(&ncand_s, mine);
    if (inc >> 16) atomicAdd(&above_s, inc >> 16);
  }
  base = __builtin_amdgcn_readlane(base, 63);
  auto put = [&](uint32_t *to) {
    to += (inc - both) & 0xffff;
#pragma unroll
    for (int r = 0; r < SEL_ROUNDS; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (in >> (4 * r + e) & 1) *to++ = __float_as_uint(f[r][e]);
  };
  if (SAMPLED && mine <= CAND_STAGE) {   // they leave as one run
    typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    put(stage[wave]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int i = 4 * lane; i < mine; i += 256) {
      const uint4 v = *reinterpret_cast<const uint4 *>(&stage[wave][i]);
      uint32_t *to = list + base + i;
      if (i + 3 < mine) {
        *reinterpret_cast<u32x4_any *>(to) = u32x4_any{v.x, v.y, v.z, v.w};
      } else {
        to[0] = v.x;
        if (i + 1 < mine) to[1] = v.y;
        if (i + 2 < mine) to[2] = v.z;
      }
    }
  } else {
    put(list + base);
  }
  __syncthreads();
  const int tokens = q.tok_end - q.tok_begin, marks = mark_ints(tokens);
  const int ncand = ncand_s;
  if (ncand <= tokens - marks) {
    constexpr int NW = CHUNK_THREADS / 64;
    uint32_t *mark = list + (tokens - marks);
    if (lane == 0) mark[wave] = (uint32_t)base;
    if (NW + 2 * (int)threadIdx.x < marks) {
      mark[NW + 2 * threadIdx.x] = above;
      mark[NW + 2 * threadIdx.x + 1] = in;
    }
  }
  if (threadIdx.x == 0) {
    rec[2 * blockIdx.x] = above_s;
    rec[2 * blockIdx.x + 1] = ncand;
  }
}

// Visits the `cnt` values of a candidate list, f(value) for each: a wave's lanes take 4
// consecutive values each with one 16-byte load (at any 4-byte address), four loads in flight.
template <class F>
__device__ __forceinline__ void for_each_cand(const uint32_t *__restrict__ l, int cnt, int lane, F &&f) {
  typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int DEPTH = 4;
  for (int i = 4 * lane; i < cnt; i += 256 * DEPTH) {
    uint32_t v[DEPTH][4];
    int have[DEPTH];
#pragma unroll
    for (int h = 0; h < DEPTH; ++h) {
      const int j = i + 256 * h;
      have[h] = min(4, cnt - j);
      if (have[h] == 4) {
        const u32x4_any t = *reinterpret_cast<const u32x4_any *>(l + j);
        v[h][0] = t.x; v[h][1] = t.y; v[h][2] = t.z; v[h][3] = t.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[h][e] = e < have[h] ? l[j + e] : 0u;
      }
    }
#pragma unroll
    for (int h = 0; h < DEPTH; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < have[h]) f(v[h][e]);
  }
}

// One workgroup per pool: the threshold key from the pool's candidates, then for every chunk of
// the pool (in head, token order) the position of its first retained token in the pool's
// output and how many threshold ties it may keep; the per-head counts.  The candidates' rank comes from the
// chunks' counts; where it says that the threshold is none of them (a sampled bracket that missed), the keys of all scores
// of the pool take their place (ST_FULL).  One workgroup goes over them then: whole selection on MI355X, us where no
// bracket misses / where all do, 32 heads of 40003 28.1 / 55.5, 17 layers of 8 x 131072 66.9 / 536 (with the scores
// themselves, one 4-byte load in flight a thread, in every pass, 1564; the candidates' loops serve both, and a key made of
// a score in them, where it is not needed, cost 5 to 20 % of a selection of long pools).
// Two passes over the candidates: (1) histogram of the upper 12 bits in which they differ -> second
// digit d2; (2) per chunk the count above d2, a histogram of the low bits (5, 8 or 11) of those inside d2,
// and those few themselves as (chunk, low bits) in a short LDS list, from which, once the last digit is
// known, every chunk's counts above and at the threshold follow.  If the list overflows (heavily
// tied scores) or the pool has more than THR_BLOCK chunks, a third pass counts instead.
// The chunks' records are fetched into LDS in blocks of THR_BLOCK (a load per chunk in turn
// would string their latencies together); inside a block the waves take the chunks in turn.  The passes
// wait for loads, not for arithmetic: with 4 waves a wave goes through several chunks of a pool one
// after the other, so 16 waves take a pool while every pool has a compute unit to itself.  With more pools
// the 16 waves only wait for each other.  Whole selection on given scores on MI355X, us with 16 / 4 waves: heads
// of 40003 tokens, 128 of them 49.1 / 52.0, 256 66 / 67, 384 92 / 88, 512 105 / 100, 768 144 / 133, 1024
// 184 / 166; of 131072, 256 131 / 138, 384 185 / 184, 640 296 / 288; layers of 8 x 8192, 256 86.6 / 88.8,
// 384 117 / 113; of 8 x 32768, 256 224 / 240, 384 345 / 349.  Behind the score kernel, selection
// alone: 256 heads of 66000 55 / 61, 384 76 / 74, 640 of 100000 130 / 121, 1536 of 40003 150 / 122.
// SAMPLED: the range of the candidates' values is any, and the threshold may be none of them.
constexpr int THR_BLOCK = 512, THR_SHORT = 2048, THR_WIDE_POOLS = 256;
template <int THR_THREADS, bool SAMPLED>
__global__ __launch_bounds__(THR_THREADS) void msel_thr_kernel(const SegTable T,
                                                               const float *__restrict__ scores,
                                                               uint32_t *__restrict__ cand,
                                                               const int *__restrict__ rec,
                                                               int *__restrict__ coff,
                                                               int *__restrict__ state,
                                                               int32_t *__restrict__ kept_cnt) {
  constexpr int NW = THR_THREADS / 64;
  __shared__ int hist[4096];
  __shared__ int wsum[NW];
  __shared__ int found[2];
  __shared__ int above_c[THR_BLOCK], cnt_c[THR_BLOCK], gt_c[THR_BLOCK], eq_c[THR_BLOCK];
  __shared__ uint32_t short_l[THR_SHORT];
  __shared__ int nshort;
  // locate the pool: segment, first head, first chunk, first token
  const int pool = blockIdx.x;
  int seg = 0;
  for (int i = 1; i < T.nseg; ++i) seg += pool >= T.s[i].pool0;
  const Seg &s = T.s[seg];
  const int ph = pool_heads(T, s);
  const int bph = s.sel_bph, csize = s.sel_chunk;
  const int head0 = s.head_begin + (pool - s.pool0) * ph;
  const int chunk0 = s.sel_blk0 + (pool - s.pool0) * ph * bph;
  const long long tok0 = s.tok0 + (long long)(pool - s.pool0) * ph * s.n;
  const int nchunks = ph * bph;
  const bool single = nchunks <= THR_BLOCK;      // all records fit LDS at once
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t lo = (uint32_t)state[pool * SEL_STATE + ST_LO];
  const uint32_t span = (uint32_t)state[pool * SEL_STATE + ST_HI] - lo;
  bool full = false;                             // the keys of all scores are the candidates' values
  auto tokens_of = [&](int c) { return chunk_tokens(c % bph * csize, csize, s.n); };
  // where chunk c of the pool begins among the pool's tokens; its candidate list
  auto token_of = [&](int c) { return (long long)(c / bph) * s.n + (long long)(c % bph) * csize; };
  auto list_of = [&](int c) { return cand + tok0 + token_of(c); };
  // records of the chunks [cb, cb + THR_BLOCK) into LDS
  auto fetch = [&](int cb) {
    __syncthreads();
    for (int u = tid; u < THR_BLOCK && cb + u < nchunks; u += THR_THREADS) {
      i32x2_any r = *reinterpret_cast<const i32x2_any *>(rec + 2 * (chunk0 + cb + u));
      if (SAMPLED && full) r = i32x2_any{0, tokens_of(cb + u)};
      above_c[u] = r.x;
      cnt_c[u] = r.y;
    }
    __syncthreads();
  };

  // the candidates of rank 1 .. inside are inside
  int need = ph * s.k_keep;
  for (int i = tid; i < 4096; i += THR_THREADS) hist[i] = 0;
  if (tid == 0) nshort = 0;
  {
    int above = 0, inside = 0;
    for (int cb = 0; cb < nchunks; cb += THR_BLOCK) {
      fetch(cb);
      for (int u = tid; u < THR_BLOCK && cb + u < nchunks; u += THR_THREADS) {
        above += above_c[u];
        inside += cnt_c[u];
      }
    }
    int all;
    block_exclusive_scan<THR_THREADS>(above, wsum, &all);
    need -= all;
    if constexpr (SAMPLED) {
      block_exclusive_scan<THR_THREADS>(inside, wsum, &all);
      full = need < 1 || need > all;
    }
  }
  int bits = span ? 32 - __clz((int)span) : 0;           // of a candidate's value
  if (SAMPLED && full) {
    lo = 0;
    bits = 32;
    need = ph * s.k_keep;
    // the lists have room for every token, and the emit does not look at the marks behind them
    const float *sp = scores + s.score_off + (long long)head0 * s.n;
    for (int c = wave; c < nchunks; c += NW) {
      const float *from = sp + token_of(c);
      uint32_t *to = list_of(c);
      const int tokens = tokens_of(c);
#pragma unroll 8
      for (int i = lane; i < tokens; i += 64) to[i] = score_key(from[i]);
    }
    if (single) fetch(0);
    __syncthreads();                                     // the lists are complete
  }
  uint32_t base = 0;                                     // the threshold's value lies in [base, base + 2^bits)
  // the 12 bits from `rest` on of the values in [base, base + 2^(rest + 12))
  auto tally = [&](int rest) {
    for (int cb = 0; cb < nchunks; cb += THR_BLOCK) {
      if (!single) fetch(cb);
      for (int u = wave; u < THR_BLOCK && cb + u < nchunks; u += NW)
        for_each_cand(list_of(cb + u), cnt_c[u], lane, [&](uint32_t v) {
          const uint32_t d = (v - base) >> rest;
          if (!SAMPLED || d < 4096) atomicAdd(&hist[d], 1);
        });
    }
  };
  if (SAMPLED && bits > 23) {                            // one pass more
    tally(bits - 12);
    __syncthreads();
    bits -= 12;
    base = (uint32_t)find_digit<THR_THREADS>(hist, 4096, &need, wsum, found) << bits;
    __syncthreads();
    for (int i = tid; i < 4096; i += THR_THREADS) hist[i] = 0;
    __syncthreads();
  }
  const int rest = bits > 12 ? bits - 12 : 0;
  const uint32_t low = (1u << rest) - 1u;
  // pass 1: the upper 12 bits of every candidate
  tally(rest);
  __syncthreads();
  const uint32_t d2 = (uint32_t)find_digit<THR_THREADS>(hist, 4096, &need, wsum, found);
  base += d2 << rest;
  const uint32_t top = base | low;
  // pass 2: the low bits of the candidates that share the second digit; per chunk those above it
  // (none: d2 is the whole value, and the third pass counts)
  const bool third = SAMPLED && rest == 0;
  if (!third) {
    for (int i = tid; i <= (int)low; i += THR_THREADS) hist[i] = 0;
    for (int cb = 0; cb < nchunks; cb += THR_BLOCK) {
      if (!single) fetch(cb); else __syncthreads();
      for (int u = wave; u < THR_BLOCK && cb + u < nchunks; u += NW) {
        int gt = 0;
        for_each_cand(list_of(cb + u), cnt_c[u], lane, [&](uint32_t v) {
          gt += v > top;
          if (v - base <= low) {
            atomicAdd(&hist[v - base], 1);
            if (single) {
              const int at = atomicAdd(&nshort, 1);
              if (at < THR_SHORT) short_l[at] = ((uint32_t)u << 11) | (v - base);
            }
          }
        });
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) gt += __shfl_xor(gt, d);
        if (lane == 0) { gt_c[u] = gt; eq_c[u] = 0; }
      }
    }
  }
  __syncthreads();
  const uint32_t d3 = third ? 0u : (uint32_t)find_digit<THR_THREADS>(hist, 1 << rest, &need, wsum, found);
  const int tie_keep = need;             // keys equal to the threshold that are retained
  const bool all_ties = hist[third ? d2 : d3] == need;
  const uint32_t at_v = base + d3;       // the threshold's value
  if (tid == 0) {
    state[pool * SEL_STATE + ST_THR] = (int)(lo + at_v);
    state[pool * SEL_STATE + ST_FULL] = full;
  }
  const bool from_short = single && !third && nshort <= THR_SHORT;
  if (from_short) {                      // the chunks' counts at the last digit, from the short list
    for (int i = tid; i < nshort; i += THR_THREADS) {
      const uint32_t e = short_l[i];
      const uint32_t l = e & 0x7ffu;
      if (l > d3) atomicAdd(&gt_c[e >> 11], 1);
      else if (l == d3) atomicAdd(&eq_c[e >> 11], 1);
    }
  }

  // every chunk's output position and tie allowance: prefix sums over the chunks in order, a block at a
  // time; a head's count is the distance between the positions at its ends
  int pos = 0, eq_before = 0, head_pos = 0;      // head_pos: where the head that a block begins in starts
  for (int cb = 0; cb < nchunks; cb += THR_BLOCK) {
    if (!from_short) {                   // pass 3: count against the full threshold
      if (!single) fetch(cb); else __syncthreads();
      for (int u = wave; u < THR_BLOCK && cb + u < nchunks; u += NW) {
        int gt = 0, eq = 0;
        for_each_cand(list_of(cb + u), cnt_c[u], lane, [&](uint32_t v) {
          gt += v > at_v;
          eq += v == at_v;
        });
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
          gt += __shfl_xor(gt, d);
          eq += __shfl_xor(eq, d);
        }
        if (lane == 0) { gt_c[u] = gt; eq_c[u] = eq; }
      }
    }
    __syncthreads();
    // THR_THREADS chunks at a time
    for (int u0 = 0; u0 < THR_BLOCK && cb + u0 < nchunks; u0 += THR_THREADS) {
      const int u = u0 + tid, cc = cb + u;
      const bool mine = u < THR_BLOCK && cc < nchunks;
      const int eq = mine ? eq_c[u] : 0;
      int eq_all = 0, kept_all, allow = eq;
      if (!all_ties) {                   // uniform
        const int eq0 = eq_before + block_exclusive_scan<THR_THREADS>(eq, wsum, &eq_all);
        allow = max(0, min(eq, tie_keep - eq0));
      }
      const int kept = mine ? above_c[u] + gt_c[u] + allow : 0;
      const int at = pos + block_exclusive_scan<THR_THREADS>(kept, wsum, &kept_all);
      if (mine) {
        *reinterpret_cast<i32x2_any *>(coff + 2 * (chunk0 + cc)) = i32x2_any{at, allow};
        eq_c[u] = at;                    // this chunk's count has been read
        gt_c[u] = at + kept;
      }
      pos += kept_all;
      eq_before += eq_all;
    }
    __syncthreads();
    for (int u = tid; u < THR_BLOCK && cb + u < nchunks; u += THR_THREADS) {
      const int cc = cb + u, hc = cc - cc % bph;        // first chunk of the head
      if (cc - hc == bph - 1) {                         // its last
        const int start = hc >= cb ? eq_c[hc - cb] : head_pos;
        kept_cnt[s.ghead0 + head0 + cc / bph] = T.layer_scope ? gt_c[u] - start : s.k_keep;
      }
    }
    const int open = (cb + THR_BLOCK) / bph * bph;      // the head that the next block begins in
    if (open >= cb + THR_BLOCK) head_pos = pos;
    else if (open >= cb && open < nchunks) head_pos = eq_c[open - cb];
  }
}

// Ordered emit of one chunk.  The marks of the candidate pass say which tokens lie above the threshold's
// range and which inside it; the latter's values stand in the list in the order of the marks, and the scores
// are only read again where the candidates left no room for marks, or the range missed the threshold.
//  (It used to read the candidates' scores, one line of memory for each, or whole rows: 112 heads of 131072
// tokens 11.3 us, 9.1 now.)  Four tokens per thread and round come in:
// a byte per such group passes through LDS, so that a thread then holds 32 consecutive tokens and one scan
// over the workgroup gives every position.  Counts are packed as (above | equal << 16), at most 8192 each.
__global__ __launch_bounds__(CHUNK_THREADS, 8) void msel_emit_kernel(const SegTable T,
                                                                   const float *__restrict__ scores,
                                                                   const uint32_t *__restrict__ cand,
                                                                   const int *__restrict__ rec,
                                                                   const int *__restrict__ coff,
                                                                   const int *__restrict__ state,
                                                                   int32_t *__restrict__ kept_idx) {
  constexpr int NW = CHUNK_THREADS / 64;
  __shared__ int wtot[NW];
  __shared__ __attribute__((aligned(8))) unsigned char quad[SEL_ROUNDS * CHUNK_THREADS];
  __shared__ uint16_t stage[SEL_CHUNK];
  const SelWhere q = sel_locate(T, blockIdx.x);
  const Seg &s = T.s[q.seg];
  const float *sp = scores + s.score_off + (long long)q.head * s.n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tokens = q.tok_end - q.tok_begin, marks = mark_ints(tokens);
  const uint32_t *list = cand + chunk_token_base(T, q), *mark = list + (tokens - marks);
  unsigned gt = 0, in = 0, eq = 0;
  int off = 0;                           // of the wave's candidates in the list
  if (marks <= tokens) {
    off = (int)mark[wave];
    if (NW + 2 * tid < marks) { gt = mark[NW + 2 * tid]; in = mark[NW + 2 * tid + 1]; }
  }
  const int ncand = rec[2 * blockIdx.x + 1];
  const int ph = pool_heads(T, s);
  const int limit = ph * s.k_keep;                       // rows of the pool's output
  int32_t *out = kept_idx + (s.kept_off + (long long)(q.head / ph) * limit);
  const uint32_t thr = (uint32_t)state[q.pool * SEL_STATE + ST_THR];
  const bool no_marks = ncand > tokens - marks || state[q.pool * SEL_STATE + ST_FULL] != 0;
  const i32x2_any pa = *reinterpret_cast<const i32x2_any *>(coff + 2 * blockIdx.x);
  const int pos0 = pa.x, allow = pa.y;
  // key > thr and key == thr as float comparisons; a threshold that is NaN (key 0) equals NaN only and
  // every number lies above it
  const float fthr = key_score(thr);
  auto is_gt = [&](float x) { return thr ? x > fthr : x == x; };
  auto is_eq = [&](float x) { return thr ? x == fthr : x != x; };
  if (no_marks) {                                        // uniform
    gt = 0;
    float f[SEL_ROUNDS][4];
    load_scores<CHUNK_THREADS, SEL_ROUNDS>(sp, q.tok_begin, q.tok_end, 0, f);
    const unsigned valid = place_scores<CHUNK_THREADS, SEL_ROUNDS>(q.tok_begin, q.tok_end, 0, f);
#pragma unroll
    for (int r = 0; r < SEL_ROUNDS; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned bit = valid & (1u << (4 * r + e));
        gt |= is_gt(f[r][e]) ? bit : 0u;
        eq |= is_eq(f[r][e]) ? bit : 0u;
      }
  } else {
    off += wave_inclusive_scan(__popc(in)) - __popc(in);
    const uint32_t thr_v = thr - (uint32_t)state[q.pool * SEL_STATE + ST_LO];
    constexpr int FLIGHT = 4;
    while (__any(in != 0)) {
      uint32_t v[FLIGHT];
      unsigned bit[FLIGHT];
#pragma unroll
      for (int j = 0; j < FLIGHT; ++j) {
        bit[j] = in & (0u - in);
        in ^= bit[j];
        v[j] = 0;
        if (bit[j]) v[j] = list[off++];
      }
#pragma unroll
      for (int j = 0; j < FLIGHT; ++j) {
        gt |= v[j] > thr_v ? bit[j] : 0u;
        eq |= v[j] == thr_v ? bit[j] : 0u;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < SEL_ROUNDS; ++r)
    quad[r * CHUNK_THREADS + tid] = (unsigned char)((gt >> (4 * r) & 0xfu) | (eq >> (4 * r) & 0xfu) << 4);
  __syncthreads();
  // this thread's tokens are now tok_begin + 32 * tid ..: low and high nibbles of 8 bytes
  const uint2 by = *reinterpret_cast<const uint2 *>(&quad[8 * tid]);
  auto packed = [](unsigned lo, unsigned hi) {           // the low nibbles of 8 bytes, 4 bits each
    auto four = [](unsigned x) {
      x &= 0x0f0f0f0fu;
      x = (x | x >> 4) & 0x00ff00ffu;
      return (x | x >> 8) & 0xffffu;
    };
    return four(lo) | four(hi) << 16;
  };
  emit_ordered<CHUNK_THREADS>(packed(by.x, by.y), packed(by.x >> 4, by.y >> 4), allow, q.tok_begin, 32 * tid,
                              limit - pos0, wtot, stage, out + pos0);
}

// ---- blend: s = z(a) + lambda z(o) (paper Eq. "scoring"), population standard deviation ------
// The sums that the two standardisations need are gathered on the way, in the score kernel's
// epilogue: per score workgroup the fp64 (sum, sum of squares) of its scores o and of the
// attention scores a of the same tokens, a shifted by the head's first element so that a nearly
// constant vector does not cancel (ostat, four doubles per workgroup).  blend_apply_kernel adds a
// head's pairs up in index order (every chunk of the head gets the same mean and deviation, bit
// for bit), rewrites the scores in place and tallies the first selection histogram.
// Mean and reciprocal deviation of a head's scores o and attention scores a from `count`
// quadruples (sum and sum of squares of o, then of a less `shift`), added in index order.
struct Moments { double mo, io, ma, ia; };
__device__ __forceinline__ Moments moments(const double *__restrict__ quads, int count, int n,
                                           double shift, double (*wd)[4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < count; i += CHUNK_THREADS) {
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] += quads[4 * i + c];
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] += __shfl_xor(v[c], d);
  }
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) wd[wave][c] = v[c];
  }
  __syncthreads();
  double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < CHUNK_THREADS / 64; ++i) {
#pragma unroll
    for (int c = 0; c < 4; ++c) t[c] += wd[i][c];
  }
  Moments m;
  // a constant vector (deviation 0) contributes nothing
  const double mo = t[0] / n, ma = t[2] / n;
  double vo = t[1] / n - mo * mo, va = t[3] / n - ma * ma;
  m.mo = mo;
  m.io = vo > 0.0 ? 1.0 / sqrt(vo) : 0.0;
  m.ma = shift + ma;
  m.ia = va > 0.0 ? 1.0 / sqrt(va) : 0.0;
  return m;
}

// Where a segment's pairs start in ostat (its first score workgroup) and how many a head has.
struct OstatIndex {
  long long first[MAX_SEG];
  int per_head[MAX_SEG];
};
// A workgroup takes a chunk in parts of PART rounds: the fp64 arithmetic of a whole chunk at once would take
// so many registers that only three workgroups fit a CU.  HALF: one part each, where whole chunks are too
// few to fill the chip; its scores are requested before the head's sums are added up, which hides a load
// latency.  Stage on MI355X, us whole / halved, heads of 16383 tokens: 64 chunks 15.7 / 10.8, 256
// 17.0 / 12.2, 512 20.1 / 16.3, 640 22.2 / 18.5, 768 23.3 / 23.1, 1024 27.3 / 27.6; heads of 8292, where the
// second half of every chunk is nearly empty: 64 12.7 / 10.8, 256 13.2 / 11.9, 512 15.0 / 14.9, 640 16.5 / 16.6,
// 768 17.6 / 21.1.  Hence halves up to 512 chunks.
template <bool HALF>
__global__ __launch_bounds__(CHUNK_THREADS) void blend_apply_kernel(
    const SegTable T, const OstatIndex X, float lambda, float *__restrict__ scores,
    const double *__restrict__ ostat, int *__restrict__ hist1) {
  __shared__ double wd[CHUNK_THREADS / 64][4];
  __shared__ int hist[HIST1_BINS];
  constexpr int PART = SEL_ROUNDS / 2;
  const SelWhere q = sel_locate(T, HALF ? blockIdx.x >> 1 : blockIdx.x);
  const int r_first = HALF ? (int)(blockIdx.x & 1) * PART : 0;
  const Seg &s = T.s[q.seg];
  if (s.attn == nullptr || 4 * r_first * CHUNK_THREADS >= q.tok_end - q.tok_begin) return;     // uniform
  const int n = s.n, tid = threadIdx.x;
  float *o = scores + s.score_off + (long long)q.head * n;
  const float *a = s.attn + (long long)q.head * n;
  const float a0 = a[0];
  float fa[PART][4], fo[PART][4];
  if (HALF) {
    load_scores<CHUNK_THREADS, PART>(a, q.tok_begin, q.tok_end, r_first, fa);
    load_scores<CHUNK_THREADS, PART>(o, q.tok_begin, q.tok_end, r_first, fo);
  }
  // where the head's sums start: its first score workgroup
  const int obph = X.per_head[q.seg];
  const long long ob = X.first[q.seg] + (long long)(q.head - s.head_begin) * obph;
  if (hist1 != nullptr)
    for (int i = tid; i < HIST1_BINS; i += CHUNK_THREADS) hist[i] = 0;
  const Moments M = moments(ostat + 4 * ob, obph, n, (double)a0, wd);     // has a barrier
  const double mo = M.mo, ma = M.ma, ia = M.ia, io = M.io * (double)lambda;
  typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll 1
  for (int r0 = r_first; r0 < (HALF ? r_first + PART : SEL_ROUNDS); r0 += PART) {
    if (!HALF) {
      if (4 * r0 * CHUNK_THREADS >= q.tok_end - q.tok_begin) break;       // uniform
      load_scores<CHUNK_THREADS, PART>(a, q.tok_begin, q.tok_end, r0, fa);
      load_scores<CHUNK_THREADS, PART>(o, q.tok_begin, q.tok_end, r0, fo);
    }
    place_scores<CHUNK_THREADS, PART>(q.tok_begin, q.tok_end, r0, fa);
    const unsigned valid = place_scores<CHUNK_THREADS, PART>(q.tok_begin, q.tok_end, r0, fo);
#pragma unroll
    for (int r = 0; r < PART; ++r) {
      const unsigned m = (valid >> (4 * r)) & 0xfu;
      if (m == 0) continue;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = (float)(((double)fa[r][e] - ma) * ia + ((double)fo[r][e] - mo) * io);
        if (hist1 != nullptr && (m >> e & 1)) atomicAdd(&hist[score_key(v[e]) >> 20], 1);
      }
      const int i0 = q.tok_begin + 4 * ((r0 + r) * CHUNK_THREADS + tid);
      if (m == 0xfu) {
        f32x4_any t;
        t.x = v[0]; t.y = v[1]; t.z = v[2]; t.w = v[3];
        *reinterpret_cast<f32x4_any *>(o + i0) = t;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (m >> e & 1) o[i0 + e] = v[e];
      }
    }
  }
  if (hist1 != nullptr) {
    __syncthreads();
    flush_hist<CHUNK_THREADS>(hist, HIST1_BINS, hist1 + (size_t)q.pool * HIST1_BINS);
  }
}

bool select_needs_pools(const SegTable &T) {
  if (T.layer_scope) return true;
  for (int i = 0; i < T.nseg; ++i)
    if (T.s[i].n > WHOLE_HEAD) return true;
  return false;
}

SelectScratch select_scratch(const SegTable &T) {
  SelectScratch z;
  long long pools = 0, rows = 0;
  for (int i = 0; i < T.nseg; ++i) {
    pools += T.s[i].head_count / pool_heads(T, T.s[i]);
    rows += (long long)T.s[i].n * T.s[i].head_count;
  }
  z.pools = (int)pools;
  z.chunks = total_blocks(T, SEL_CHUNK, 4, false);
  z.cand_ints = rows;
  z.rec_ints = z.chunks * 2;
  z.coff_ints = z.chunks * 2;
  z.state_ints = pools * SEL_STATE;
  return z;
}

long long select_chunks(const SegTable &T) { return total_blocks(T, SEL_CHUNK, 4, false); }

// Whether the first digit of a launch's pools comes from a tally of all scores and not from a sample: few pools, one of
// them long.  A tally is a pass over the scores and a launch more; a sample's bracket widens with the pool and with
// how alike neighbouring scores are, and one workgroup looks at what is inside it (and at all scores where it misses).
// Whole selection on MI355X (graph replay), us sampled / tallied, for leverage scores, the same averaged over 7 and over
// 63 neighbours: layers of 8 x 131072, 2 of them 49.0 / 47.5, 51.0 / 48.1, 70.2 / 53.7, 8 56.4 / 57.9, 60.2 / 59.0, 79.8 /
// 66.7, 12 60.9 / 66.9, 64.2 / 67.9, 84.3 / 78.6; of 8 x 65536, 4 37.1 / 36.2, 40.0 / 37.2, 49.3 / 46.5, 12 41.1 /
// 42.2, 43.9 / 43.3, 54.6 / 55.6; of 8 x 32768, 4 30.9 / 29.8, 32.1 / 30.2, 38.1 / 33.4, 12 31.8 / 32.1, 33.3 / 32.5,
// 39.7 / 39.4; of 32 x 131072, 4 135 / 143, 142 / 143, 211 / 164, 8 149 / 169, 158 / 169, 232 / 198; heads of 131072, 8
// of them 27.7 / 26.6, 28.4 / 27.3, 33.1 / 30.7, 32 30.0 / 30.3, 31.9 / 31.2, 37.1 / 35.9, 64 36.3 / 39.5, 38.2 / 40.8,
// 44.0 / 47.4.  Shorter pools lose in a stream of calls, where the launch counts, what they gain on the card: 8 of 98304
// 27.6 / 26.7 and 32.6 / 33.3, 8 of 80000 27.5 / 26.8 and 32.1 / 33.8, 8 of 131072 28.3 / 26.8 and 32.3 / 31.8.
constexpr int TALLY_POOLS = 8, TALLY_POOL = 98304, TALLY_SCORES = 16 << 20;
bool select_by_tally(const SegTable &T) {
  long long pools = 0, longest = 0, rows = 0;
  for (int i = 0; i < T.nseg; ++i) {
    const Seg &s = T.s[i];
    const long long pool = (long long)pool_heads(T, s) * s.n;
    longest = pool > longest ? pool : longest;
    pools += s.head_count / pool_heads(T, s);
    rows += (long long)s.n * s.head_count;
  }
  return pools <= TALLY_POOLS && longest > TALLY_POOL && rows <= TALLY_SCORES;
}

hipError_t launch_select_pools(const SegTable &T, const float *scores, const int *hist1, int *tally, int *sel,
                               int32_t *kept_idx, int32_t *kept_cnt, hipStream_t st) {
  if (T.nheads <= 0) return hipSuccess;
  const SelectScratch z = select_scratch(T);
  if (z.chunks > 0x7fffffffll) return hipErrorInvalidValue;
  uint32_t *cand = reinterpret_cast<uint32_t *>(sel);
  int *rec = sel + z.cand_ints, *coff = rec + z.rec_ints, *state = coff + z.coff_ints;
  const unsigned nb = (unsigned)z.chunks;
  const Range range = hist1 != nullptr ? CAME : tally != nullptr ? TALLIED : SAMPLED_RANGE;
  const bool sampled = range == SAMPLED_RANGE;
  if (range == TALLIED) {
    hipLaunchKernelGGL(fill_zero_kernel, dim3(256), dim3(256), 0, st, tally, (long long)z.pools * HIST1_BINS);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(msel_hist1_kernel, dim3(nb), dim3(CHUNK_THREADS), 0, st, T, scores, tally);
  } else if (sampled) {
    hipLaunchKernelGGL(msel_sample_kernel, dim3((unsigned)z.pools), dim3(SAMPLE_THREADS), 0, st, T, scores, state);
  }
  if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
  const auto candidates = range == CAME      ? msel_cand_kernel<CAME>
                          : range == TALLIED ? msel_cand_kernel<TALLIED>
                                             : msel_cand_kernel<SAMPLED_RANGE>;
  hipLaunchKernelGGL(candidates, dim3(nb), dim3(CHUNK_THREADS), 0, st, T, scores, range == TALLIED ? tally : hist1, cand,
                     rec, state);
  if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
  const int threads = z.pools <= THR_WIDE_POOLS ? 1024 : 256;          // see msel_thr_kernel
  const auto thr = threads == 1024 ? (sampled ? msel_thr_kernel<1024, true> : msel_thr_kernel<1024, false>)
                                   : (sampled ? msel_thr_kernel<256, true> : msel_thr_kernel<256, false>);
  hipLaunchKernelGGL(thr, dim3((unsigned)z.pools), dim3(threads), 0, st, T, scores, cand, rec, coff, state, kept_cnt);
  if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
  hipLaunchKernelGGL(msel_emit_kernel, dim3(nb), dim3(CHUNK_THREADS), 0, st, T, scores, cand, rec,
                     coff, state, kept_idx);
  return hipGetLastError();
}

hipError_t launch_select(const SegTable &T, const float *scores, const int *hist1,
                         int32_t *kept_idx, int32_t *kept_cnt, hipStream_t st) {
  if (T.nheads <= 0) return hipSuccess;
  if (select_needs_pools(T)) return hipErrorInvalidValue;     // longer heads: launch_select_pools
  int most = 0;
  for (int i = 0; i < T.nseg; ++i) most = T.s[i].n > most ? T.s[i].n : most;
  constexpr int ROUND = 4 * SELECT_THREADS;
  const bool h = hist1 != nullptr;
  const auto kernel = most <= ROUND       ? (h ? select_kernel<1, true> : select_kernel<1, false>)
                      : most <= 2 * ROUND ? (h ? select_kernel<2, true> : select_kernel<2, false>)
                      : most <= 4 * ROUND ? (h ? select_kernel<4, true> : select_kernel<4, false>)
                                          : (h ? select_kernel<8, true> : select_kernel<8, false>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)T.nheads), dim3(SELECT_THREADS), 0, st, T, scores, hist1, kept_idx,
                     kept_cnt);
  return hipGetLastError();
}

bool blend_wanted(const SegTable &T) {
  for (int i = 0; i < T.nseg; ++i)
    if (T.s[i].attn != nullptr) return true;
  return false;
}

hipError_t launch_blend(const SegTable &T, float lambda, int score_tokens, float *scores,
                        const double *ostat, int *hist1, hipStream_t st) {
  if (!blend_wanted(T) || T.nheads <= 0) return hipSuccess;
  const bool half = select_chunks(T) <= 512;        // see blend_apply_kernel
  const long long nb = select_chunks(T) * (half ? 2 : 1);
  if (nb > 0x7fffffffll) return hipErrorInvalidValue;
  OstatIndex X;
  long long ob = 0;
  for (int i = 0; i < MAX_SEG; ++i) {
    X.first[i] = ob;
    X.per_head[i] = i < T.nseg ? blocks_per_head(T.s[i].n, score_tokens, SCORE_STEP) : 0;
    if (i < T.nseg) ob += (long long)X.per_head[i] * T.s[i].head_count;
  }
  if (half)
    hipLaunchKernelGGL(blend_apply_kernel<true>, dim3((unsigned)nb), dim3(CHUNK_THREADS), 0, st, T, X, lambda,
                       scores, ostat, hist1);
  else
    hipLaunchKernelGGL(blend_apply_kernel<false>, dim3((unsigned)nb), dim3(CHUNK_THREADS), 0, st, T, X, lambda,
                       scores, ostat, hist1);
  return hipGetLastError();
}

}  // namespace cmp
