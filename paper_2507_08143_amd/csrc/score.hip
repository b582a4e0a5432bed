// Per-row quadratic form (paper Algorithm 1 lines 5-6): o_i = || W^T k_i ||^2, the squared row
// norm of U~ = K_hat V~ Sigma~^{-1} written with the Cholesky factor instead of the SVD.
//
// The contraction runs over the channel axis, which is contiguous in memory, so a key row is an
// MFMA B operand as it stands (16 B per lane); W^T (k_s x 128, as bf16 planes) is staged once
// per workgroup in LDS and read as the A operand.  The output
// tile D[sketch row][token] leaves every lane with 4 sketch rows of one token: squares are
// summed in-lane and two cross-lane exchanges finish the row norm.
//
// W^T reaches the MFMA as a sum of bf16 planes (hi + lo = 16 mantissa bits with two planes):
// bf16 x bf16 products are exact in the fp32 accumulator, so the only rounding besides the
// accumulation itself is the 2^-17 relative error of the split.
#include "factor.h"

namespace cmp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int WPITCH = 136;   // bf16 per LDS row of W^T and of staged key rows (272 B)

// LDS layout of the W^T planes: k_s full rows of 128 channels.  Each row carries 16 bytes of padding:
// consecutive rows are then 68 banks apart and the 16 rows an MFMA operand read touches fall on distinct banks.
template <int M>
struct WLayout {
  static constexpr int PLANE = M * WPITCH;                       // bf16 per plane
  static constexpr int CHUNKS = M * 16;                          // 16-byte pieces per plane
};

// The sum of a lane and the lane 32 away, in both: after swapping the upper half of one copy with the lower half of
// the other the two results of a lane are its own value and the other's.
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float halves_sum(float x) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Where a score workgroup works.  Every wave does this scalar work before its first load can leave, so the
// per-segment numbers come precomputed in the table (index_score_blocks) and one division remains.
__device__ __forceinline__ Where score_locate(const SegTable &T) {
  Where w{0, 0, 0, 0, 0};
  for (int i = 1; i < T.nseg; ++i) w.seg += (int)blockIdx.x >= T.s[i].score_blk0;
  const Seg &s = T.s[w.seg];
  const int local = (int)blockIdx.x - s.score_blk0;
  const int hh = (int)((unsigned)local / (unsigned)s.score_bph);
  w.head = s.head_begin + hh;
  w.lhead = s.lhead0 + hh;
  w.tile = local - hh * s.score_bph;
  w.chunk = s.score_chunk;
  return w;
}

// The way out of a workgroup's scores: bursts of BURST from LDS, and for the blend (a head whose request brings
// attention scores a) this thread's share of the sums and sums of squares of the scores and of a over the
// workgroup's tokens.  a is shifted by the head's first element so that a nearly constant vector does not cancel.
template <int BURST>
struct RunOut {
  static constexpr int APT = BURST / 256;          // a-values per thread and burst
  bool want_stat;
  const float *ap;                                 // of the workgroup's first token
  float a_first;                                   // (converted where it is used: not waited for before)
  double s1 = 0.0, s2 = 0.0, a1 = 0.0, a2 = 0.0;
  float *sp;                                       // of the workgroup's first token

  __device__ __forceinline__ RunOut(const Seg &s, const Where &w, int tok_begin, float *scores, const double *ostat) {
    want_stat = ostat != nullptr && s.attn != nullptr;
    const float *head = want_stat ? s.attn + (long long)w.head * s.n : nullptr;
    a_first = want_stat ? head[0] : 0.f;
    ap = head + tok_begin;
    sp = scores + s.score_off + (long long)w.head * s.n + tok_begin;
  }
  __device__ __forceinline__ void fetch_a(int b0, int cnt, float (&av)[APT]) const {
    if (!want_stat) return;              // uniform
#pragma unroll
    for (int j = 0; j < APT; ++j) av[j] = ap[b0 + min((int)threadIdx.x + 256 * j, cnt - 1)];
  }
  // The scores of tokens [b0, b0 + cnt) of the run leave as 16-byte streaming stores (they disturb
  // the other workgroups' reads least: 1 to 4 % of the kernel's time against plain stores); a
  // burst that does not start on a 16-byte boundary (odd n) gets up to 3 single stores in front.
  __device__ __forceinline__ void burst(const float *sc_l, int b0, int cnt, const float (&av)[APT]) {
    const int tid = threadIdx.x;
    float *dst = sp + b0;
    const int mis = (int)((reinterpret_cast<uintptr_t>(dst) >> 2) & 3u);
    const int lead = min(cnt, mis ? 4 - mis : 0);
    if (tid < lead) dst[tid] = sc_l[tid];
    if (lead == 0) {
      for (int i = 4 * tid; i + 3 < cnt; i += 4 * 256)
        store_stream16(dst + i, *reinterpret_cast<const uint4 *>(&sc_l[i]));
    } else {
      for (int i = lead + 4 * tid; i + 3 < cnt; i += 4 * 256)
        store_stream16(dst + i, make_uint4(__float_as_uint(sc_l[i]), __float_as_uint(sc_l[i + 1]),
                                           __float_as_uint(sc_l[i + 2]), __float_as_uint(sc_l[i + 3])));
    }
    for (int i = lead + ((cnt - lead) & ~3) + tid; i < cnt; i += 256) dst[i] = sc_l[i];
    if (want_stat) {
      const double a_shift = (double)a_first;
#pragma unroll
      for (int j = 0; j < APT; ++j) {
        const int i = tid + 256 * j;
        if (i < cnt) {
          const double x = (double)sc_l[i], y = (double)av[j] - a_shift;
          s1 += x;
          s2 += x * x;
          a1 += y;
          a2 += y * y;
        }
      }
    }
  }
  // The workgroup's sums for the blend, in a fixed order: lanes stride every burst, then a butterfly per wave, then
  // the 4 waves.
  __device__ __forceinline__ void leave_stat(double (*red)[4], double *__restrict__ ostat) {
    if (!want_stat) return;
    const int tid = threadIdx.x, wave = tid >> 6;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      s1 += __shfl_xor(s1, d);
      s2 += __shfl_xor(s2, d);
      a1 += __shfl_xor(a1, d);
      a2 += __shfl_xor(a2, d);
    }
    if ((tid & 63) == 0) { red[wave][0] = s1; red[wave][1] = s2; red[wave][2] = a1; red[wave][3] = a2; }
    __syncthreads();
    if (tid < 4)
      ostat[4 * (size_t)blockIdx.x + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
  }
};

// The workgroup's histogram of the first radix digit (hl: two 16-bit counters per word) is added to the pool's.  A
// head that will be blended gets its histogram from the blend, over the final scores.
__device__ __forceinline__ void leave_hist(const SegTable &T, const Seg &s, const Where &w, const unsigned *hl,
                                           int *__restrict__ hist1) {
  if (hist1 == nullptr || s.attn != nullptr) return;
  const int tid = threadIdx.x;
  // integer adds: order independent
  int *h1 = hist1 + (size_t)(w.lhead / pool_heads(T, s)) * HIST1_BINS;
  // 16 consecutive bins per thread, fetched with two LDS reads; few of them are occupied
  static_assert(HIST1_BINS == 16 * 256, "16 bins per thread");
  const uint4 ha = *reinterpret_cast<const uint4 *>(&hl[8 * tid]);
  const uint4 hb = *reinterpret_cast<const uint4 *>(&hl[8 * tid + 4]);
  const unsigned wd[8] = {ha.x, ha.y, ha.z, ha.w, hb.x, hb.y, hb.z, hb.w};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int lo = (int)(wd[j] & 0xffffu), hi = (int)(wd[j] >> 16);
    if (lo) atomicAdd(&h1[hist_at(16 * tid + 2 * j)], lo);
    if (hi) atomicAdd(&h1[hist_at(16 * tid + 2 * j + 1)], hi);
  }
}

// Sketched mode.  A workgroup walks tokens_per_wg tokens of one head in steps of 128 (32 per wave, two 16-token
// sub-tiles).  Key rows arrive with fully coalesced streaming loads (a wave instruction covers
// four whole 256-byte rows), pass through a wave-private LDS buffer, and are read back in the
// MFMA B-operand arrangement; a step of loads is in flight while the one before is multiplied.  With two the kernel
// is 1 to 3 % slower where the memory is busy: 256 heads of 32768 tokens, 48 rows, 343 us, 352 with two, 345 where both are waited
// for together; 16 rows 326.6, 338.3 and 328.2, 512 of 8192 token by token 169.3, 180.9 and 173.3.
// Two workgroups a unit, also at 16 rows, where registers and LDS (if not for ROOM) allow three: the third costs as much as
// a second step in flight, 256 heads of 32768 326.6 -> 337.2, 192 of 34660 token by token 283.6 -> 290.6, 512 of 8192 169.3 ->
// 180.4.
// The multiply loop needs no workgroup barrier: a wave only reads what it wrote itself.  The
// scores collect in LDS and leave in bursts of BURST tokens; a run may span several bursts (up to
// SCORE_MAX_RUN tokens), so that what a workgroup pays once (staging W^T, the histogram, filling
// and draining its load pipeline) is spread over more rows; the loads of the steps that follow a
// burst are already in flight while it is written.
//
// SOLVE: every workgroup factors its head itself, from the shares of S, and W^T goes straight into its LDS.  The
// work is done many times over, but by compute units that would wait for it, and a launch and two passes of W^T
// through memory are saved (see score_solves).
// (At M = 64 its LDS leaves room for one on a unit, which is also all that score_solves asks for.)
template <int M, bool SOLVE>
__global__ __launch_bounds__(256, SOLVE && M == 64 ? 1 : 2) void score_kernel(
    const SegTable T, const uint16_t *__restrict__ wt, const ScoreSolve V, float *__restrict__ scores,
    int32_t *__restrict__ status, int *__restrict__ hist1, double *__restrict__ ostat) {
  constexpr int NSUB = 2, WTOK = 16 * NSUB, STEP = 4 * WTOK;     // tokens per wave / per WG step
  constexpr int NLD = WTOK * 16 / 64;                            // 16-B loads per lane per step
  typedef WLayout<M> WL;
  constexpr int ROOM = W_TERMS * (M < 32 ? WLayout<32>::PLANE : WL::PLANE);      // keeps a third workgroup off a unit
  __shared__ __attribute__((aligned(16))) uint16_t wl[ROOM];
  constexpr int BURST = SCORE_BURST, BSTEPS = BURST / STEP;
  static_assert((BURST & (BURST - 1)) == 0, "bursts wrap round in LDS");
  struct Stream {
    // a wave stages 16 tokens at a time (its 32 tokens of a step in two halves); measured, a third
    // workgroup per CU does not pay, the smaller staging buffer does on the long-context shapes
    uint16_t kl[4][16 * WPITCH];
    // first radix digit of the selection, tallied on the way out: two 16-bit counters per word
    unsigned hl[HIST1_BINS / 2];
    // The scores collect here and leave in bursts: 4-byte stores trickling out between the
    // streaming reads cost 12 % of the kernel's time.
    float sc_l[BURST];
  };
  union Lds {                            // the factorisation is over when the first key is staged
    Stream s;
    SketchFactor<SOLVE ? M : 16> f;
  };
  __shared__ __attribute__((aligned(16))) Lds lds;
  auto &kl = lds.s.kl;
  auto &hl = lds.s.hl;
  auto &sc_l = lds.s.sc_l;
  __shared__ double red[4][4];
  static_assert(3 * (sizeof(wl) + sizeof(lds) + sizeof(red)) > 160 * 1024, "two workgroups a unit");

  PhiRegs<SOLVE ? M : 16> ph;
  if constexpr (SOLVE) ph.fetch(V.phi);
  const Where w = score_locate(T);
  const Seg &s = T.s[w.seg];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t16 = lane & 15, g = lane >> 4;
  const int n = s.n;
  const int tok_begin = w.tile * w.chunk;
  const int tok_end = min(n, tok_begin + w.chunk);
  const int nsteps = (tok_end - tok_begin + STEP - 1) / STEP;
  const long long stride_t = s.stride_t;
  const uint16_t *kp = head_ptr(s.k_score, s, w.head);
  const int ld_row = lane >> 4, ld_chunk = lane & 15;            // loader: 16 lanes per row

  // A run's last step reads copies of its last row, whose scores nobody stores: with a load under a condition the number of
  // loads under way depends on the way taken, and the wait for the shares of S, requested before, is one for the keys too.
  const int last_row = tok_end - tok_begin - 1;
  const uint16_t *run = kp + (long long)tok_begin * stride_t + ld_chunk * 8;
  const uint16_t *lane_base = run + (long long)(wave * WTOK + ld_row) * stride_t;
  const long long row4 = 4 * stride_t, step_stride = (long long)STEP * stride_t;
  auto load_step = [&](int it, uint4 (&to)[NLD]) {
    const uint16_t *at[NLD];
    if (it * STEP + (wave + 1) * WTOK <= last_row + 1) {         // uniform: every step but a run's last
      const uint16_t *p = lane_base + it * step_stride;
#pragma unroll
      for (int i = 0; i < NLD; ++i) at[i] = p + i * row4;
    } else {
#pragma unroll
      for (int i = 0; i < NLD; ++i) at[i] = run + min(it * STEP + wave * WTOK + ld_row + 4 * i, last_row) * stride_t;
    }
#pragma unroll
    for (int i = 0; i < NLD; ++i) to[i] = load_stream16(at[i]);
    __builtin_amdgcn_sched_barrier(0);             // they leave before what is multiplied meanwhile
  };

  RunOut<BURST> out(s, w, tok_begin, scores, ostat);
  // the shares of S are wanted first, and loads arrive in order
  ShareSum<SOLVE ? M : 16> ss;
  const double *shares = nullptr;
  if constexpr (SOLVE) {
    shares = V.shares + (long long)w.lhead * V.nshares * Share<M>::DOUBLES;
    ss.fetch(shares);
    __builtin_amdgcn_sched_barrier(0);
  }
  uint4 stg[NLD];
  load_step(0, stg);
  // W^T follows the first step of keys through the load queue and waits in registers, so that the second step can be
  // requested as soon as the first has arrived and not only once W^T is in LDS
  constexpr int WN = (W_TERMS * WL::CHUNKS + 255) / 256;
  uint4 wreg[WN];
  if constexpr (SOLVE) {
    double sum[Share<M>::TILES];
    ss.add(shares, V.nshares, sum);
    // The memory would wait for the factorisation: the rows of the next two steps are brought as far as the L2 by one dword
    // a line, a few at a time by the waves that wait for pivots.  More, or all at once, keep those waves from their part of the
    // factorisation.  Whole call on MI355X, us with 0 / 2 / 4 / 5 / 6 steps: scores of 8 heads of 40007, k_s = 32, 48.6 / 47.5 /
    // 47.7 / 48.6 / 49.7, 4 x 8 x 16383 blended 128.8 / 128.0 / 128.1 / 128.8 / 130.3, 8 heads of 131072 165.4 / 165.5 / 165.9 /
    // 166.2 / 167.6; four steps by all waves before the factorisation 50.2, 133 and 171.
    constexpr int AHEAD = 2, POINTS = M / 16, EACH = (AHEAD * STEP / 32 + 3 * POINTS - 1) / (3 * POINTS);
    unsigned ahead[POINTS * EACH] = {};
    sketch_factor<M>(lds.f, sum, ph, V.ridge_rel,
                     [&](int t, int row, int ch, uint16_t v) { wl[t * WL::PLANE + row * WPITCH + ch] = v; },
                     [&](auto jc) {
                       constexpr int j = decltype(jc)::value;
#pragma unroll
                       for (int u = j * EACH; u < (j + 1) * EACH; ++u) {
                         const int at = STEP + 32 * (3 * u + wave - 1), rows = tok_end - tok_begin;
                         if (at < min(rows, (1 + AHEAD) * STEP))       // uniform
                           ahead[u] = *reinterpret_cast<const unsigned *>(
                               kp + ((long long)tok_begin + min(at + (lane >> 1), rows - 1)) * stride_t + 64 * (lane & 1));
                       }
                     });
#pragma unroll
    for (int u = 0; u < POINTS * EACH; ++u) asm volatile("" ::"v"(ahead[u]));
    __syncthreads();
    if (w.tile == 0 && tid == 0 && lds.f.flag) atomicOr(&status[s.ghead0 + w.head], lds.f.flag);
    __syncthreads();
  }
  const uint16_t *wh = wt + (size_t)w.lhead * (W_TERMS * M * D);
#pragma unroll
  for (int i = 0; i < (SOLVE ? 0 : WN); ++i) {
    const int cidx = tid + 256 * i;
    wreg[i] = make_uint4(0, 0, 0, 0);
    if (cidx < W_TERMS * WL::CHUNKS) {
      const int t = cidx / WL::CHUNKS, c = cidx - t * WL::CHUNKS, row = c >> 4, ch = c & 15;
      wreg[i] = *reinterpret_cast<const uint4 *>(wh + (t * M + row) * D + ch * 8);
    }
  }
  for (int i = tid; i < HIST1_BINS / 2; i += 256) hl[i] = 0;

  uint16_t *kw = kl[wave];
  bool bad = false;

  bf16x8 kb[NSUB][4];
  auto redistribute = [&](const uint4 (&from)[NLD]) {
    // redistribute through the wave's LDS buffer: rows in, B operands out.  Lanes exchange
    // data here without a workgroup barrier (LDS operations of one wave execute in order), so
    // wave-scope fences keep the compiler from moving the reads and writes across each other.
#pragma unroll
    for (int st = 0; st < NSUB; ++st) {
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < NLD / NSUB; ++i)
        *reinterpret_cast<uint4 *>(&kw[(ld_row + 4 * i) * WPITCH + ld_chunk * 8]) = from[st * (NLD / NSUB) + i];
      wave_lds_fence();
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        kb[st][kk] = *reinterpret_cast<const bf16x8 *>(&kw[t16 * WPITCH + 32 * kk + 8 * g]);
    }
  };
  auto multiply = [&](int it) {
    float sums[NSUB];
#pragma unroll
    for (int st = 0; st < NSUB; ++st) sums[st] = 0.f;
    constexpr int JB_UNROLL = M <= 48 ? M / 16 : 1;
#pragma unroll JB_UNROLL
    for (int jb = 0; jb < M / 16; ++jb) {   // rolled for many rows: unrolling hoists their operands
      f32x4 acc[NSUB];
#pragma unroll
      for (int st = 0; st < NSUB; ++st) acc[st] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int wrow = (jb * 16 + t16) * WPITCH;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
        for (int t = 0; t < W_TERMS; ++t) {
          const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&wl[t * WL::PLANE + wrow + 32 * kk + 8 * g]);
#pragma unroll
          for (int st = 0; st < NSUB; ++st)
            acc[st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, kb[st][kk], acc[st], 0, 0, 0);
        }
      }
#pragma unroll
      for (int st = 0; st < NSUB; ++st)
        sums[st] += acc[st][0] * acc[st][0] + acc[st][1] * acc[st][1] +
                    acc[st][2] * acc[st][2] + acc[st][3] * acc[st][3];
    }
    // lanes (t16, g = 0..3) hold the four quarter-sums of token t16 of both sub-tiles; after
    // the exchange lanes with g < 2 hold the full sum of sub-tile g
    // (row swaps: two shuffles, round trips through LDS, took 0.2 us a step)
    const float x0 = halves_sum(sums[0]), x1 = halves_sum(sums[1]);
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
    const float x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    const int tok = tok_begin + it * STEP + wave * WTOK + (lane & 31);   // 16*(g&1) + t16
    if (g < 2 && tok < tok_end) {
      sc_l[(tok - tok_begin) & (BURST - 1)] = x;
      bad |= !(fabsf(x) <= 3.0e38f);
      const uint32_t bin = score_key(x) >> 20;
      atomicAdd(&hl[bin >> 1], 1u << (16 * (bin & 1)));
    }
  };

  redistribute(stg);
  if (nsteps > 1) load_step(1, stg);                            // uniform
#pragma unroll
  for (int i = 0; i < (SOLVE ? 0 : WN); ++i) {
    const int cidx = tid + 256 * i;
    if (cidx < W_TERMS * WL::CHUNKS) {
      const int t = cidx / WL::CHUNKS, c = cidx - t * WL::CHUNKS, row = c >> 4, ch = c & 15;
      *reinterpret_cast<uint4 *>(&wl[t * WL::PLANE + row * WPITCH + ch * 8]) = wreg[i];
    }
  }
  __syncthreads();

  auto leave = [&](int b0) {
    const int cnt = min(BURST, tok_end - tok_begin - b0);
    float av[RunOut<BURST>::APT];
    out.fetch_a(b0, cnt, av);    // on their way while the waves meet
    __syncthreads();
    out.burst(sc_l, b0, cnt, av);
  };
  // the operands of step `it` are in registers (kb) and the loads of the next one in flight
  for (int it = 0; it + 1 < nsteps; ++it) {
    multiply(it);
    if ((it + 1) % BSTEPS == 0) {                   // uniform: a burst is complete
      leave((it / BSTEPS) * BURST);
      __syncthreads();                              // before the next burst's scores overwrite these
    }
    redistribute(stg);
    if (it + 2 < nsteps) load_step(it + 2, stg);    // uniform
  }
  multiply(nsteps - 1);
  leave((nsteps - 1) / BSTEPS * BURST);
  if (__any(bad)) {
    if (lane == 0) atomicOr(&status[s.ghead0 + w.head], COMPACTOR_STATUS_NONFINITE);
  }
  out.leave_stat(red, ostat);
  leave_hist(T, s, w, hl, hist1);
}

// Exact mode: W^T = L^{-1}, 128 rows, lower triangular (row j is zero beyond channel j): 20 of 32 blocks of 16 rows x
// 32 channels to multiply.  Wave w of a workgroup owns the 16-row blocks w and 7 - w, five of those 20 each, as MFMA
// operands in registers (40 of them), and multiplies every token of the workgroup with them; the four waves' shares
// of a row norm meet in LDS.  The keys of a step (64 tokens) are staged once per workgroup, in two buffers, so that a
// step needs one barrier: a wave that writes a buffer has passed the barrier behind the last reads of it.
// Bound by the stream of keys (5.4 TB/s under the power limit, matrix cores half busy): 32 heads of 50001 tokens on
// MI355X 87 us, 75 at best, against 93 and 86 with W^T in LDS, where two workgroups a CU of 79 KB read 10 KB of
// operands for 16 tokens and waited 42 % of the time; whole compression 300 -> 292 us, 256 heads of 16384, scores alone,
// 408 -> 397.  Four steps in flight leave registers for two workgroups only: 202 instead of 189 us for the scores of the
// 32 heads.
constexpr int EX_STEP = 64;

__global__ __launch_bounds__(256, 3) void score_exact_kernel(
    const SegTable T, const uint16_t *__restrict__ wt, float *__restrict__ scores,
    int32_t *__restrict__ status, int *__restrict__ hist1, double *__restrict__ ostat) {
  constexpr int M = 128, TILES = EX_STEP / 16, NLD = EX_STEP / 16, AHEAD = 2;      // loads per lane per step; steps in flight
  constexpr int BURST = SCORE_EXACT_BURST, BSTEPS = BURST / EX_STEP;
  static_assert(TILES == 4 && AHEAD % 2 == 0 && (BURST & (BURST - 1)) == 0, "a lane a token, buffers in turn");
  __shared__ __attribute__((aligned(16))) uint16_t kl[2][EX_STEP * WPITCH];
  __shared__ __attribute__((aligned(16))) unsigned hl[HIST1_BINS / 2];
  __shared__ __attribute__((aligned(16))) float sc_l[BURST];
  __shared__ float part[2][4][EX_STEP];
  __shared__ double red[4][4];

  const Where w = score_locate(T);
  const Seg &s = T.s[w.seg];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t16 = lane & 15, g = lane >> 4;
  const int tok_begin = w.tile * w.chunk;
  const int tok_end = min(s.n, tok_begin + w.chunk);
  const int nsteps = (tok_end - tok_begin + EX_STEP - 1) / EX_STEP;
  const int last_row = tok_end - tok_begin - 1;
  const long long stride_t = s.stride_t;
  // loader: 16 lanes per row, 16 rows of a step per wave; past the run's end its last row, whose copies nobody adds up
  const uint16_t *run = head_ptr(s.k_score, s, w.head) + tok_begin * stride_t + t16 * 8;
  auto load_step = [&](int it, uint4 (&stg)[NLD]) {
#pragma unroll
    for (int i = 0; i < NLD; ++i)
      stg[i] = load_stream16(run + min(it * EX_STEP + wave * 16 + g + 4 * i, last_row) * stride_t);
  };
  uint4 stg[AHEAD][NLD];
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) load_step(u, stg[u]);
  // blocks kk = 0 .. 2 of the wave's later rows, then their last or, where they have three, the second of the
  // earlier rows, then the first of those
  bf16x8 wr[5][W_TERMS];
  const bool four = wave < 2;
  {
    const int hi = 7 - wave, lo = wave;
    const uint16_t *wh = wt + (size_t)w.lhead * (W_TERMS * M * D) + t16 * D + 8 * g;
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      const int jb = b < 3 || (b == 3 && four) ? hi : lo, kk = b < 3 ? b : b == 4 ? 0 : four ? 3 : 1;
#pragma unroll
      for (int t = 0; t < W_TERMS; ++t)
        wr[b][t] = *reinterpret_cast<const bf16x8 *>(wh + (t * M + jb * 16) * D + 32 * kk);
    }
  }
  for (int i = tid; i < HIST1_BINS / 2; i += 256) hl[i] = 0;

  RunOut<BURST> out(s, w, tok_begin, scores, ostat);
  bool bad = false;
  // the barrier between what waves put into LDS and what others take out; loads from memory stay in flight
  auto meet = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  // this wave's share of the row norms of a step, lane l token l
  auto multiply = [&](auto last_blocks, int buf) {
    constexpr int HI = decltype(last_blocks)::value;
    float sums[TILES];
#pragma unroll
    for (int st = 0; st < TILES; ++st) {
      bf16x8 kb[HI];
#pragma unroll
      for (int kk = 0; kk < HI; ++kk)
        kb[kk] = *reinterpret_cast<const bf16x8 *>(&kl[buf][(16 * st + t16) * WPITCH + 32 * kk + 8 * g]);
      f32x4 hi{0.f, 0.f, 0.f, 0.f}, lo{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < HI; ++kk)
#pragma unroll
        for (int t = 0; t < W_TERMS; ++t) {
          hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[kk][t], kb[kk], hi, 0, 0, 0);
          if (kk < 5 - HI) lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[kk == 0 ? 4 : 3][t], kb[kk], lo, 0, 0, 0);
        }
      sums[st] = hi[0] * hi[0] + hi[1] * hi[1] + hi[2] * hi[2] + hi[3] * hi[3] +
                 (lo[0] * lo[0] + lo[1] * lo[1] + lo[2] * lo[2] + lo[3] * lo[3]);
    }
    // lanes (t16, g = 0..3) hold four quarter-sums of token t16 of every tile: two exchanges leave
    // tile g's sum in lanes (t16, g)
    float x[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(sums[h]), __float_as_uint(sums[h + 2]), false, false);
      x[h] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[0]), __float_as_uint(x[1]), false, false);
    part[buf][wave][lane] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  // the row norms of step `it` from the waves' shares, by one wave
  auto add_up = [&](int it) {
    if (wave != (it & 3)) return;
    const int at = it * EX_STEP + lane;
    const auto &p = part[it & 1];
    const float x = (p[0][lane] + p[1][lane]) + (p[2][lane] + p[3][lane]);
    if (tok_begin + at < tok_end) {
      sc_l[at & (BURST - 1)] = x;
      bad |= !(fabsf(x) <= 3.0e38f);
      const uint32_t bin = score_key(x) >> 20;
      atomicAdd(&hl[bin >> 1], 1u << (16 * (bin & 1)));
    }
  };
  auto leave = [&](int b0, int cnt) {
    float av[RunOut<BURST>::APT];
    out.fetch_a(b0, cnt, av);            // on their way while the waves meet
    meet();
    out.burst(sc_l, b0, cnt, av);        // read before the barrier behind which scores are added up next
  };

  int it0 = 0;
  for (; it0 < nsteps; it0 += AHEAD) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const int it = it0 + u;
#pragma unroll
      for (int i = 0; i < NLD; ++i)
        *reinterpret_cast<uint4 *>(&kl[u & 1][(wave * 16 + g + 4 * i) * WPITCH + t16 * 8]) = stg[u][i];
      load_step(it + AHEAD, stg[u]);
      meet();
      if (it > 0) {
        add_up(it - 1);
        if (u == 0 && it % BSTEPS == 0) leave((it - BSTEPS) * EX_STEP, BURST);
      }
      if (four) multiply(std::integral_constant<int, 4>{}, u & 1);
      else multiply(std::integral_constant<int, 3>{}, u & 1);
    }
  }
  meet();
  add_up(it0 - 1);
  const int b0 = (nsteps - 1) / BSTEPS * BURST;
  leave(b0, tok_end - tok_begin - b0);
  if (__any(bad)) {
    if (lane == 0) atomicOr(&status[s.ghead0 + w.head], COMPACTOR_STATUS_NONFINITE);
  }
  out.leave_stat(red, ostat);
  leave_hist(T, s, w, hl, hist1);
}

// Whether the score workgroups of a launch factor their heads themselves: where each has a compute unit of its own.
// The pivots of two on a unit, and the shares that all of them read, take longer than what is saved (8 heads of
// 131072 tokens in 512 workgroups: 36 us before the first score, against 16 for the kernel that does it once).  With 64
// sketch rows up to runs of 1536 tokens: 32 heads of 30000, 256 workgroups, 125 against 119 us.
bool score_solves(const SegTable &T, int ks, int tokens_per_wg, int cus) {
  if (ks == 0 || (ks > 48 && tokens_per_wg > 1536)) return false;
  return total_blocks(T, tokens_per_wg, SCORE_STEP, false) <= cus;
}

template <int M, bool SOLVE>           // M = 128: exact mode
static hipError_t launch_m(const SegTable &T, int tokens_per_wg, const uint16_t *wt, const ScoreSolve &V,
                           float *scores, int32_t *status, int *hist1, double *ostat,
                           hipStream_t st) {
  SegTable Ti = T;
  const long long nb = index_score_blocks(Ti, tokens_per_wg);
  if (nb <= 0) return hipSuccess;
  if (nb > 0x7fffffffll) return hipErrorInvalidValue;
  if constexpr (M == 128)
    hipLaunchKernelGGL(score_exact_kernel, dim3((unsigned)nb), dim3(256), 0, st, Ti, wt, scores, status, hist1, ostat);
  else
    hipLaunchKernelGGL((score_kernel<M, SOLVE>), dim3((unsigned)nb), dim3(256), 0, st, Ti, wt, V, scores, status,
                     hist1, ostat);
  return hipGetLastError();
}

hipError_t launch_score(const SegTable &T, int ks, int tokens_per_wg, const uint16_t *wt, const ScoreSolve *solve,
                        float *scores, int32_t *status, int *hist1, double *ostat, hipStream_t st) {
  const ScoreSolve V = solve ? *solve : ScoreSolve{nullptr, 0, nullptr, 0.f};
  const auto launch = ks == 16   ? (solve ? launch_m<16, true> : launch_m<16, false>)
                      : ks == 32 ? (solve ? launch_m<32, true> : launch_m<32, false>)
                      : ks == 48 ? (solve ? launch_m<48, true> : launch_m<48, false>)
                      : ks == 64 ? (solve ? launch_m<64, true> : launch_m<64, false>)
                                 : launch_m<128, false>;
  if (!(ks == 16 || ks == 32 || ks == 48 || ks == 64 || (ks == 0 && !solve))) return hipErrorInvalidValue;
  return launch(T, tokens_per_wg, wt, V, scores, status, hist1, ostat, st);
}

}  // namespace cmp
