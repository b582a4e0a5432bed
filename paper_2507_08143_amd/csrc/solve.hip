// Small per-head factorisation (paper Algorithm 1 line 4, in the Cholesky form; Appendix C
// notes that routes other than the SVD give the same scores).
//
//   sketched:  S = Phi^T G Phi + rho I  (k_s x k_s),   exact:  S = G + rho I  (d x d)
//   S = L L^T,   W^T = L^{-1} Phi^T  (k_s x d)   [exact: W^T = L^{-1}]
//
// so that the score of a token is o_i = || W^T k_i ||^2 = k^_i^T S^{-1} k^_i, which equals
// diag(U~ U~^T) of Algorithm 1 lines 5-6 when rho = 0.  All arithmetic here is fp64; W^T leaves
// as a sum of bf16 planes for the MFMA score pass.
#include <algorithm>

#include "factor.h"

namespace cmp {

__device__ __forceinline__ Where locate_head(const SegTable &T, int lhead) {
  Where w{0, 0, lhead, 0, 0};
  for (int i = 0; i < T.nseg; ++i) {
    const int hh = lhead - T.s[i].lhead0;
    if (hh < T.s[i].head_count || i == T.nseg - 1) {
      w.seg = i;
      w.head = T.s[i].head_begin + hh;
      return w;
    }
  }
  return w;
}

// ---- sketched mode: partial Gram blocks -> S -> L -> L^{-1} -> W^T ------------------------------
// Every O(n^3)-ish piece runs on the fp64 matrix cores (16x16x4 MFMA: A[i][k] in lane (i = l & 15,
// k = l >> 4), B[k][j] in lane (j = l & 15, k = l >> 4), register v of lane l of the result is
// D[4v + (l >> 4)][l & 15]):
//   1. S = Phi^T G Phi, G summed in fp64 from the head's partial blocks
//   2. blocked right-looking Cholesky of S + rho I with 16-wide panels: wave 0 inverts the factor
//      of the diagonal block in registers (the only serial part, 16 pivots), the panel below is
//      L_qp = A_qp X_pp^T and the trailing blocks get A_qr -= L_qp L_rp^T
//   3. W^T = L^{-1} Phi^T by forward substitution (sketch_factor; exact mode: X = L^{-1} itself, block by block)
//   4. W^T split into bf16 planes
// Steps 2 to 4 stand in factor.h.
//
// Step 1 is linear in the blocks and in the partials of a head, so it is cut into shares: share
// (r, w) is the contribution of stored blocks 2w and 2w + 1 of the r-th part of the head's
// partials, w < SHARE_BLOCKS.  B = sum over blocks (I, J) of Phi_J^T G_IJ^T Phi_I, the diagonal
// blocks halved, gives S = B + B^T.  The shares of a head are added in their order, whoever
// computes them: with room in the workspace they are computed by workgroups of their own
// (sketch_share_kernel) and added by the factorisation, otherwise one workgroup per head computes
// them one after the other.  Both give the same bits.  Many heads go another way whatever the room (sketch_direct_kernel).
// The stored upper block number b is block (I, J) of G.
__device__ __forceinline__ void upper_block_pos(int b, int &I, int &J) {
  I = (b >= 4) + (b >= 7) + (b >= 9);
  J = b - upper_block(I, I) + I;
}

// The fp64 sum, in their order, of Q float4, 512 floats apart, over `count` partials.  A batch costs a round trip of about
// 1 us, so the next batch leaves before one is added, and no load stands under a condition: each of those would be waited
// for by itself (a batch repeats the last partial instead, and does not add it; one or two left over go by themselves).  With two
// float4 a batch is four partials: with eight the share kernel has registers for two workgroups a unit instead of three, 128 heads of
// 34660, k_s = 48, 393 us and not 390, and eight heads no less.  Whole
// scores on MI355X, us, k_s = 48, 8 heads of 3000 / 10000, 64 of 7000: 28.3 -> 27.4, 35.6 -> 34.2, 66.9 -> 65.4; exact mode, where
// one load waited for the other, 8 heads of 3000 / 10000: 46.0 -> 44.6, 54.5 -> 49.7.
// HALVES: partial i is the fp32 sum of those at 2i and 2i + 1, as far as they lie within least .. most.
template <int Q, int FLIGHT = 8, bool HALVES = false>
__device__ __forceinline__ void sum_quads(const float *__restrict__ src, int count, double (&g)[4 * Q], int least = 0,
                                          int most = 0) {
  constexpr int FEW = FLIGHT >= 8 ? 2 : 1;
  struct Batch {
    float4 v[FLIGHT][Q], w[HALVES ? FLIGHT : 1][Q];
    bool two[FLIGHT];
  };
  auto load = [&](int s0, Batch &b, auto n) {
#pragma unroll
    for (int u = 0; u < decltype(n)::value; ++u) {
      const int i = min(s0 + u, count - 1), lo = HALVES ? max(2 * i, least) : i, hi = HALVES ? min(2 * i + 1, most) : i;
      b.two[u] = lo < hi;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        b.v[u][q] = *reinterpret_cast<const float4 *>(src + (long long)lo * GRAM_PARTIAL_FLOATS + 512 * q);
        if constexpr (HALVES)
          b.w[u][q] = *reinterpret_cast<const float4 *>(src + (long long)hi * GRAM_PARTIAL_FLOATS + 512 * q);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto add = [&](int u, const Batch &b) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      float4 x = b.v[u][q];
      if constexpr (HALVES) {
        const float4 y = b.w[u][q];
        const bool two = b.two[u];         // (no branch: what waits in it would be waited for apart)
        x = make_float4(x.x + (two ? y.x : 0.f), x.y + (two ? y.y : 0.f), x.z + (two ? y.z : 0.f), x.w + (two ? y.w : 0.f));
      }
      g[4 * q] += x.x; g[4 * q + 1] += x.y; g[4 * q + 2] += x.z; g[4 * q + 3] += x.w;
    }
  };
  auto add_all = [&](const Batch &b) {
#pragma unroll
    for (int u = 0; u < FLIGHT; ++u) add(u, b);
  };
  auto add_some = [&](int n, const Batch &b) {
#pragma unroll
    for (int u = 0; u < FLIGHT; ++u)
      if (u < n) add(u, b);                // uniform
  };
  const std::integral_constant<int, FLIGHT> all;
#pragma unroll
  for (int i = 0; i < 4 * Q; ++i) g[i] = 0.0;
  if (count <= 0) return;                  // uniform
  Batch a, b;
  load(0, a, all);
  int sp = 0;
  for (; sp + 2 * FLIGHT < count; sp += 2 * FLIGHT) {
    load(sp + FLIGHT, b, all);
    add_all(a);
    load(sp + 2 * FLIGHT, a, all);
    add_all(b);
  }
  const int left = count - sp - FLIGHT;
  if (left > FEW) {
    load(sp + FLIGHT, b, all);
    add_all(a);
    add_some(left, b);
  } else if (left > 0) {
    load(sp + FLIGHT, b, std::integral_constant<int, FEW>{});
    add_all(a);
    add(0, b);
    if (FEW > 1 && left > 1) add(FEW - 1, b);
  } else {
    add_some(count - sp, a);
  }
}

// Share w of the partials src[0 .. count): B of it, in two halves, is left in ba and bb (M rows of
// pitch M + 1; the share is ba + bb), complete after a barrier.  A wave takes 16 columns of a
// block: lane (l16, lq) reads rows 4lq .. 4lq + 3 and 16 + 4lq .. of column l16 with two 16-byte
// loads per partial and holds them as A operands of T = G^T Phi_I as they are (step (h, s) of the
// contraction takes row 16h + 4lq + s of lane group lq); T's accumulators are the B operands of
// Phi_J^T T.  Nothing of G or T passes through LDS.
template <int M, bool HALVES = false>
__device__ __forceinline__ void sketch_share(const float *__restrict__ src, int count, int w,
                                             const float *__restrict__ phi, double *ba, double *bb, int least = 0, int most = 0) {
  constexpr int CT = M / 16, SP = M + 1;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = 2 * w + (wave >> 1), half = wave & 1;
  int I, J;
  upper_block_pos(b, I, J);
  const float *p = src + (b * 1024 + (32 * lq + 16 * half + l16) * 4);
  // operands of both products from Phi, requested before the partials
  float pi[8][CT], pj[4][CT];
#pragma unroll
  for (int q = 0; q < 8; ++q)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      pi[q][ct] = phi[(32 * I + 16 * (q >> 2) + 4 * lq + (q & 3)) * M + 16 * ct + l16];
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      pj[v][ct] = phi[(32 * J + 16 * half + 4 * v + lq) * M + 16 * ct + l16];
  double g[8];
  sum_quads<2, HALVES ? 2 : 4, HALVES>(p, count, g, least, most);
  f64x4 tacc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) tacc[ct] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 8; ++q)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      tacc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[q], (double)pi[q][ct], tacc[ct], 0, 0, 0);
  const double sc = I == J ? 0.5 : 1.0;
  f64x4 sacc[CT][CT];
#pragma unroll
  for (int at = 0; at < CT; ++at)
#pragma unroll
    for (int bt = 0; bt < CT; ++bt) sacc[at][bt] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int at = 0; at < CT; ++at)
#pragma unroll
      for (int bt = 0; bt < CT; ++bt)
        sacc[at][bt] = __builtin_amdgcn_mfma_f64_16x16x4f64(sc * (double)pj[v][at], tacc[bt][v],
                                                            sacc[at][bt], 0, 0, 0);
  // (wave 0 + wave 2) into ba, (wave 1 + wave 3) into bb
  double *dst = (wave & 1) ? bb : ba;
  if (wave >= 2) {
#pragma unroll
    for (int at = 0; at < CT; ++at)
#pragma unroll
      for (int bt = 0; bt < CT; ++bt)
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[(16 * at + 4 * v + lq) * SP + 16 * bt + l16] = sacc[at][bt][v];
  }
  __syncthreads();
  if (wave < 2) {
#pragma unroll
    for (int at = 0; at < CT; ++at)
#pragma unroll
      for (int bt = 0; bt < CT; ++bt)
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[(16 * at + 4 * v + lq) * SP + 16 * bt + l16] += sacc[at][bt][v];
  }
}

// Part r of `parts` of a head's nsplit partials.
__device__ __forceinline__ void split_part(int nsplit, int parts, int r, int &first, int &count) {
  const int per = (nsplit + parts - 1) / parts;
  first = min(nsplit, r * per);
  count = min(nsplit, first + per) - first;
}

// One workgroup per (head, part, share).  Bound by latency: one batch of partials after the
// other, 60 MFMAs (k_s = 48) a wave, two barriers: 7 to 10 us for 8 heads with 8 to 64 partials
// each, where one workgroup per head took 34 (8 partials, 4-byte loads) to 185 us (64) for this
// step.  At 256 heads (24 us) the fp64 matrix cores count, 1200 MFMAs of 64 clocks a head: see sketch_direct_kernel.
// The slot where the halves of a head's partial `first` are (of which pb is the first's), or would be, and which of the slots from
// there on are the head's.
struct HalfRuns {
  long long slot;
  int least, most;
  __device__ __forceinline__ HalfRuns(long long t0, int tph, int lhead, long long pb, int first) {
    int count;
    const long long mine = partial_base(t0, tph, lhead, GRAM_HALF_RUN, count);
    slot = 2 * (pb - lhead + first) + lhead;
    least = (int)(mine - slot);
    most = least + count - 1;
  }
};

// HALVES: the partials are those of workgroups of half a run (GRAM_HALF), numbered as such; they are paired, and the pairs dealt out
// and added in their order, as the partials of whole runs are.
template <int M, bool HALVES>
__global__ __launch_bounds__(256, 2) void sketch_share_kernel(
    const SegTable T, int tiles_per_wg, int parts, const float *__restrict__ partials,
    const float *__restrict__ phi, double *__restrict__ shares, int32_t *__restrict__ status,
    int *__restrict__ zero, long long zero_ints) {
  constexpr int SP = M + 1;
  __shared__ double ba[M * SP], bb[M * SP];
  const int unit = blockIdx.x / SHARE_BLOCKS, w = blockIdx.x - unit * SHARE_BLOCKS;
  const int lhead = unit / parts, r = unit - lhead * parts;
  if (status != nullptr && r == 0 && w == 0 && threadIdx.x == 0) {
    const Where at = locate_head(T, lhead);
    status[T.s[at.seg].ghead0 + at.head] = 0;
  }
  int tph = 0, nsplit, first, count;
  const long long t0 = head_tiles(T, lhead, tph);
  const long long pb = partial_base(t0, tph, lhead, HALVES ? 2 * GRAM_HALF_RUN : tiles_per_wg, nsplit);
  split_part(nsplit, parts, r, first, count);
  if constexpr (HALVES) {
    const HalfRuns hr(t0, tph, lhead, pb, first);
    sketch_share<M, true>(partials + hr.slot * GRAM_PARTIAL_FLOATS, count, w, phi, ba, bb, hr.least, hr.most);
  } else {
    sketch_share<M>(partials + (pb + first) * GRAM_PARTIAL_FLOATS, count, w, phi, ba, bb);
  }
  zero_slice(zero, zero_ints);   // histograms that the score and selection kernels add into
  __syncthreads();
  double *out = shares + (long long)blockIdx.x * Share<M>::DOUBLES;
  for_lower_tiles<M>([&](int t, int a, int b) {
    out[t * 256 + threadIdx.x] = (ba[a * SP + b] + bb[a * SP + b]) + (ba[b * SP + a] + bb[b * SP + a]);
  });
}

// One workgroup (4 waves) per head, steps 2 to 4; step 1 from the shares (partials and zero are not used
// then: the share kernel has cleared it), or from the partials.
template <int M, bool SHARES>
__global__ __launch_bounds__(256, 2) void sketch_solve_kernel(
    const SegTable T, int tiles_per_wg, int parts, const float *__restrict__ partials,
    const double *__restrict__ shares, const float *__restrict__ phi, float ridge_rel,
    uint16_t *__restrict__ wt, int32_t *__restrict__ status, int *__restrict__ zero,
    long long zero_ints) {
  constexpr int SP = M + 1, TILES = Share<M>::TILES;
  // before the factorisation, the two halves of a share
  union Lds {
    SketchFactor<M> f;
    double halves[2][SHARES ? 1 : M * SP];
  };
  __shared__ __attribute__((aligned(16))) Lds lds;
  SketchFactor<M> &F = lds.f;

  const int lhead = blockIdx.x;
  const int tid = threadIdx.x;

  PhiRegs<M> ph;
  if constexpr (SHARES) ph.fetch(phi);

  // ---- 1. S = Phi^T G Phi ----
  double sum[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t) sum[t] = 0.0;
  const int nshares = parts * SHARE_BLOCKS;
  if constexpr (SHARES) {
    const double *in = shares + (long long)lhead * nshares * Share<M>::DOUBLES;
    ShareSum<M> ss;
    ss.fetch(in);
    ss.add(in, nshares, sum);
  } else {
    double *ba = lds.halves[0], *bb = lds.halves[1];
    int nsplit;
    const long long pb = partial_base(T, lhead, tiles_per_wg, nsplit);
#pragma unroll 1
    for (int s = 0; s < nshares; ++s) {
      const int r = s / SHARE_BLOCKS, w = s - r * SHARE_BLOCKS;
      int first, count;
      split_part(nsplit, parts, r, first, count);
      sketch_share<M>(partials + (pb + first) * GRAM_PARTIAL_FLOATS, count, w, phi, ba, bb);
      __syncthreads();
      for_lower_tiles<M>([&](int t, int a, int b) {
        sum[t] += (ba[a * SP + b] + bb[a * SP + b]) + (ba[b * SP + a] + bb[b * SP + a]);
      });
      __syncthreads();
    }
    ph.fetch(phi);
    zero_slice(zero, zero_ints);
  }
  uint16_t *wh = wt + (size_t)lhead * (W_TERMS * M * D);
  sketch_factor<M>(F, sum, ph, ridge_rel, [&](int tt, int row, int ch, uint16_t v) { wh[(tt * M + row) * D + ch] = v; },
                   [](auto) {});
  __syncthreads();
  if (tid == 0) {
    const Where w = locate_head(T, lhead);
    status[T.s[w.seg].ghead0 + w.head] = F.flag;
  }
}

// Many heads (solve_plan): one workgroup per head takes step 1 too, each of its waves half of the columns of two of the four
// column blocks J of G (0 and 3, or 1 and 2: five stored blocks either way).  A wave sums its blocks over the partials in
// registers, as in sketch_share, and goes on with all of a column block: T_J = sum over I of G_IJ^T Phi_I in one chain, and one
// Phi_J^T T_J for it, 192 products (k_s = 48) a wave where the shares, block by block, take 300, and nothing of S passes through
// memory.  Bound by the fp64 matrix cores (192 x 64 clocks, 5 us) and by the chain of pivots: 2048 heads of 500 tokens, k_s = 48,
// whole scores 293 -> 231 us, 256 heads of 2048 78.9 -> 69.8.
template <int M, int FIRST, int SECOND>
__device__ __forceinline__ void sketch_columns(const double (&g)[5][8], const float *PH, int half, f64x4 (&sacc)[M / 16][M / 16]) {
  constexpr int CT = M / 16, PP = SketchFactor<M>::PP;
  const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
#pragma unroll
  for (int at = 0; at < CT; ++at)
#pragma unroll
    for (int bt = 0; bt < CT; ++bt) sacc[at][bt] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    const int J = part ? SECOND : FIRST, b0 = part ? FIRST + 1 : 0;
    f64x4 tacc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) tacc[ct] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int I = 0; I <= J; ++I)
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const double a = I == J ? 0.5 * g[b0 + I][q] : g[b0 + I][q];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          tacc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(
              a, (double)PH[(32 * I + 16 * (q >> 2) + 4 * lq + (q & 3)) * PP + 16 * ct + l16], tacc[ct], 0, 0, 0);
      }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int at = 0; at < CT; ++at) {
        const double a = (double)PH[(32 * J + 16 * half + 4 * v + lq) * PP + 16 * at + l16];
#pragma unroll
        for (int bt = 0; bt < CT; ++bt)
          sacc[at][bt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, tacc[bt][v], sacc[at][bt], 0, 0, 0);
      }
  }
}

// (At M = 64 the accumulators of S take 128 registers, so one workgroup on a unit.)
template <int M, bool HALVES>
__global__ __launch_bounds__(256, M > 48 ? 1 : 2) void sketch_direct_kernel(
    const SegTable T, int tiles_per_wg, const float *__restrict__ partials, const float *__restrict__ phi, float ridge_rel,
    uint16_t *__restrict__ wt, int32_t *__restrict__ status, int *__restrict__ zero, long long zero_ints) {
  constexpr int CT = M / 16, SP = M + 1, PP = SketchFactor<M>::PP, FLIGHT = 2;      // partials, or both halves of one, at a time
  struct Sketch {
    double halves[2][M * SP];
    float PH[D * PP];
  };
  union Lds {
    SketchFactor<M> f;
    Sketch s;
  };
  __shared__ __attribute__((aligned(16))) Lds lds;
  const int lhead = blockIdx.x, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = wave & 1;
  const bool inner = wave >= 2;          // columns of blocks 1 and 2, the others of 0 and 3

  PhiRegs<M> ph;
  ph.fetch(phi);
  int tph = 0, nsplit;
  const long long t0 = head_tiles(T, lhead, tph);
  long long pb = partial_base(t0, tph, lhead, HALVES ? 2 * GRAM_HALF_RUN : tiles_per_wg, nsplit);
  int least = 0, most = nsplit - 1;
  if constexpr (HALVES) {
    const HalfRuns hr(t0, tph, lhead, pb, 0);
    pb = hr.slot;
    least = hr.least;
    most = hr.most;
  }
  const float *p = partials + pb * GRAM_PARTIAL_FLOATS + (32 * lq + 16 * half + l16) * 4;
  double g[5][8];
#pragma unroll
  for (int b = 0; b < 5; ++b)
#pragma unroll
    for (int q = 0; q < 8; ++q) g[b][q] = 0.0;
  for (int sp = 0; sp <= most; sp += FLIGHT) {
    float4 a[FLIGHT][5], c[FLIGHT][5];
#pragma unroll
    for (int u = 0; u < FLIGHT; ++u) {
      const float *pu = p + (long long)min(HALVES ? max(sp + u, least) : sp + u, most) * GRAM_PARTIAL_FLOATS;
#pragma unroll
      for (int b = 0; b < 5; ++b) {      // stored blocks (0,0) (0,3) (1,3) (2,3) (3,3), or (0,1) (1,1) (0,2) (1,2) (2,2)
        constexpr int outer_at[5] = {0, 3, 6, 8, 9}, inner_at[5] = {1, 4, 2, 5, 7};
        const float *pb4 = pu + 1024 * (inner ? inner_at[b] : outer_at[b]);
        a[u][b] = *reinterpret_cast<const float4 *>(pb4);
        c[u][b] = *reinterpret_cast<const float4 *>(pb4 + 512);
      }
    }
    if constexpr (HALVES) {
      if (sp >= least && sp < most) {    // uniform: both are the head's, else they are the same
#pragma unroll
        for (int b = 0; b < 5; ++b) {
          a[0][b] = make_float4(a[0][b].x + a[1][b].x, a[0][b].y + a[1][b].y, a[0][b].z + a[1][b].z, a[0][b].w + a[1][b].w);
          c[0][b] = make_float4(c[0][b].x + c[1][b].x, c[0][b].y + c[1][b].y, c[0][b].z + c[1][b].z, c[0][b].w + c[1][b].w);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < (HALVES ? 1 : FLIGHT); ++u)
      if (sp + u <= most) {              // uniform
#pragma unroll
        for (int b = 0; b < 5; ++b) {
          g[b][0] += a[u][b].x; g[b][1] += a[u][b].y; g[b][2] += a[u][b].z; g[b][3] += a[u][b].w;
          g[b][4] += c[u][b].x; g[b][5] += c[u][b].y; g[b][6] += c[u][b].z; g[b][7] += c[u][b].w;
        }
      }
  }
#pragma unroll
  for (int i = 0; i < PhiRegs<M>::N; ++i) {
    const int c4 = tid + 256 * i;
    *reinterpret_cast<typename PhiRegs<M>::quad *>(&lds.s.PH[c4 / (M / 4) * PP + c4 % (M / 4) * 4]) = ph.v[i];
  }
  __syncthreads();
  f64x4 sacc[CT][CT];
  if (inner) sketch_columns<M, 1, 2>(g, lds.s.PH, half, sacc);
  else sketch_columns<M, 0, 3>(g, lds.s.PH, half, sacc);
  zero_slice(zero, zero_ints);   // histograms that the score and selection kernels add into
  double *dst = lds.s.halves[half];
  auto each = [&](auto &&f) {
#pragma unroll
    for (int at = 0; at < CT; ++at)
#pragma unroll
      for (int bt = 0; bt < CT; ++bt)
#pragma unroll
        for (int v = 0; v < 4; ++v) f(dst[(16 * at + 4 * v + lq) * SP + 16 * bt + l16], sacc[at][bt][v]);
  };
  if (inner) each([](double &d, double x) { d = x; });
  __syncthreads();
  if (!inner) each([](double &d, double x) { d += x; });
  __syncthreads();
  double sum[Share<M>::TILES];
  {
    const double *ba = lds.s.halves[0], *bb = lds.s.halves[1];
    for_lower_tiles<M>([&](int t, int i, int j) {
      sum[t] = (ba[i * SP + j] + bb[i * SP + j]) + (ba[j * SP + i] + bb[j * SP + i]);
    });
  }
  __syncthreads();
  uint16_t *wh = wt + (size_t)lhead * (W_TERMS * M * D);
  sketch_factor<M>(lds.f, sum, ph, ridge_rel, [&](int tt, int row, int ch, uint16_t v) { wh[(tt * M + row) * D + ch] = v; },
                   [](auto) {});
  __syncthreads();
  if (tid == 0) {
    const Where w = locate_head(T, lhead);
    status[T.s[w.seg].ghead0 + w.head] = lds.f.flag;
  }
}

// ---- exact mode: partial Gram blocks -> G + rho I -> L -> L^{-1} = W^T --------------------------
// The same blocked factorisation on the full 128 x 128 Gram matrix (8 panels of 16).  Like S in
// sketched mode, G is summed by workgroups of their own (gram_sum_kernel, one per stored block)
// where the workspace has room, with the same bits.
constexpr int EXACT_THREADS = 512;

__global__ __launch_bounds__(256) void gram_sum_kernel(const SegTable T, int tiles_per_wg,
                                                       const float *__restrict__ partials,
                                                       double *__restrict__ sums, int *__restrict__ zero,
                                                       long long zero_ints) {
  const int lhead = blockIdx.x / 10, b = blockIdx.x - 10 * lhead;
  int nsplit;
  const long long pb = partial_base(T, lhead, tiles_per_wg, nsplit);
  double g[4];
  sum_quads<1>(partials + pb * GRAM_PARTIAL_FLOATS + b * 1024 + threadIdx.x * 4, nsplit, g);
  zero_slice(zero, zero_ints);   // histograms that the score and selection kernels add into
  double *out = sums + (long long)blockIdx.x * 1024 + threadIdx.x * 4;
#pragma unroll
  for (int c = 0; c < 4; ++c) out[c] = g[c];
}

template <bool SUMS>
__global__ __launch_bounds__(EXACT_THREADS) void exact_solve_kernel(
    const SegTable T, int tiles_per_wg, const float *__restrict__ partials,
    const double *__restrict__ sums, float ridge_rel, uint16_t *__restrict__ wt,
    int32_t *__restrict__ status, int *__restrict__ zero, long long zero_ints) {
  constexpr int M = D, P = M / 16, SP = factor_pitch(M), NW = EXACT_THREADS / 64;
  __shared__ __attribute__((aligned(16))) double Ss[M * SP];        // G, then L and X = L^{-1} (factor_panels)
  __shared__ __attribute__((aligned(16))) double Xd[P][16][XD_PITCH];
  __shared__ double d0_s[M];
  __shared__ int flag_s;

  const int lhead = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid == 0) flag_s = 0;

  // ---- 1. G: the head's 10 upper blocks, five for each half of the workgroup ----
  const int f = tid & 255, half = __builtin_amdgcn_readfirstlane(tid >> 8);
  int row0, col;
  partial_quad(f, row0, col);     // this thread's float4 of a block: rows row0..+3 of column col
  double g[5][4];
  if constexpr (SUMS) {
    const double *in = sums + ((long long)lhead * 10 + half) * 1024 + f * 4;
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) g[i][c] = in[i * 2048 + c];
  } else {
    int nsplit;
    const long long pb = partial_base(T, lhead, tiles_per_wg, nsplit);
    const float *src = partials + pb * GRAM_PARTIAL_FLOATS + half * 1024 + f * 4;
#pragma unroll
    for (int i = 0; i < 5; ++i) sum_quads<1, 2>(src + i * 2048, nsplit, g[i]);      // heads of a partial or two
    zero_slice(zero, zero_ints);   // histograms that the score and selection kernels add into
  }
  // into the lower triangle: block (I, J), I < J, holds G[32I + r][32J + c] = G[32J + c][32I + r]
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    int I, J;
    upper_block_pos(2 * i + half, I, J);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (I == J) Ss[(32 * I + row0 + c) * SP + 32 * J + col] = g[i][c];
      else        Ss[(32 * J + col) * SP + 32 * I + row0 + c] = g[i][c];
    }
  }
  __syncthreads();

  // ridge: rho = ridge_rel * trace(G) / M (every wave sums in the same order)
  double tr = Ss[lane * SP + lane] + Ss[(lane + 64) * SP + lane + 64];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) tr += __shfl_xor(tr, d);
  const double rho = (double)ridge_rel * tr / (double)M;
  __syncthreads();
  if (tid < M) {
    const double v = Ss[tid * SP + tid] + rho;
    Ss[tid * SP + tid] = v;
    d0_s[tid] = v;
  }
  __syncthreads();

  // ---- 2 and 3, W^T = X split into bf16 planes row by row.  The score kernel reads of row j the
  // channels of its group of 32 and of the groups before it. ----
  uint16_t *wh = wt + (size_t)lhead * (W_TERMS * M * D);
  factor_panels<P, NW, true>(Ss, Xd, d0_s, &flag_s, [&](int p, int i, int nw) {
    // a wave: 16 rows x 32 channels, a lane 8 consecutive channels of one row
    const int r = lane & 15, c8 = 8 * (lane >> 4);
    for (int g32 = i; g32 <= p >> 1; g32 += nw) {
      const int ch0 = 32 * g32 + c8, cb = ch0 >> 4;
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        double v = 0.0;
        if (cb == p) v = Xd[p][r][(ch0 & 15) + e];
        else if (cb < p) v = Ss[(ch0 + e) * SP + 16 * p + r];
        x[e] = (float)v;
      }
#pragma unroll
      for (int t = 0; t < W_TERMS; ++t) {
        unsigned w[4];
#pragma unroll
        for (int e = 0; e < 8; e += 2) w[e >> 1] = split_bf16(x[e], x[e + 1]);
        *reinterpret_cast<uint4 *>(&wh[(t * M + 16 * p + r) * D + ch0]) = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
  });
  if (tid == 0) {
    const Where w = locate_head(T, lhead);
    status[T.s[w.seg].ghead0 + w.head] = flag_s;
  }
}

// Longest run of partials a share of its own takes before the head's partials are cut into parts:
// two batches of four are in flight at a time, about 1 us each.
// (Where partials may come in halves, half as many: the halves are what is loaded.)
constexpr int SHARE_SPLITS = 64, SHARE_PARTS_MAX = 8;

// Above DIRECT_HEADS heads sketch_direct_kernel forms and factors S, unless some head may have more partials than direct_most: its one
// workgroup adds them two by two, about 0.6 us each, where shares are added side by side but cost a launch, more products and, for
// 48 and 64 rows, the matrix cores' time, which grows with the number of heads.  (Above a head a unit the shares of a head are formed
// one after the other: 384 heads, 16 of them of 6000 tokens, k_s = 16, 13 partials, 67.5 / 71.5; k_s = 32, 17 partials, 224 / 225.)
// Up to 128 heads the score workgroups factor short heads themselves (128 x 2048, k_s = 16, 40.2 with shares / 41.6 direct; 48 53.9 /
// 54.0).  Scores alone on MI355X, us with shares / direct, 192 heads, 8 of them longer, partials of those in brackets:
//   k_s = 16  (3) 87.1/83.5  (6) 71.9/71.4  (8) 92.3/93.4   (13) 61.2/64.0  (19) 60.9/72.3  (28) 64.4/84.4
//   k_s = 32  (4) 93.3/89.9  (12) 81.9/81.6 (13) 63.1/62.9  (14) 68.8/69.6  (18) 72.4/74.6  (28) 70.0/76.1
//   k_s = 48  (6) 86.2/80.6  (14) 87.9/85.2 (18) 92.0/90.7  (19) 73.0/72.7  (23) 86.9/87.8  (28) 78.5/81.3
//   k_s = 64  (6) 101/91.0   (14) 103/95.1  (18) 107/99.9   (28) 92.4/89.8  (32) 102/101
// 256 heads, k_s = 16 (6) 67.1/67.4, (7) 69.6/71.8, (13) 54.0/60.9; k_s = 48 (17) 116/107.
// Where shares lead to score workgroups that factor their heads (score_solves) they save a launch more: 136 to 256 heads of 64 to
// 4000 tokens (2 or 3) k_s = 16 -2 to +5 us, k_s = 32 0 to +4.5, 48 +1 to +9, 64 +5 to +18; 192 heads, 8 of them longer, k_s = 16
// (5) 59.6/62.7, (8) 59.3/67.2; k_s = 32 (5) 59.9/66.3; k_s = 48 (5) 67.5/71.9, (7) 62.7/65.0; k_s = 64 (8) 85.3/84.2, (10) 85.6/84.3,
// (12) 78.7/79.2.
static long long direct_most(int ks, int heads, int cus, bool in_score) {
  if (heads <= DIRECT_HEADS) return 0;
  if (heads > cus) return ks - 4;
  if (in_score) return ks == 16 ? 2 : ks <= 48 ? 3 : 11;
  return ks == 16 ? 6 : ks == 32 ? 13 : ks == 48 ? 20 : 36;
}

// most: partials that a head may have; splits: of a part; direct_up_to: see direct_most.
static SolvePlan plan_of(const SegTable &T, int ks, long long most, int splits, long long direct_up_to) {
  SolvePlan p;
  p.parts = 1;
  p.nshares = 0;
  p.direct = false;
  if (ks == 0) {
    p.share_bytes = (size_t)T.nheads * 10 * 1024 * sizeof(double);
    return p;
  }
  p.direct = most <= direct_up_to;
  const long long parts = (most + splits - 1) / splits;
  p.parts = parts > SHARE_PARTS_MAX ? SHARE_PARTS_MAX : (int)parts;
  const int P = ks / 16;
  p.nshares = p.parts * SHARE_BLOCKS;
  p.share_bytes = (size_t)T.nheads * p.nshares * (P * (P + 1) / 2 * 256) * sizeof(double);
  return p;
}

static int longest_head(const SegTable &T) {
  int tiles = 0;
  for (int i = 0; i < T.nseg; ++i)
    if (tiles_of(T.s[i].n) > tiles) tiles = tiles_of(T.s[i].n);
  return tiles;
}

SolvePlan solve_plan(const SegTable &T, int ks, int tiles_per_wg, bool halves, bool in_score, int cus) {
  return plan_of(T, ks, (longest_head(T) + tiles_per_wg - 1) / tiles_per_wg + 1, halves ? SHARE_SPLITS / 2 : SHARE_SPLITS,
                 direct_most(ks, T.nheads, cus, in_score));
}

size_t share_bytes_most(const SegTable &T, int ks, int least_run, long long most_wgs, bool halves, int cus) {
  const long long longest = longest_head(T), total = total_tiles(T);
  const long long by_run = (longest + least_run - 1) / least_run, by_wgs = (most_wgs * longest + total - 1) / total;
  const long long always = std::min(direct_most(ks, T.nheads, cus, false), direct_most(ks, T.nheads, cus, true));
  if (ks > 0 && by_run + 1 <= always) return 0;            // whatever the proportions
  return plan_of(T, ks, std::min(by_run, by_wgs) + 1, halves ? SHARE_SPLITS / 2 : SHARE_SPLITS, 0).share_bytes;
}

template <int M>
static hipError_t launch_sketched(const SegTable &T, int tiles_per_wg, const SolvePlan &plan,
                                  const float *partials, bool halves, double *shares, const float *phi,
                                  float ridge_rel, uint16_t *wt, int32_t *status, int *zero,
                                  long long zero_ints, hipStream_t st) {
  if (plan.direct) {
    hipLaunchKernelGGL((halves ? sketch_direct_kernel<M, true> : sketch_direct_kernel<M, false>), dim3((unsigned)T.nheads), dim3(256), 0, st, T, tiles_per_wg, partials, phi,
                       ridge_rel, wt, status, zero, zero_ints);
  } else if (shares != nullptr) {
    hipLaunchKernelGGL((halves ? sketch_share_kernel<M, true> : sketch_share_kernel<M, false>), dim3((unsigned)(T.nheads * plan.parts * SHARE_BLOCKS)),
                       dim3(256), 0, st, T, tiles_per_wg, plan.parts, partials, phi, shares,
                       wt == nullptr ? status : nullptr, zero, zero_ints);
    if (wt == nullptr) return hipGetLastError();
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL((sketch_solve_kernel<M, true>), dim3((unsigned)T.nheads), dim3(256), 0, st, T,
                       tiles_per_wg, plan.parts, nullptr, shares, phi, ridge_rel, wt, status, nullptr, 0);
  } else {
    hipLaunchKernelGGL((sketch_solve_kernel<M, false>), dim3((unsigned)T.nheads), dim3(256), 0, st, T,
                       tiles_per_wg, plan.parts, partials, shares, phi, ridge_rel, wt, status, zero, zero_ints);
  }
  return hipGetLastError();
}

// Sketched mode: partial Gram blocks -> W^T (see above); wt null: the shares only.
hipError_t launch_sketch_solve(const SegTable &T, int ks, int tiles_per_wg, const SolvePlan &plan,
                               const float *partials, bool halves, double *shares, const float *phi,
                               float ridge_rel, uint16_t *wt, int32_t *status, int *zero,
                               long long zero_ints, hipStream_t st) {
  if (T.nheads <= 0) return hipSuccess;
  if ((shares == nullptr || plan.direct) && wt == nullptr) return hipErrorInvalidValue;
  if (halves && shares == nullptr && !plan.direct) return hipErrorInvalidValue;
  switch (ks) {
    case 16: return launch_sketched<16>(T, tiles_per_wg, plan, partials, halves, shares, phi, ridge_rel, wt, status, zero, zero_ints, st);
    case 32: return launch_sketched<32>(T, tiles_per_wg, plan, partials, halves, shares, phi, ridge_rel, wt, status, zero, zero_ints, st);
    case 48: return launch_sketched<48>(T, tiles_per_wg, plan, partials, halves, shares, phi, ridge_rel, wt, status, zero, zero_ints, st);
    case 64: return launch_sketched<64>(T, tiles_per_wg, plan, partials, halves, shares, phi, ridge_rel, wt, status, zero, zero_ints, st);
    default: return hipErrorInvalidValue;
  }
}

// Subsampled randomized Hadamard sketch (paper App. D) as a dense Phi: the sign bits and the
// chosen rows of H travel as kernel arguments.
struct SrhtSpec {
  uint32_t sign_bits[D / 32];
  uint8_t cols[64];
};
__global__ __launch_bounds__(256) void srht_phi_kernel(SrhtSpec spec, int ks, float value,
                                                       float *__restrict__ phi) {
  for (int idx = threadIdx.x + blockIdx.x * 256; idx < D * ks; idx += 256 * gridDim.x) {
    const int i = idx / ks, j = idx - i * ks;
    const unsigned neg = ((spec.sign_bits[i >> 5] >> (i & 31)) & 1u) ^
                         (__popc((unsigned)i & (unsigned)spec.cols[j]) & 1u);
    phi[idx] = neg ? -value : value;
  }
}

hipError_t launch_srht_phi(int ks, const uint8_t *signs, const int32_t *cols, float *phi,
                           hipStream_t st) {
  SrhtSpec spec;
  for (int w = 0; w < D / 32; ++w) spec.sign_bits[w] = 0;
  for (int i = 0; i < D; ++i)
    if (signs[i]) spec.sign_bits[i >> 5] |= 1u << (i & 31);
  for (int j = 0; j < 64; ++j) spec.cols[j] = j < ks ? (uint8_t)cols[j] : 0;
  hipLaunchKernelGGL(srht_phi_kernel, dim3(8), dim3(256), 0, st, spec, ks,
                     sqrtf((float)D / (float)ks), phi);
  return hipGetLastError();
}

// Exact mode: partial Gram blocks -> Cholesky of G + rho I -> W^T = L^{-1}.
hipError_t launch_exact_solve(const SegTable &T, int tiles_per_wg, const float *partials,
                              double *shares, float ridge_rel, uint16_t *wt, int32_t *status,
                              int *zero, long long zero_ints, hipStream_t st) {
  if (T.nheads <= 0) return hipSuccess;
  if (shares != nullptr) {
    hipLaunchKernelGGL(gram_sum_kernel, dim3((unsigned)T.nheads * 10), dim3(256), 0, st, T, tiles_per_wg,
                       partials, shares, zero, zero_ints);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL((exact_solve_kernel<true>), dim3((unsigned)T.nheads), dim3(EXACT_THREADS), 0, st, T,
                       tiles_per_wg, nullptr, shares, ridge_rel, wt, status, nullptr, 0);
  } else {
    hipLaunchKernelGGL((exact_solve_kernel<false>), dim3((unsigned)T.nheads), dim3(EXACT_THREADS), 0, st, T,
                       tiles_per_wg, partials, shares, ridge_rel, wt, status, zero, zero_ints);
  }
  return hipGetLastError();
}

}  // namespace cmp
