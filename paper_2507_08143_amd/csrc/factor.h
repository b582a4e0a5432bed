// The factorisation of S = Phi^T G Phi + rho I, from the shares of S to the bf16 planes of W^T = L^{-1} Phi^T: for a
// kernel of its own (solve.hip) and for score workgroups that factor their head themselves (score.hip).
#pragma once

#include <type_traits>

#include "common.h"

namespace cmp {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Two floats as bf16, round to nearest even, the first in the lower half; split_bf16 also leaves what that misses of them.
__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{x, y}), bf16x2));
}
__device__ __forceinline__ unsigned split_bf16(float &x, float &y) {
  const unsigned p = pack_bf16(x, y);
  x -= __uint_as_float(p << 16);
  y -= __uint_as_float(p & 0xffff0000u);
  return p;
}

// A pivot below this fraction of its own (ridged) diagonal entry is below what the fp32-
// accumulated Gram matrix resolves: the direction is dropped and the head flagged.
constexpr double PIVOT_REL = 1.4901161193847656e-08;   // 2^-26

// All lanes of a wave's 16-lane row get the value of lane K of that row.
template <int K>
__device__ __forceinline__ double bcast16(double x) {
  constexpr int ROW_NEWBCAST = 0x150;
  return __builtin_amdgcn_mov_dpp(x, ROW_NEWBCAST + K, 0xf, 0xf, true);
}

// Compile-time loop: f(integral_constant<int, B>) ... f(integral_constant<int, E - 1>).
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Stops the compiler from moving the computation of x past this point.
__device__ __forceinline__ void computed_here(double &x) { asm volatile("" : "+v"(x)); }

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// acc -= (a of lane K of the row) * b in one instruction.  The compiler does not see that the asm reads a across lanes: two
// instructions have to lie between what writes a and the first of these (chol16_inverse: the update of the next column and
// its reciprocal; tests/test_device_code.py looks at what is made of it).
template <int K>
__device__ __forceinline__ void sub_bcast16(double &acc, double a, double b) {
  asm volatile("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(a), "v"(b), "n"(K));
}

// Inverse of the Cholesky factor of a 16 x 16 diagonal block, by one wave.  Lane i of every
// 16-lane row holds row i of the block (row[], the lanes above 15 repeat what lanes 0..15 do) and
// the ridged diagonal entry d0 of its row; on return x[i] of lane j is X[i][j], X = L^{-1}.  A
// pivot that is not above PIVOT_REL d0 is dropped (row and column of X zero, or NaN where the block
// is not finite: such a head's scores have to come out as NaN); returns whether none was.
// Bound: one wave's instructions, one after the other.  The elimination is the square-root free one (u_i the
// column before scaling, t_i = u_i / d): what the next pivot waits for is a reciprocal (2^-24, then a cubic step), its
// broadcast, a product and an fma, eight clocks each and the reciprocal 20; an update is four clocks with the broadcast
// of t_j inside it, and those that the previous pivot still owes the columns behind this one stand between the links of
// the chain.  The square roots of all 16 pivots are taken at once at the end.  Nothing passes through LDS or scalar
// registers.  The inverse takes the same broadcasts in the same pass (lane j solves column j).
__device__ __forceinline__ bool chol16_inverse(double (&row)[16], double d0, double (&x)[16]) {
  const int l16 = threadIdx.x & 15;
  double d_mine = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = (i == l16) ? 1.0 : 0.0;
  double u_prev = 0.0, t_prev = 0.0;               // column k - 1
  const double least = PIVOT_REL * d0;
  static_for<0, 16>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    // what pivot k - 1 still owes: to x[k], then to row[j] and x[j] of the columns j behind this one
    constexpr int OWED = k > 0 ? 1 + 2 * (15 - k) : 0;
    auto owed = [&](auto from, auto to) {
      static_for<decltype(from)::value, decltype(to)::value>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = i == 0 ? k : k + 1 + (i - 1) / 2;
        if constexpr (i > 0 && (i & 1)) sub_bcast16<j>(row[j], t_prev, u_prev);
        else sub_bcast16<j>(x[j], t_prev, x[k > 0 ? k - 1 : 0]);
      });
      __builtin_amdgcn_sched_barrier(0);
    };
    // the last seven between the links, the others behind the reciprocal
    constexpr int C0 = OWED > 7 ? OWED - 7 : 0;
    auto cut = [](auto sc) {
      constexpr int c = C0 + decltype(sc)::value;
      return std::integral_constant<int, c < OWED ? c : OWED>{};
    };
    const double u = row[k];                       // of lane k: the pivot
    double r = __builtin_amdgcn_rcp(u);
    computed_here(r);
    __builtin_amdgcn_sched_barrier(0);
    owed(std::integral_constant<int, 0>{}, cut(std::integral_constant<int, 0>{}));
    double u_next = 0.0;
    if constexpr (k < 15) u_next = bcast16<k + 1>(u);
    if (l16 == k) d_mine = u;
    r = u > least ? r : 0.0;                       // false for NaN too
    computed_here(r);
    computed_here(u_next);
    __builtin_amdgcn_sched_barrier(0);
    owed(cut(std::integral_constant<int, 0>{}), cut(std::integral_constant<int, 1>{}));
    double e = fma(-u, r, 1.0);
    computed_here(e);
    owed(cut(std::integral_constant<int, 1>{}), cut(std::integral_constant<int, 2>{}));
    e = fma(e, e, e);
    computed_here(e);
    owed(cut(std::integral_constant<int, 2>{}), cut(std::integral_constant<int, 3>{}));
    r = fma(r, e, r);
    computed_here(r);
    owed(cut(std::integral_constant<int, 3>{}), cut(std::integral_constant<int, 5>{}));
    r = bcast16<k>(r);
    computed_here(r);
    owed(cut(std::integral_constant<int, 5>{}), cut(std::integral_constant<int, 6>{}));
    double t = u * r;                              // lane i: L[i][k] / L[k][k] for i > k
    computed_here(t);
    owed(cut(std::integral_constant<int, 6>{}), std::integral_constant<int, OWED>{});
    u_prev = u;
    t_prev = t;
    if constexpr (k < 15) row[k + 1] = fma(-u_next, t, row[k + 1]);
  });
  const bool ok = d_mine > least && d_mine < 1.0e300;
  const double rs = ok ? rsqrt(d_mine) : 0.0;
  static_for<0, 16>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    x[i] *= bcast16<i>(rs);
  });
  return __all(ok);
}

// Doubles from a row of the factored matrix, and of a diagonal block of X, to the next.  With 2 modulo 16 the 16 rows that a
// product's operands are read from begin four banks apart, so that neither 8- nor 16-byte reads of them collide (a pitch
// of 1 modulo 16 does, twofold).
constexpr int factor_pitch(int m) { return m + 2; }
constexpr int XD_PITCH = factor_pitch(16);
// Four consecutive doubles of a row, 16-byte aligned: a lane's part of an operand of a 16 x 16 x 16 product, of which step
// ks takes element ks in all lanes (so that lane group lq contributes k = 4 lq + ks).
struct Quad { double v[4]; };
__device__ __forceinline__ Quad quad_at(const double *p) {
  const double2 a = *reinterpret_cast<const double2 *>(p), b = *reinterpret_cast<const double2 *>(p + 2);
  return Quad{{a.x, a.y, b.x, b.y}};
}

// Steps 2 and 3 for a matrix of P panels, by NW waves.  Ss (16P rows of factor_pitch(16P) doubles) holds
// S + rho I in its lower 16 x 16 blocks; on return L is below the diagonal blocks, the diagonal
// blocks of X = L^{-1} are in Xd and the blocks of X below the diagonal, transposed, in the upper
// blocks of Ss (element X[j][c], block of j below block of c, is at Ss[c][j]).
// The serial chain is wave 0's: the diagonal block takes its last update and is eliminated.  In
// its shadow the other waves apply what the previous panel owes the trailing matrix and X (Y_qc =
// sum over r of L_qr X_rc grows in the place of X_qc) and hand on finished rows of X: row_done(p,
// i, n) is called by n waves, i = 0 .. n - 1, when block row p of X is complete.  In eight panels
// (exact mode) the work in the shadow is 22 of 52 us when it is not there (on the slower pivots of an earlier chol16_inverse).
// !INVERSE: X is not wanted, only L and the diagonal blocks of X; waves 1 .. NW - 1 call row_done(p) (a compile-time
// p) when X_pp and the blocks of L below it are complete.
template <int P, int NW, bool INVERSE, class F>
__device__ __forceinline__ void factor_panels(double *Ss, double (*Xd)[16][XD_PITCH], const double *d0_s,
                                              int *flag, F &&row_done) {
  constexpr int SP = factor_pitch(16 * P);
  const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // A_qr -= L_qp L_rp^T
  auto trail = [&](int q, int r, int p) {
    const Quad a = quad_at(&Ss[(16 * q + l16) * SP + 16 * p + 4 * lq]);
    const Quad b = quad_at(&Ss[(16 * r + l16) * SP + 16 * p + 4 * lq]);
    f64x4 acc;
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = Ss[(16 * q + 4 * v + lq) * SP + 16 * r + l16];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.v[ks], b.v[ks], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) Ss[(16 * q + 4 * v + lq) * SP + 16 * r + l16] = acc[v];
  };
  // Y_qc += L_qp X_pc, c <= p
  auto grow = [&](int q, int c, int p) {
    double *y = &Ss[(16 * c + l16) * SP + 16 * q + lq];        // transposed: row 4v + lq, column l16
    const Quad a = quad_at(&Ss[(16 * q + l16) * SP + 16 * p + 4 * lq]);
    Quad b;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    if (c < p) {
      b = quad_at(&Ss[(16 * c + l16) * SP + 16 * p + 4 * lq]);
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = y[4 * v];
    } else {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) b.v[ks] = Xd[p][4 * lq + ks][l16];
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a.v[ks], b.v[ks], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) y[4 * v] = acc[v];
  };
  // wave 0: the diagonal block
  auto pivots = [&](int p) {
    if (p > 0) {
      trail(p, p, p - 1);
      wave_fence();
    }
    double row[16], x[16];
#pragma unroll
    for (int j = 0; j < 16; j += 4) {
      const Quad r = quad_at(&Ss[(16 * p + l16) * SP + 16 * p + j]);
#pragma unroll
      for (int e = 0; e < 4; ++e) row[j + e] = r.v[e];
    }
    if (!chol16_inverse(row, d0_s[16 * p + l16], x) && lane == 0) *flag = COMPACTOR_STATUS_PIVOT;
    if (lane < 16) {
#pragma unroll
      for (int i = 0; i < 16; ++i) Xd[p][i][lane] = x[i];
    }
  };
  // The others meanwhile: what panel p - 1 owes, without block (p, p): of every row q >= p the blocks c < p of Y and c >= p of
  // A, dealt out in turn.
  auto owed = [&](int p) {
    if constexpr (INVERSE) {
      const int row0 = p * (p + 1) / 2;                        // blocks of the rows before
      int q = p;
      for (int i = wave - 1; i < P * (P + 1) / 2 - row0 - 1; i += NW - 1) {
        const int g = row0 + i + (i >= p);
        while (g >= (q + 1) * (q + 2) / 2) ++q;
        const int c = g - q * (q + 1) / 2;
        if (c < p) grow(q, c, p - 1);
        else trail(q, c, p - 1);
      }
    } else {
      int t = 1;
      for (int q = p; q < P; ++q)
        for (int r = p; r <= q; ++r) {
          if (r == p && q == p) continue;
          if (t == wave) trail(q, r, p - 1);
          t = t == NW - 1 ? 1 : t + 1;
        }
    }
  };
  // all: the panel below the diagonal block, L_qp = A_qp X_pp^T, and row p of X, X_pc = -X_pp Y_pc
  auto panel = [&](int p) {
    __syncthreads();
    for (int i = wave; i < P; i += NW) {
      if (i == p || (!INVERSE && i < p)) continue;
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      if (i > p) {
        double *l = &Ss[(16 * i) * SP + 16 * p];
        const Quad a = quad_at(l + l16 * SP + 4 * lq), b = quad_at(&Xd[p][l16][4 * lq]);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a.v[ks], b.v[ks], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) l[(4 * v + lq) * SP + l16] = acc[v];
      } else {
        double *y = &Ss[(16 * i + l16) * SP + 16 * p + lq];
        const Quad a = quad_at(&Xd[p][l16][4 * lq]), b = quad_at(&Ss[(16 * i + l16) * SP + 16 * p + 4 * lq]);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.v[ks], b.v[ks], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) y[4 * v] = acc[v];
      }
    }
    __syncthreads();
  };
  // Every wave passes the same barriers, wave 0 in code of its own: registers that row_done keeps from row to row are
  // not held through the pivots.
  if constexpr (INVERSE) {
#pragma unroll 1
    for (int p = 0; p < P; ++p) {
      if (wave == 0) {
        pivots(p);
      } else if (p > 0) {
        owed(p);
        row_done(p - 1, wave - 1, NW - 1);
      }
      panel(p);
    }
    row_done(P - 1, wave, NW);
  } else {
    // Wave 0 first, and not as two sides of one condition: the compiler would join them before wave 0's side, which would
    // then wait for everything that the other waves have requested by their end and, with it, for all loads of its own.
    if (wave == 0) {
#pragma unroll 1
      for (int p = 0; p < P; ++p) {
        pivots(p);
        panel(p);
      }
    }
    int other = wave;
    asm volatile("" : "+s"(other));
    if (other != 0) {
      static_for<0, P>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        if constexpr (p > 0) {
          owed(p);
          row_done(std::integral_constant<int, p - 1>{});
        }
        panel(p);
      });
      row_done(std::integral_constant<int, P - 1>{});
    }
  }
}

constexpr int SHARE_BLOCKS = 5;
template <int M>
struct Share {
  static constexpr int P = M / 16, TILES = P * (P + 1) / 2;     // lower 16 x 16 tiles of S
  static constexpr int DOUBLES = TILES * 256;                   // thread e of tile t: t * 256 + e
};

// f(t, row, column) for the lower tiles t of S, with the element of each that this thread has.
template <int M, class F>
__device__ __forceinline__ void for_lower_tiles(F &&f) {
  const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
  int t = 0;
#pragma unroll
  for (int a = 0; a < M / 16; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b, ++t) f(t, 16 * a + r, 16 * b + c);
}

// Phi on its way to LDS, in registers of a workgroup of 256.
template <int M>
struct PhiRegs {
  static constexpr int N = D * M / 4 / 256;
  typedef float quad __attribute__((ext_vector_type(4)));
  quad v[N];
  __device__ __forceinline__ void fetch(const float *__restrict__ phi) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = reinterpret_cast<const quad *>(phi)[threadIdx.x + 256 * i];
  }
};

// The lower tiles of S from the shares of a head, added in their order, SHARE_BLOCKS at a time: fetch() requests the
// first ones, add() adds them and all others; sum[t] is this thread's element of tile t.
template <int M>
struct ShareSum {
  static constexpr int TILES = Share<M>::TILES;
  double v[SHARE_BLOCKS][TILES];
  __device__ __forceinline__ void fetch(const double *__restrict__ shares) {
#pragma unroll
    for (int u = 0; u < SHARE_BLOCKS; ++u)
#pragma unroll
      for (int t = 0; t < TILES; ++t) v[u][t] = shares[u * Share<M>::DOUBLES + t * 256 + threadIdx.x];
  }
  __device__ __forceinline__ void add(const double *__restrict__ shares, int nshares, double (&sum)[TILES]) const {
#pragma unroll
    for (int t = 0; t < TILES; ++t) sum[t] = 0.0;
#pragma unroll
    for (int u = 0; u < SHARE_BLOCKS; ++u)
#pragma unroll
      for (int t = 0; t < TILES; ++t) sum[t] += v[u][t];
#pragma unroll 1
    for (int s0 = SHARE_BLOCKS; s0 < nshares; s0 += SHARE_BLOCKS) {
      double x[SHARE_BLOCKS][TILES];
#pragma unroll
      for (int u = 0; u < SHARE_BLOCKS; ++u)
#pragma unroll
        for (int t = 0; t < TILES; ++t) x[u][t] = shares[(long long)(s0 + u) * Share<M>::DOUBLES + t * 256 + threadIdx.x];
#pragma unroll
      for (int u = 0; u < SHARE_BLOCKS; ++u)
#pragma unroll
        for (int t = 0; t < TILES; ++t) sum[t] += x[u][t];
    }
  }
};

// Scratch of sketch_factor in LDS.
template <int M>
struct SketchFactor {
  alignas(16) double Ss[M * factor_pitch(M)];      // S, then L (factor_panels)
  alignas(16) double Xd[M / 16][16][XD_PITCH];
  double d0[M];
  static constexpr int PP = M + 4;                 // pitch of Phi: conflict-free reads
  float PH[D * PP];
  int flag;
};

// One workgroup of 256: steps 2 to 4 (see solve.hip) from S in lower tiles and Phi.  store(plane, row, channel, bf16)
// gets the planes of W^T; F.flag is the status, complete for all threads after a barrier.  shadow(j), j = 0 .. M / 16 - 1, is
// called by waves 1 to 3 before they wait for the pivots of panel j.
// W^T = L^{-1} Phi^T by forward substitution, row blocks of 16: W_p = X_pp R_p with R_q = Phi_q^T - sum over r < q of
// L_qr W_r, which wants no more of L^{-1} than its diagonal blocks X_pp.  Waves 1 to 3 do it in the shadow of the next
// panel's pivots, each for its channels: a product's accumulators are the next one's operand as they are, so that
// nothing of R or W passes through LDS, and behind the last pivot there are 12 products (k_s = 48; with rows of
// L^{-1} times Phi^T there were 24: factorisation of 256 heads 18.5 us before, 16 now).
template <int M, class STORE, class SHADOW>
__device__ __forceinline__ void sketch_factor(SketchFactor<M> &F, const double (&sum)[Share<M>::TILES],
                                              const PhiRegs<M> &ph, float ridge_rel, STORE &&store, SHADOW &&shadow) {
  constexpr int P = M / 16, SP = factor_pitch(M), PP = SketchFactor<M>::PP;
  constexpr int OWN = 3;                           // channel tiles of a wave: w - 1, w + 2, w + 5
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double *Ss = F.Ss;
  if (tid == 0) F.flag = 0;
  for_lower_tiles<M>([&](int t, int a, int b) {
    Ss[a * SP + b] = sum[t];
    if (a == b) F.d0[a] = sum[t];
  });
#pragma unroll
  for (int i = 0; i < PhiRegs<M>::N; ++i) {
    const int c4 = tid + 256 * i;
    *reinterpret_cast<typename PhiRegs<M>::quad *>(&F.PH[c4 / (M / 4) * PP + c4 % (M / 4) * 4]) = ph.v[i];
  }
  __syncthreads();

  // ridge: rho = ridge_rel * trace(S) / M (every wave sums in the same order); without one, 0 unless S is not finite
  double tr = lane < M ? F.d0[lane] : 0.0;
  if (ridge_rel != 0.f || __any(!(fabs(tr) < 1.0e300))) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) tr += __shfl_xor(tr, d);
    const double rho = (double)ridge_rel * tr / (double)M;
    __syncthreads();
    if (tid < M) {
      const double v = F.d0[tid] + rho;
      Ss[tid * SP + tid] = v;
      F.d0[tid] = v;
    }
    __syncthreads();
  }

  f64x4 R[OWN][P] = {};
  if (wave > 0) {                                  // uniform
    float r[OWN][P][4];
#pragma unroll
    for (int u = 0; u < OWN; ++u)
#pragma unroll
      for (int q = 0; q < P; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v)                // as a 16x16x4 product leaves it: row 4v + lq, channel l16
          r[u][q][v] = F.PH[(16 * min(wave - 1 + 3 * u, D / 16 - 1) + l16) * PP + 16 * q + 4 * v + lq];
#pragma unroll
    for (int u = 0; u < OWN; ++u)
#pragma unroll
      for (int q = 0; q < P; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) R[u][q][v] = (double)r[u][q][v];
  }
  const bool third = wave + 5 < D / 16;            // its third tile exists
  if (wave > 0) shadow(std::integral_constant<int, 0>{});
  factor_panels<P, 4, false>(Ss, F.Xd, F.d0, &F.flag, [&](auto pc) {
    constexpr int pp = decltype(pc)::value;
    double a[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a[ks] = F.Xd[pp][l16][4 * ks + lq];
    f64x4 w[OWN];
#pragma unroll
    for (int u = 0; u < OWN; ++u) w[u] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int u = 0; u < OWN; ++u)
        if (u < 2 || third) w[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks], R[u][pp][ks], w[u], 0, 0, 0);
    static_for<pp + 1, P>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      double l[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) l[ks] = -Ss[(16 * q + l16) * SP + 16 * pp + 4 * ks + lq];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int u = 0; u < OWN; ++u)
          if (u < 2 || third) R[u][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(l[ks], w[u][ks], R[u][q], 0, 0, 0);
    });
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      if (u == 2 && !third) continue;
#pragma unroll
      for (int v = 0; v < 4; v += 2) {
        float x = (float)w[u][v], y = (float)w[u][v + 1];
#pragma unroll
        for (int tt = 0; tt < W_TERMS; ++tt) {
          const unsigned b = split_bf16(x, y);
          store(tt, 16 * pp + 4 * v + lq, 16 * (wave - 1 + 3 * u) + l16, (uint16_t)b);
          store(tt, 16 * pp + 4 * v + 4 + lq, 16 * (wave - 1 + 3 * u) + l16, (uint16_t)(b >> 16));
        }
      }
    }
    if constexpr (pp + 1 < P) shadow(std::integral_constant<int, pp + 1>{});
  });
}

}  // namespace cmp
