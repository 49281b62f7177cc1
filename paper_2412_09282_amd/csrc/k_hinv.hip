// Diagonal of the inverse of the damped Hessian proxy, the denominator of the W-A channel importance
// (Sec. 4.1 Eq. 7): [(H + delta I)^-1]_jj with H = X X^T and delta = damp * mean_j H_jj, in fp64.
//
// With the Cholesky factor L of A = H + delta I and T = L^-1 (lower triangular), A^-1 = T^T T, so
// [A^-1]_jj = sum_i T_ij^2: the squared norms of T's columns.  The matrix is padded to a multiple of 64
// with an identity block, which leaves the leading part's inverse unchanged; only H's lower triangle is
// read.
//   1. A right-looking sweep over 64-wide block columns k forms L: the panel L_ik = A_ik D_k^T (i > k)
//      with D_k = L_kk^-1, then the trailing update A_ij -= L_ik L_jk^T (k < j <= i).  The first
//      workgroup of the update takes the next diagonal block, factors it and forms D_(k+1) while the
//      others update the rest, so the factorization's latency chain is hidden by the update (or hides
//      it, late in the sweep).
//   2. T from its diagonal blocks D_k by doubling: with the inverses T1, T2 of two neighbouring diagonal
//      blocks of size s, the block below T1 is -T2 (L21 T1).  Two launches per size, all pairs at once,
//      long products instead of one rank-64 update per block column.
//   3. The squared column sums, row slabs folded in order.
// All products run on the fp64 matrix cores.  N = 4096: 2.14 ms (5.77 ms when T was formed by a forward
// substitution beside the factorization, with a rank-64 update of both per block column, and every
// workgroup of a panel factored the diagonal block by itself, 59 us; now 15 us beside the update).
// The sweep takes 1.65 ms, bound by the update's memory traffic in its first half (35 us at rank 64) and
// by the diagonal block's chain in its second, the doubling 0.53 ms.
#include "f64_tile.h"

namespace crvq {
namespace {

constexpr int kHb = 64;     // block size
constexpr int kHr = 66;     // LDS stride of the diagonal block: MFMA operand reads are conflict-free
constexpr int kSlabs = 16;  // row slabs of the squared column sums

struct HinvWs {
  double* A;     // Np x Np: H + delta I, then L (blocks below the diagonal)
  double* T;     // Np x Np: T on and below the diagonal blocks, scratch of the doubling above them
  double* sq;    // kSlabs x Np: squared column sums of row slabs
  double* prm;   // [0] delta
  int* flag;     // [0] nonzero once a pivot was not positive and finite
};

HinvWs carve_hinv(WsCursor& c, int64_t Np) {
  HinvWs w;
  w.A = c.take<double>(static_cast<size_t>(Np * Np));
  w.T = c.take<double>(static_cast<size_t>(Np * Np));
  w.sq = c.take<double>(static_cast<size_t>(kSlabs * Np));
  w.prm = c.take<double>(4);
  w.flag = c.take<int>(4);
  return w;
}

// delta = damp * (sum_j H_jj) / N, summed in a fixed order; clears the flag.
__global__ __launch_bounds__(256) void hinv_delta_kernel(const double* __restrict__ H, int64_t ldh, int64_t N,
                                                         double damp, double* __restrict__ prm, int* __restrict__ flag) {
  __shared__ double s[256];
  const int tid = threadIdx.x;
  double a = 0.0;
  for (int64_t j = tid; j < N; j += 256) a += H[j * ldh + j];
  s[tid] = a;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) s[tid] += s[tid + h];
    __syncthreads();
  }
  if (tid == 0) {
    prm[0] = damp * (s[0] / static_cast<double>(N));
    flag[0] = 0;
  }
}

// A = H + delta I on the leading N x N (lower triangle read), identity on the padding; one block row of
// 64 columns per wave and row, the blocks above the diagonal are never read.
__global__ __launch_bounds__(256) void hinv_init_kernel(const double* __restrict__ H, int64_t ldh, int64_t N,
                                                        int64_t Np, const double* __restrict__ prm,
                                                        double* __restrict__ A) {
  const double delta = prm[0];
  const int64_t i = blockIdx.x, jend = (i / kHb + 1) * kHb;
  for (int64_t j = threadIdx.x; j < jend; j += 256) {
    double a;
    if (i < N && j < N)
      a = (j <= i) ? H[i * ldh + j] + (i == j ? delta : 0.0) : 0.0;
    else
      a = (i == j) ? 1.0 : 0.0;
    A[i * Np + j] = a;
  }
}

// 1 / sqrt(x) and 1 / x for x > 0: the hardware estimates (good to about 2^-22) refined by two Newton
// steps, each of which squares the relative error; a few ulps from the rounded quotient.  rcp_f64 needs x and
// 1 / x to be normal numbers, kPivotMin <= x <= kPivotMax; rsqrt_f64 gives NaN, 0 or inf for x that is not positive
// or not finite.
constexpr double kPivotMin = 0x1p-1020, kPivotMax = 0x1p1020;
__device__ __forceinline__ double rsqrt_f64(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double h = x * y;                      // ~ sqrt(x)
    const double e = __builtin_fma(-h, y, 1.0);  // 1 - x y^2
    y = __builtin_fma(0.5 * y, e, y);
  }
  return y;
}
__device__ __forceinline__ double rcp_f64(double x) {
  double y = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double e = __builtin_fma(-x, y, 1.0);
    y = __builtin_fma(y, e, y);
  }
  return y;
}

// Lane J of the 16 lanes' row, in all of them.
template <int J>
__device__ __forceinline__ double bcast16(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + J, 0xf, 0xf, false);  // row_newbcast
}
template <int C, int J>
__device__ __forceinline__ void panel_rest(double (&x)[16], double (&z)[16], double w) {
  if constexpr (J < 16) {
    const double wj = bcast16<J>(w);
    z[J] = __builtin_fma(-z[C], wj, z[J]);
    x[J] = __builtin_fma(-x[C], wj, x[J]);
    panel_rest<C, J + 1>(x, z, w);
  }
}
template <int C>
__device__ __forceinline__ void panel_column(double (&x)[16], double (&z)[16], double before) {
  if constexpr (C < 16) {
    const double d = bcast16<C>(z[C]);
    const double inv = rcp_f64(d);
    // column C - 1 leaves the columns after C while the reciprocal is formed
    if constexpr (C > 0) panel_rest<C - 1, C + 1>(x, z, before);
    const double w = z[C] * inv;
    if constexpr (C < 15) {
      const double wj = bcast16<C + 1>(w);
      z[C + 1] = __builtin_fma(-z[C], wj, z[C + 1]);
      x[C + 1] = __builtin_fma(-x[C], wj, x[C + 1]);
    }
    panel_column<C + 1>(x, z, w);
  }
}
template <int C>
__device__ __forceinline__ void panel_scale(double (&x)[16], double r) {
  if constexpr (C < 16) {
    x[C] = x[C] * bcast16<C>(r);
    panel_scale<C + 1>(x, r);
  }
}
// The same sweep with every column divided by the root of its pivot at once, without reciprocals.
template <int C>
__device__ __forceinline__ void panel_column_any(double (&x)[16], double (&z)[16]) {
  if constexpr (C < 16) {
    const double r = rsqrt_f64(bcast16<C>(z[C]));
    x[C] = x[C] * r;
    z[C] = z[C] * r;
    panel_rest<C, C + 1>(x, z, z[C]);
    panel_column_any<C + 1>(x, z);
  }
}
// 16 columns of a lower triangular factorization: x is a row of them (or, started as a unit vector, a
// column of the diagonal block's inverse factor: forward substitution on the identity is the same
// sweep); z is row lane % 16 of their diagonal block, so that every 16 lanes hold the whole block and a
// pivot row's element reaches the others by one DPP move.  The sweep keeps the columns unscaled,
// x_j -= x_c (z_jc / d_c), so that from one pivot to the next stand only the reciprocal, a product, a
// fused multiply-add and two moves; the columns are divided by sqrt(d_c) at the end, lane c of 16
// forming the root of d_c.  ok becomes false when d_c is not a pivot that rcp_f64 takes.  ANY: any positive pivots
// (chain of the root and its reciprocal per column); ok becomes false when one is not positive and finite.
template <bool ANY>
__device__ __forceinline__ void panel16(double (&x)[16], double (&z)[16], int lane, bool& ok) {
  if constexpr (ANY)
    panel_column_any<0>(x, z);
  else
    panel_column<0>(x, z, 0.0);
  // ANY: the pivot times the estimate of its root's reciprocal, NaN unless 0 < pivot < inf
  double d = z[0];
#pragma unroll
  for (int c = 1; c < 16; ++c) d = (lane & 15) == c ? z[c] : d;
  ok = ok && (ANY ? d > 0.0 && d < __builtin_inf() : d >= kPivotMin && d <= kPivotMax);
  if constexpr (!ANY) panel_scale<0>(x, rsqrt_f64(d));
}

// LDS of the diagonal block's factorization: L on and below the diagonal of Ab; the inverse's 16 x 16
// diagonal blocks in Td, its block (i, j), i > j, at the place of block (j, i) of Ab.
struct DiagLds {
  double Ab[kHb][kHr];
  double Td[4][16][18];
  int ok;  // every pivot was one
};

// acc += P Q for 16 x 16 tiles in LDS (row-major, strides sp and sq), two chains of products
struct Acc2 {
  d4v a = d4v{0.0, 0.0, 0.0, 0.0}, b = d4v{0.0, 0.0, 0.0, 0.0};
  __device__ __forceinline__ double get(int r) const { return a[r] + b[r]; }
};
__device__ __forceinline__ void mma16(const double* P, int sp, const double* Q, int sq, Acc2& acc, int li, int lk) {
  acc.a = __builtin_amdgcn_mfma_f64_16x16x4f64(P[li * sp + lk], Q[lk * sq + li], acc.a, 0, 0, 0);
  acc.b = __builtin_amdgcn_mfma_f64_16x16x4f64(P[li * sp + 4 + lk], Q[(4 + lk) * sq + li], acc.b, 0, 0, 0);
  acc.a = __builtin_amdgcn_mfma_f64_16x16x4f64(P[li * sp + 8 + lk], Q[(8 + lk) * sq + li], acc.a, 0, 0, 0);
  acc.b = __builtin_amdgcn_mfma_f64_16x16x4f64(P[li * sp + 12 + lk], Q[(12 + lk) * sq + li], acc.b, 0, 0, 0);
}

// LDS written by other lanes of this wave
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// M = sum over k = j .. i - 1 of L_ik T_kj, to the place of diagonal block t of L (not read again)
__device__ __forceinline__ void inverse_sum(DiagLds& S, int i, int j, int t, int li, int lk) {
  Acc2 acc;
  for (int k = j; k < i; ++k)
    mma16(&S.Ab[16 * i][16 * k], kHr, k == j ? &S.Td[j][0][0] : &S.Ab[16 * j][16 * k], k == j ? 18 : kHr, acc, li, lk);
#pragma unroll
  for (int r = 0; r < 4; ++r) S.Ab[16 * t + lk + 4 * r][16 * t + li] = acc.get(r);
  wave_sync();
}
// T_ij = -T_ii M with M at diagonal block t
__device__ __forceinline__ void inverse_block(DiagLds& S, int i, int j, int t, int li, int lk) {
  Acc2 acc;
  mma16(&S.Td[i][0][0], 18, &S.Ab[16 * t][16 * t], kHr, acc, li, lk);
#pragma unroll
  for (int r = 0; r < 4; ++r) S.Ab[16 * j + lk + 4 * r][16 * i + li] = -acc.get(r);
  wave_sync();
}

// Factors the 64 x 64 block in S.Ab and writes its inverse factor T (zeros above the diagonal) to out.
// Four panels of 16 columns: wave 0 holds the panel's rows down to 63 in registers, wave 1 forms the
// inverse of the panel's diagonal block; then the rank-16 update of the rest on the matrix cores.
// T_ij = -T_ii sum_k L_ik T_kj: waves 2 and 3 form the blocks whose operands are there beside the
// panels, so that only the last row's product with T_33 is left.  Bound by the chain of 64 pivots.  Returns
// whether every pivot was in the range of panel16<ANY>; if not, the results are nothing.
template <bool ANY>
__device__ __forceinline__ bool factor_sweep(DiagLds& S, double* __restrict__ out, int64_t ld) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  bool ok = true;
  for (int b = 0; b < 4; ++b) {
    const int c0 = 16 * b;
    if (wave < 2) {
      double x[16], z[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) z[j] = S.Ab[c0 + li][c0 + j];
      if (wave == 0) {
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = S.Ab[lane][c0 + j];
      } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = j == li ? 1.0 : 0.0;
      }
      panel16<ANY>(x, z, lane, ok);
      if (wave == 0) {
        // wave 1 may still be reading the diagonal block's rows; the rows below are wave 0's alone
        if (lane >= c0 + 16) {
#pragma unroll
          for (int j = 0; j < 16; ++j) S.Ab[lane][c0 + j] = x[j];
        }
      } else if (lane < 16) {
#pragma unroll
        for (int r = 0; r < 16; ++r) S.Td[b][r][lane] = x[r];
      }
    } else if (b == 2 && wave == 2) {
      inverse_sum(S, 1, 0, 0, li, lk);
      inverse_block(S, 1, 0, 0, li, lk);
    } else if (b == 3) {
      const int j = wave - 2;
      inverse_sum(S, 2, j, j, li, lk);
      inverse_block(S, 2, j, j, li, lk);
      inverse_sum(S, 3, j, j, li, lk);
      if (j == 1) inverse_sum(S, 3, 2, 2, li, lk);
    }
    __syncthreads();
    // tiles (ti, tj), b < tj <= ti, numbered in turn: Ab_ti,tj -= L_ti,b L_tj,b^T
    int n = 0;
    for (int ti = b + 1; ti < 4; ++ti)
      for (int tj = b + 1; tj <= ti; ++tj, ++n) {
        if ((n & 3) != wave) continue;
        Acc2 acc;
#pragma unroll
        for (int ks = 0; ks < 16; ks += 8) {
          acc.a = __builtin_amdgcn_mfma_f64_16x16x4f64(S.Ab[16 * ti + li][c0 + ks + lk], S.Ab[16 * tj + li][c0 + ks + lk],
                                                       acc.a, 0, 0, 0);
          acc.b = __builtin_amdgcn_mfma_f64_16x16x4f64(S.Ab[16 * ti + li][c0 + ks + 4 + lk],
                                                       S.Ab[16 * tj + li][c0 + ks + 4 + lk], acc.b, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double& v = S.Ab[16 * ti + lk + 4 * r][16 * tj + li];
          v = v - acc.get(r);
        }
      }
    if (b < 3) __syncthreads();
  }
  if (wave == 0) {
    const bool all = __ballot(!ok) == 0;
    if (lane == 0) S.ok = all;
  }
  if (wave < 3) inverse_block(S, 3, wave, wave, li, lk);
  __syncthreads();
#pragma unroll
  for (int s = 0; s < kHb * kHb / 256; ++s) {
    const int e = tid + 256 * s, r = e >> 6, c = e & 63, rb = r >> 4, cb = c >> 4;
    const double* v = rb == cb ? &S.Td[rb][r & 15][c & 15] : &S.Ab[16 * cb + (r & 15)][16 * rb + (c & 15)];
    out[r * ld + c] = rb >= cb ? *v : 0.0;
  }
  return S.ok != 0;
}
// The same with the pivots outside rcp_f64's range (a block in memory that holds magnitudes past 1e+-307: hardly
// ever) in a second sweep, from the block's copy in memory.
__device__ __forceinline__ void factor_diag(DiagLds& S, const double* __restrict__ block, double* __restrict__ out,
                                            int64_t ld, int* __restrict__ flag) {
  if (factor_sweep<false>(S, out, ld)) return;
  __syncthreads();
  for (int e = threadIdx.x; e < kHb * kHb; e += 256) S.Ab[e >> 6][e & 63] = block[(e >> 6) * ld + (e & 63)];
  __syncthreads();
  if (!factor_sweep<true>(S, out, ld) && threadIdx.x == 0) flag[0] = 1;
}

// acc = sum_k a(i, k) b(k, j) over K (a multiple of 16) for a 64 x (32 MB) tile, 32 x (16 MB) per wave.
// KA: a(i, k) = a[k * lda + i], else a[i * lda + k]; KB: b(k, j) = b[k * ldb + j], else b[j * ldb + k].
// Two LDS buffers, one barrier per 16 k, AHEAD stages of operands in registers on their way to LDS.
template <bool KA, bool KB, int MB, int AHEAD>
struct Tile {
  using OpA = Operand<kHb, KA, double>;
  using OpB = Operand<32 * MB, KB, double>;
  struct Lds {
    double a[2][OpA::kSize];
    double b[2][OpB::kSize];
  };
  d4v acc[2][MB];
  __device__ __forceinline__ void run(Lds& S, const double* __restrict__ a, int64_t lda, const double* __restrict__ b,
                                      int64_t ldb, int64_t K) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    const int wi = (wave >> 1) * 32, wj = (wave & 1) * 16 * MB;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < MB; ++y) acc[x][y] = d4v{0.0, 0.0, 0.0, 0.0};
    OpA oa[AHEAD];
    OpB ob[AHEAD];
    const int64_t sa = KA ? kKs * lda : kKs, sb = KB ? kKs * ldb : kKs;
#pragma unroll
    for (int p = 0; p < AHEAD; ++p)
      if (p * kKs < K) {
        oa[p].fetch(a + p * sa, lda, tid);
        ob[p].fetch(b + p * sb, ldb, tid);
      }
    const int64_t stages = K / kKs;
    for (int64_t s0 = 0; s0 < stages; s0 += 2 * AHEAD)
#pragma unroll
      for (int p = 0; p < 2 * AHEAD; ++p) {  // register set p % AHEAD, LDS buffer p % 2
        const int64_t st = s0 + p;
        if (st >= stages) break;
        oa[p % AHEAD].store(S.a[p & 1], tid);
        ob[p % AHEAD].store(S.b[p & 1], tid);
        // the other buffer's readers have passed this barrier's predecessor
        __syncthreads();
        if (st + AHEAD < stages) {
          oa[p % AHEAD].fetch(a + (st + AHEAD) * sa, lda, tid);
          ob[p % AHEAD].fetch(b + (st + AHEAD) * sb, ldb, tid);
        }
#pragma unroll
        for (int ks = 0; ks < kKs; ks += 4) {
          double av[2], bv[MB];
#pragma unroll
          for (int t = 0; t < 2; ++t) av[t] = OpA::get(S.a[p & 1], wi + 16 * t + li, ks + lk);
#pragma unroll
          for (int t = 0; t < MB; ++t) bv[t] = OpB::get(S.b[p & 1], wj + 16 * t + li, ks + lk);
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < MB; ++y)
              acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], bv[y], acc[x][y], 0, 0, 0);
        }
      }
  }
  // f(i, j, v) for this thread's elements (i, j) of the tile and their sums v
  template <class F>
  __device__ __forceinline__ void each(F f) const {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < MB; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          f((wave >> 1) * 32 + 16 * x + (lane >> 4) + 4 * r, (wave & 1) * 16 * MB + 16 * y + (lane & 15), acc[x][y][r],
            (x * MB + y) * 4 + r);
  }
};
using UpdateTile = Tile<false, false, 2, 4>;  // rank 64: all four stages in flight at once

// g = a (a + 1) / 2 + b, 0 <= b <= a
__device__ __forceinline__ void tri_index(int64_t g, int64_t& a, int64_t& b) {
  a = static_cast<int64_t>((sqrt(8.0 * static_cast<double>(g) + 1.0) - 1.0) * 0.5);
  while (a * (a + 1) / 2 > g) --a;
  while ((a + 1) * (a + 2) / 2 <= g) ++a;
  b = g - a * (a + 1) / 2;
}

// The first diagonal block.
__global__ __launch_bounds__(256) void hinv_first_kernel(const double* __restrict__ A, double* __restrict__ T, int64_t Np,
                                                         int* __restrict__ flag) {
  __shared__ DiagLds S;
  for (int e = threadIdx.x; e < kHb * kHb; e += 256) S.Ab[e >> 6][e & 63] = A[(e >> 6) * Np + (e & 63)];
  __syncthreads();
  factor_diag(S, A, T, Np, flag);
}

// The panel of block column k in place, L_ik = A_ik D_k^T: 16 rows per workgroup (so that the few block
// rows still spread over the device), 16 columns per wave.
__global__ __launch_bounds__(256) void hinv_panel_kernel(double* __restrict__ A, const double* __restrict__ T, int64_t Np,
                                                         int64_t k) {
  __shared__ double Dr[kHb][kHr];
  __shared__ double Ar[16][kHr];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int64_t kb = k * kHb;
  double* C = A + ((k + 1) * kHb + static_cast<int64_t>(blockIdx.x) * 16) * Np + kb;
  const double* D = T + kb * Np + kb;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int e = tid + 256 * s, r = e >> 5, m = (e & 31) * 2;
    *reinterpret_cast<d2v*>(&Dr[r][m]) = ld2(D + r * Np + m);
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int e = tid + 256 * s, r = e >> 5, m = (e & 31) * 2;
    *reinterpret_cast<d2v*>(&Ar[r][m]) = ld2(C + r * Np + m);
  }
  __syncthreads();
  // two chains of products (even and odd groups of four k), added at the end
  d4v acc[2] = {d4v{0.0, 0.0, 0.0, 0.0}, d4v{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int ks = 0; ks < kHb; ks += 4)
    acc[(ks >> 2) & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(Ar[li][ks + lk], Dr[16 * wave + li][ks + lk], acc[(ks >> 2) & 1],
                                                              0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) C[(lk + 4 * r) * Np + 16 * wave + li] = acc[0][r] + acc[1][r];
}

// The trailing update A_ij -= L_ik L_jk^T, k < j <= i.  Workgroup 0 takes the next diagonal block and
// factors it.
__global__ __launch_bounds__(256) void hinv_update_kernel(double* __restrict__ A, double* __restrict__ T, int64_t Np,
                                                          int64_t k, int* __restrict__ flag) {
  __shared__ union {
    UpdateTile::Lds tile;
    DiagLds diag;
  } S;
  int64_t a, b;
  tri_index(blockIdx.x, a, b);
  const int64_t kb = k * kHb, ib = (k + 1 + a) * kHb, jb = (k + 1 + b) * kHb;
  double* C = A + ib * Np + jb;  // (jb = ib for workgroup 0)
  double old[16];
  UpdateTile t;
  t.each([&](int i, int j, double, int n) { old[n] = C[i * Np + j]; });
  t.run(S.tile, A + ib * Np + kb, Np, A + jb * Np + kb, Np, kHb);
  if (blockIdx.x == 0) {
    __syncthreads();  // the operand buffers are the diagonal block's memory
    t.each([&](int i, int j, double v, int n) {
      S.diag.Ab[i][j] = old[n] - v;
      C[i * Np + j] = old[n] - v;
    });
    __syncthreads();
    factor_diag(S.diag, C, T + ib * Np + ib, Np, flag);
    return;
  }
  t.each([&](int i, int j, double v, int n) { C[i * Np + j] = old[n] - v; });
}

// One doubling of T: diagonal blocks of nb tiles (64 nb rows) in pairs blockIdx.y, with first rows
// o1 = 2 nb y and o2 = o1 + nb (in tiles), the second of n2 = min(nb, tiles - o2) tiles.
// Step 1 writes M^T = (L21 T1)^T above the diagonal: M^T_ji = sum_{k >= j} T1_kj^T L21_ik^T.  Step 2 writes
// T21_ij = -sum_{k <= i} T2_ik M_kj.  The sums have 1 .. nb tiles: a workgroup takes the results with
// the m-th longest and the m-th shortest sum in turn, in halves of 32 columns (blockIdx.z), so that all
// workgroups do the same work.
template <int STEP>
__global__ __launch_bounds__(256) void hinv_double_kernel(const double* __restrict__ A, double* __restrict__ T, int64_t Np,
                                                          int64_t tiles, int64_t nb) {
  using DTile = Tile<STEP == 1, false, 1, 2>;
  __shared__ typename DTile::Lds S;
  const int64_t o1 = 2 * nb * blockIdx.y, o2 = o1 + nb, n2 = tiles - o2 < nb ? tiles - o2 : nb;
  const int64_t m = blockIdx.x / nb, other = blockIdx.x % nb, c0 = static_cast<int64_t>(blockIdx.z) * 32;
  for (int h = 0; h < 2; ++h) {
    const int64_t q = h == 0 ? m : nb - 1 - m;  // the tile index that fixes the sum's length
    if (h == 1 && q == m) break;
    const int64_t i = STEP == 1 ? other : q, j = STEP == 1 ? q : other;
    if (i >= n2) continue;
    DTile t;
    double* C;
    if (h == 1) __syncthreads();  // the first result's last stage is still being read
    if (STEP == 1) {
      // rows j of T1^T, columns i of L21^T, k from tile j
      t.run(S, T + (o1 + j) * kHb * Np + (o1 + j) * kHb, Np, A + ((o2 + i) * kHb + c0) * Np + (o1 + j) * kHb, Np,
            (nb - j) * kHb);
      C = T + (o1 + j) * kHb * Np + (o2 + i) * kHb + c0;
    } else {
      t.run(S, T + (o2 + i) * kHb * Np + o2 * kHb, Np, T + ((o1 + j) * kHb + c0) * Np + o2 * kHb, Np, (i + 1) * kHb);
      C = T + (o2 + i) * kHb * Np + (o1 + j) * kHb + c0;
    }
    t.each([&](int r, int c, double v, int) { C[r * Np + c] = STEP == 1 ? v : -v; });
  }
}

// sq[slab][j] = sum of T_ij^2 over the slab's rows i (rows in order per wave, then the four waves): one
// workgroup per 64 columns and slab.
__global__ __launch_bounds__(256) void hinv_square_kernel(const double* __restrict__ T, int64_t Np, int64_t rows,
                                                          double* __restrict__ sq) {
  __shared__ double red[4][kHb];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kHb;
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * rows, r1 = r0 + rows < Np ? r0 + rows : Np;
  double s = 0.0;
#pragma unroll 4
  for (int64_t i = (r0 > j0 ? r0 : j0) + wave; i < r1; i += 4) {
    const double t = T[i * Np + j0 + lane];
    s = __builtin_fma(t, t, s);
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave == 0)
    sq[blockIdx.y * Np + j0 + lane] = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
}

// hinv[j] = sum_i T_ij^2 and scale[j] = float(1 / (2 hinv[j])), or NaN for all when the flag is set.
__global__ __launch_bounds__(256) void hinv_finish_kernel(int64_t N, int64_t Np, const double* __restrict__ sq,
                                                          const int* __restrict__ flag, double* __restrict__ hinv,
                                                          float* __restrict__ scale) {
  const bool bad = flag[0] != 0;
  for (int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; j < N;
       j += static_cast<int64_t>(gridDim.x) * 256) {
    double v = 0.0;
    for (int p = 0; p < kSlabs; ++p) v = v + sq[p * Np + j];
    if (bad) v = __builtin_nan("");
    if (hinv) hinv[j] = v;
    if (scale) scale[j] = static_cast<float>(1.0 / (2.0 * v));
  }
}

}  // namespace

size_t hinv_ws_bytes(int64_t N) {
  const int64_t Np = (N + kHb - 1) / kHb * kHb;
  WsCursor c(nullptr);
  (void)carve_hinv(c, Np);
  return c.used;
}

hipError_t launch_hinv(const double* H, int64_t ldh, int64_t N, double damp, double* hinv, float* scale, void* ws,
                       hipStream_t stream) {
  const int64_t nblk = (N + kHb - 1) / kHb, Np = nblk * kHb;
  WsCursor c(ws);
  const HinvWs w = carve_hinv(c, Np);
  hipLaunchKernelGGL(hinv_delta_kernel, dim3(1), dim3(256), 0, stream, H, ldh, N, damp, w.prm, w.flag);
  hipLaunchKernelGGL(hinv_init_kernel, dim3(static_cast<unsigned>(Np)), dim3(256), 0, stream, H, ldh, N, Np, w.prm, w.A);
  hipLaunchKernelGGL(hinv_first_kernel, dim3(1), dim3(256), 0, stream, w.A, w.T, Np, w.flag);
  for (int64_t k = 0; k + 1 < nblk; ++k) {
    const int64_t nbelow = nblk - 1 - k;
    hipLaunchKernelGGL(hinv_panel_kernel, dim3(static_cast<unsigned>(4 * nbelow)), dim3(256), 0, stream, w.A, w.T, Np, k);
    hipLaunchKernelGGL(hinv_update_kernel, dim3(static_cast<unsigned>(nbelow * (nbelow + 1) / 2)), dim3(256), 0, stream,
                       w.A, w.T, Np, k, w.flag);
  }
  for (int64_t nb = 1; nb < nblk; nb *= 2) {
    // pairs whose second block holds at least one tile
    const dim3 grid(static_cast<unsigned>((nb + 1) / 2 * nb), static_cast<unsigned>(cdiv(nblk - nb, 2 * nb)), 2);
    hipLaunchKernelGGL(hinv_double_kernel<1>, grid, dim3(256), 0, stream, w.A, w.T, Np, nblk, nb);
    hipLaunchKernelGGL(hinv_double_kernel<2>, grid, dim3(256), 0, stream, w.A, w.T, Np, nblk, nb);
  }
  const int64_t rows = cdiv(Np, kSlabs);
  hipLaunchKernelGGL(hinv_square_kernel, dim3(static_cast<unsigned>(nblk), kSlabs), dim3(256), 0, stream, w.T, Np, rows,
                     w.sq);
  hipLaunchKernelGGL(hinv_finish_kernel, dim3(static_cast<unsigned>(std::min<int64_t>(cdiv(N, 256), 4096))),
                     dim3(256), 0, stream, N, Np, w.sq, w.flag, hinv, scale);
  return hipGetLastError();
}

}  // namespace crvq
