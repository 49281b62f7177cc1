// fp64 matrix products on the matrix cores: the Hessian proxy H = X^T X, the products R H of the
// refinement and the rank-k updates of its code search.
#include "f64_tile.h"

namespace crvq {
namespace {

// C[i][j] = sum_k opA(i, k) B(k, j) (C[i][j] - that sum when SUB), opA(i, k) = A[i * lda + k], or
// A[k * lda + i] when TRANS_A; products exact for fp32 operands, accumulated in k order (within a
// group of four by the matrix core).  A workgroup of 2 x 2 waves forms a 32 MA x 32 MB tile, each wave
// MA x MB v_mfma_f64_16x16x4f64 tiles: lane l supplies A[i0 + l % 16][k + l / 16] and
// B[k + l / 16][j0 + l % 16] and holds C[i0 + l / 16 + 4 r][j0 + l % 16], r < 4.  blockIdx.z takes the k
// range [z kchunk, (z + 1) kchunk) and writes its own slice of C.
// SYM (A and B the same array, TRANS_A, MA = MB): only the tiles on and below the diagonal are formed
// (blockIdx.x numbers them), every element below it is written twice; a product does not depend on
// the order of its factors, so the mirrored half holds the bits it would have been given.
//
// Bound by the matrix core (128 flop per CU and cycle in fp64, 64 cycles per MFMA).  Two LDS buffers
// and one barrier per stage; the next stage's operands travel to registers during the MFMAs and
// interior tiles load 16 bytes without bounds tests: 4096 x 4096 x 4096 takes 2.09 ms (66 TFLOP/s; with
// one buffer, two barriers and tested 8-byte loads 2.70 ms).
template <bool SUB, bool SYM, int MA, int MB, typename TA, typename TB, bool TRANS_A>
__global__ __launch_bounds__(256, 2) void gemm_f64_kernel(int64_t M, int64_t Nc, int64_t Kd,
                                                          const TA* __restrict__ A, int64_t lda,
                                                          const TB* __restrict__ B, int64_t ldb,
                                                          double* __restrict__ C, int64_t ldc, int64_t kchunk,
                                                          int64_t c_part, int vec) {
  constexpr int TM = 32 * MA, TN = 32 * MB;
  using OpA = Operand<TM, TRANS_A, TA>;
  using OpB = Operand<TN, true, TB>;
  __shared__ double As[2][OpA::kSize];
  __shared__ double Bs[2][OpB::kSize];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = (wave >> 1) * 16 * MA, wj = (wave & 1) * 16 * MB;
  const int li = lane & 15, lk = lane >> 4;
  int64_t bi, bj;
  if (SYM) {
    const int64_t g = blockIdx.x;  // g = bi (bi + 1) / 2 + bj, 0 <= bj <= bi
    bi = static_cast<int64_t>((sqrt(8.0 * static_cast<double>(g) + 1.0) - 1.0) * 0.5);
    while (bi * (bi + 1) / 2 > g) --bi;
    while ((bi + 1) * (bi + 2) / 2 <= g) ++bi;
    bj = g - bi * (bi + 1) / 2;
  } else {
    bi = blockIdx.y;
    bj = blockIdx.x;
  }
  const int64_t i0 = bi * TM, j0 = bj * TN;
  const int64_t kb = static_cast<int64_t>(blockIdx.z) * kchunk;
  const int64_t ke = kb + kchunk < Kd ? kb + kchunk : Kd;
  C += static_cast<int64_t>(blockIdx.z) * c_part;
  const bool full = vec && i0 + TM <= M && j0 + TN <= Nc;
  const TA* ap = A + (TRANS_A ? i0 : i0 * lda);
  const TB* bp = B + j0;
  OpA oa;
  OpB ob;
  auto fetch = [&](int64_t k0) {
    const TA* a = ap + (TRANS_A ? k0 * lda : k0);
    const TB* b = bp + k0 * ldb;
    if (full && k0 + kKs <= ke) {
      oa.fetch(a, lda, tid);
      ob.fetch(b, ldb, tid);
    } else {
      oa.fetch_edge(a, lda, M - i0, ke - k0, tid);
      ob.fetch_edge(b, ldb, Nc - j0, ke - k0, tid);
    }
  };
  d4v acc[MA][MB];
#pragma unroll
  for (int a = 0; a < MA; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[a][b] = d4v{0.0, 0.0, 0.0, 0.0};
  if (kb < ke) {
    fetch(kb);
    oa.store(As[0], tid);
    ob.store(Bs[0], tid);
  }
  int cur = 0;
  for (int64_t k0 = kb; k0 < ke; k0 += kKs) {
    // this buffer is filled, and every wave has left the other one
    __syncthreads();
    const bool more = k0 + kKs < ke;
    if (more) fetch(k0 + kKs);
    const double* as = As[cur];
    const double* bs = Bs[cur];
#pragma unroll
    for (int ks = 0; ks < kKs; ks += 4) {
      double a[MA], b[MB];
#pragma unroll
      for (int t = 0; t < MA; ++t) a[t] = OpA::get(as, wi + 16 * t + li, ks + lk);
#pragma unroll
      for (int t = 0; t < MB; ++t) b[t] = OpB::get(bs, wj + 16 * t + li, ks + lk);
#pragma unroll
      for (int ta = 0; ta < MA; ++ta)
#pragma unroll
        for (int tb = 0; tb < MB; ++tb)
          acc[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
    }
    cur ^= 1;
    if (more) {
      oa.store(As[cur], tid);
      ob.store(Bs[cur], tid);
    }
  }
  const bool inside = i0 + TM <= M && j0 + TN <= Nc;
#pragma unroll
  for (int ta = 0; ta < MA; ++ta)
#pragma unroll
    for (int tb = 0; tb < MB; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gi = i0 + wi + 16 * ta + lk + 4 * r, gj = j0 + wj + 16 * tb + li;
        if (!inside && (gi >= M || gj >= Nc)) continue;
        const double v = acc[ta][tb][r];
        if (SYM) {
          if (gi < gj) continue;
          C[gi * ldc + gj] = v;
          if (gi > gj) C[gj * ldc + gi] = v;
        } else {
          C[gi * ldc + gj] = SUB ? C[gi * ldc + gj] - v : v;
        }
      }
}

// C[i][j] = sum over parts p = 0 .. P - 1 in order of part[p][i][j] (the split-k partial products).
__global__ __launch_bounds__(256) void sum_parts_kernel(int64_t M, int64_t Nc, int P, const double* __restrict__ part,
                                                        double* __restrict__ C, int64_t ldc) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (e >= M * Nc) return;
  double acc = part[e];
  for (int p = 1; p < P; ++p) acc = acc + part[static_cast<int64_t>(p) * M * Nc + e];
  const int64_t i = e / Nc, j = e - i * Nc;
  C[i * ldc + j] = acc;
}

// Rows that start at multiples of a pair of elements, so that interior tiles may load pairs.
template <typename T>
int pair_aligned(const T* p, int64_t ld) {
  return (ld % 2 == 0 && reinterpret_cast<uintptr_t>(p) % (2 * sizeof(T)) == 0) ? 1 : 0;
}

// Column tiles per wave pair: narrow outputs take the tile that covers them.
int tile_b(int64_t Nc) { return Nc > 96 ? 4 : static_cast<int>(cdiv(Nc, 32)); }

template <bool SUB, int MA, int MB>
void launch_plain(int64_t M, int64_t Nc, int64_t Kd, const double* A, int64_t lda, const double* B, int64_t ldb,
                  double* C, int64_t ldc, int64_t kchunk, int64_t parts, int64_t c_part, hipStream_t stream) {
  const dim3 grid(static_cast<unsigned>(cdiv(Nc, 32 * MB)), static_cast<unsigned>(cdiv(M, 32 * MA)),
                  static_cast<unsigned>(parts));
  hipLaunchKernelGGL((gemm_f64_kernel<SUB, false, MA, MB, double, double, false>), grid, dim3(256), 0, stream, M, Nc,
                     Kd, A, lda, B, ldb, C, ldc, kchunk, c_part, pair_aligned(A, lda) & pair_aligned(B, ldb));
}

}  // namespace

hipError_t launch_gram_f64(int64_t N, int64_t rows, const void* X, int type, int64_t ld, double* H, int64_t ldh,
                           hipStream_t stream) {
  if (N <= 0) return hipSuccess;
  // 64 x 64 tiles: at N = 4096 the lower triangle is 2080 of them, and only 528 of 128 x 128, which
  // leaves a last round of 16 (0.76 against 0.90 ms; 1.74 ms when all tiles were formed)
  const int64_t nt = cdiv(N, 64);
  const dim3 grid(static_cast<unsigned>(nt * (nt + 1) / 2));
  if (type == ET_F32) {
    const float* x = static_cast<const float*>(X);
    hipLaunchKernelGGL((gemm_f64_kernel<false, true, 2, 2, float, float, true>), grid, dim3(256), 0, stream, N, N, rows,
                       x, ld, x, ld, H, ldh, rows, int64_t{0}, pair_aligned(x, ld));
  } else {
    const double* x = static_cast<const double*>(X);
    hipLaunchKernelGGL((gemm_f64_kernel<false, true, 2, 2, double, double, true>), grid, dim3(256), 0, stream, N, N,
                       rows, x, ld, x, ld, H, ldh, rows, int64_t{0}, pair_aligned(x, ld));
  }
  return hipGetLastError();
}

hipError_t launch_gemm_f64(int64_t M, int64_t Nc, int64_t Kd, const double* A, int64_t lda, const double* B,
                           int64_t ldb, double* C, int64_t ldc, bool sub, hipStream_t stream) {
  if (M <= 0 || Nc <= 0) return hipSuccess;
  // The rank-k updates read and write C, so they want many workgroups in flight: 64 x 64 tiles (the
  // updates of a 4096 x 4096 code search 1.50 ms, 2.97 ms before at rank 64; 128 x 128 tiles 1.65 ms).
  // A plain product takes 128 x 128 tiles when they fill whole rounds of two per CU: 4096 x 4096 x 4096
  // (1024 tiles) 2.09 against 2.25 ms, and 64 x 64 tiles otherwise: 4500 x 3000 (864 tiles) 1.56 against
  // 1.84 ms, 1000 x 1000 (64 tiles) 95 against 213 us.
  const int64_t tiles = cdiv(M, 128) * cdiv(Nc, 128), last = tiles % 512;
  const bool big = tiles >= 2048 || (tiles >= 512 && (last == 0 || last >= 384));
  if (sub)
    launch_plain<true, 2, 2>(M, Nc, Kd, A, lda, B, ldb, C, ldc, Kd, 1, 0, stream);
  else if (big)
    launch_plain<false, 4, 4>(M, Nc, Kd, A, lda, B, ldb, C, ldc, Kd, 1, 0, stream);
  else
    launch_plain<false, 2, 2>(M, Nc, Kd, A, lda, B, ldb, C, ldc, Kd, 1, 0, stream);
  return hipGetLastError();
}

// C = A B split over k into P parts of at least 256 when the output grid alone is too small to fill
// the device; part products go to ws (P x M x Nc doubles) and are summed in part order, so the result
// does not depend on scheduling.
int64_t gemm_split_parts(int64_t M, int64_t Nc, int64_t Kd) {
  const int64_t tiles = cdiv(Nc, 32 * tile_b(Nc)) * cdiv(M, 128);
  int64_t P = tiles >= 256 ? 1 : cdiv(512, tiles);
  const int64_t maxp = Kd / 256 > 1 ? Kd / 256 : 1;
  return P < maxp ? P : maxp;
}

hipError_t launch_gemm_f64_split(int64_t M, int64_t Nc, int64_t Kd, const double* A, int64_t lda, const double* B,
                                 int64_t ldb, double* C, int64_t ldc, double* ws, hipStream_t stream) {
  if (M <= 0 || Nc <= 0) return hipSuccess;
  const int64_t P = gemm_split_parts(M, Nc, Kd);
  const int64_t kchunk = P > 1 ? cdiv(cdiv(Kd, P), kKs) * kKs : Kd;
  const int64_t parts = P > 1 ? cdiv(Kd, kchunk) : 1;
  double* out = P > 1 ? ws : C;
  const int64_t ldo = P > 1 ? Nc : ldc;
  switch (tile_b(Nc)) {
    case 1: launch_plain<false, 4, 1>(M, Nc, Kd, A, lda, B, ldb, out, ldo, kchunk, parts, M * Nc, stream); break;
    case 2: launch_plain<false, 4, 2>(M, Nc, Kd, A, lda, B, ldb, out, ldo, kchunk, parts, M * Nc, stream); break;
    case 3: launch_plain<false, 4, 3>(M, Nc, Kd, A, lda, B, ldb, out, ldo, kchunk, parts, M * Nc, stream); break;
    default: launch_plain<false, 4, 4>(M, Nc, Kd, A, lda, B, ldb, out, ldo, kchunk, parts, M * Nc, stream); break;
  }
  if (P > 1)
    hipLaunchKernelGGL(sum_parts_kernel, dim3(static_cast<unsigned>(cdiv(M * Nc, 256))), dim3(256), 0, stream, M, Nc,
                       static_cast<int>(parts), ws, C, ldc);
  return hipGetLastError();
}

}  // namespace crvq
