// fp64 operand tiles of the matrix-core products, shared by k_gemm.hip and k_hinv.hip.
#pragma once

#include "crvq_internal.h"

namespace crvq {

typedef double d4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
constexpr int kKs = 16;  // k per LDS stage

__device__ __forceinline__ d2v ld2(const double* p) { return *reinterpret_cast<const d2v*>(p); }
__device__ __forceinline__ d2v ld2(const float* p) {
  const f2v v = *reinterpret_cast<const f2v*>(p);
  return d2v{static_cast<double>(v[0]), static_cast<double>(v[1])};
}

__device__ __forceinline__ double lane_f64(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), lane);
  return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
}

// One operand tile of `rows` (a multiple of 32) by kKs, staged through LDS as fp64 (fp32 operands are
// widened exactly).  KMAJ: element (i, k) lies at src[k * ld + i]; otherwise at src[i * ld + k].  The
// LDS layout keeps the memory order, so a 16-byte load becomes one 16-byte LDS write: k-major with a
// row stride of 16 mod 32 doubles, row-major with a stride of 18; in both, the 16 rows x 2 k that half a
// wave reads for an MFMA operand fall on distinct banks.
template <int ROWS, bool KMAJ, typename T>
struct Operand {
  static constexpr int kStride = KMAJ ? ROWS + 16 : kKs + 2;
  static constexpr int kSize = KMAJ ? kKs * kStride : ROWS * kStride;
  static constexpr int kLoads = ROWS * kKs / 2 / 256;
  d2v r[kLoads];
  // The pair of element (i, k) that load s of thread tid holds (the pair runs along i when KMAJ).
  static __device__ __forceinline__ void at(int tid, int s, int& i, int& k) {
    const int e = tid + 256 * s;
    if (KMAJ) {
      k = e / (ROWS / 2);
      i = e % (ROWS / 2) * 2;
    } else {
      i = e / (kKs / 2);
      k = e % (kKs / 2) * 2;
    }
  }
  // src points at the tile's first element; full tiles with 16-byte (fp32: 8-byte) aligned rows
  __device__ __forceinline__ void fetch(const T* __restrict__ src, int64_t ld, int tid) {
#pragma unroll
    for (int s = 0; s < kLoads; ++s) {
      int i, k;
      at(tid, s, i, k);
      r[s] = ld2(src + (KMAJ ? k * ld + i : i * ld + k));
    }
  }
  // any alignment; elements past n_i rows or n_k columns are zero
  __device__ __forceinline__ void fetch_edge(const T* __restrict__ src, int64_t ld, int64_t n_i, int64_t n_k, int tid) {
#pragma unroll
    for (int s = 0; s < kLoads; ++s) {
      int i, k;
      at(tid, s, i, k);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int ii = KMAJ ? i + h : i, kk = KMAJ ? k : k + h;
        r[s][h] = (ii < n_i && kk < n_k) ? static_cast<double>(src[KMAJ ? kk * ld + ii : ii * ld + kk]) : 0.0;
      }
    }
  }
  __device__ __forceinline__ void store(double* lds, int tid) const {
#pragma unroll
    for (int s = 0; s < kLoads; ++s) {
      int i, k;
      at(tid, s, i, k);
      *reinterpret_cast<d2v*>(lds + (KMAJ ? k * kStride + i : i * kStride + k)) = r[s];
    }
  }
  static __device__ __forceinline__ double get(const double* lds, int i, int k) {
    return lds[KMAJ ? k * kStride + i : i * kStride + k];
  }
};

}  // namespace crvq
