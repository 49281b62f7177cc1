// Nearest codeword of at most 256 (d <= 16) in one launch: codebook pack, screen, exact winner,
// certificate and exact search of the rows it leaves uncertain.
#include <climits>

#include "screen_common.h"

namespace crvq {
namespace {

// Row i of d = 8 H packed, 16-byte aligned elements.  FT 1: fp32, FT 2: bf16.
template <int H, int FT>
__device__ __forceinline__ void packed_row(const void* base, int64_t i, float (&v)[8 * H]) {
  if constexpr (FT == 1) {
    const f4* p = static_cast<const f4*>(base) + 2 * H * i;
#pragma unroll
    for (int q = 0; q < 2 * H; ++q) {
      const f4 a = p[q];
#pragma unroll
      for (int t = 0; t < 4; ++t) v[4 * q + t] = a[t];
    }
  } else {
    const uint4* p = static_cast<const uint4*>(base) + H * i;
#pragma unroll
    for (int q = 0; q < H; ++q) {
      const uint4 a = p[q];
      const uint32_t u[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        v[8 * q + 2 * t] = __uint_as_float(u[t] << 16);
        v[8 * q + 2 * t + 1] = __uint_as_float(u[t] & 0xffff0000u);
      }
    }
  }
}

constexpr float kFar = 3.0e38f;  // screen value of a padding codeword, past every searchable one

// The smaller (larger) of this lane's value and that of lane ^ 16 or ^ 32, in both.
template <int MASK>
__device__ __forceinline__ void both(float v, float& a, float& b) {
  const uint32_t u = __float_as_uint(v);
  if constexpr (MASK == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  }
}
template <int MASK>
__device__ __forceinline__ void merge_groups(float& m1, float& m2) {
  float a1, b1, a2, b2;
  both<MASK>(m1, a1, b1);
  both<MASK>(m2, a2, b2);
  m2 = fminf(fminf(a2, b2), fmaxf(a1, b1));
  m1 = fminf(a1, b1);
}

// A wave screens 16 CB rows at a time against the whole book with the split-bf16 operands of SplitOps
// (one MFMA per 8 dimensions and 16 x 16 tile), the book packed into LDS by every workgroup for itself.
// It tracks cells: the four codewords 16 T + 4 g .. + 3 whose values tile T gives lane group g.  A cell's
// minimum carries the cell's number 4 T + g in its six lowest bits (2^-17 of the value at most, part of
// the bound), so keeping the smallest and the second smallest cell takes five VALU operations per four
// values and no index registers.  The winning cell's codewords are compared in fp32 and, where two are
// within its error, exactly in fp64 in (D, k) order; the winner is certain when no codeword outside the
// cell can reach its distance (the bound of finalize_kernel with R = ||x|| + sqrt(D)).  The other rows
// (about one in 300) are searched exactly by their wave.  fp64 distances are formed only where they are
// asked for.  FT: packed aligned rows of one type (packed_row), 0 any layout; H: halves of 8
// dimensions.  Bound by VALU issue (about 1800 instructions per 128 rows of 8, a third of them the split
// of the rows; 80 % of the cycles).  5.6 M fp32 rows of 8 against 256 codewords: 185 us;
// with a codebook launch, every winning
// cell scored in fp64, six operations per cell and a rescue launch 250 us.  1 M rows of 16: 65 us (fp32
// matrix instructions and a finalize pass 186 us).  8192 rows: 5 us (17 us in three launches).
template <int H, int FT, int CB>
__global__ __launch_bounds__(256) void assign_small_kernel(RowSrc src, const void* __restrict__ C, int ct, int K,
                                                           float acc_ulps, float split_coef,
                                                           int32_t* __restrict__ codes, float* __restrict__ dist,
                                                           double* __restrict__ rowD, int* __restrict__ rowK) {
  constexpr int DM = 8 * H;
  constexpr int kChunks = 8 * H;  // 16-byte chunks of a cell of four codewords
  __shared__ uint16_t apack[H][256 * 16];
  __shared__ f4 cn4[64];
  __shared__ f4 cf[256 * 2 * H];  // fp32 codewords; a cell's chunk j at j ^ (cell mod kChunks): spread over the banks
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, jl = lane & 15, g = lane >> 4;
  const int d = src.d;
  const int64_t n = src.n;
  {
    const int k = tid;
    float c[DM];
    load_codeword<DM>(C, ct, k, d, k < K, c);
    float nrm = 0.0f;
#pragma unroll
    for (int t = 0; t < DM; ++t) nrm = nrm + c[t] * c[t];
    reinterpret_cast<float*>(cn4)[k] = k < K ? nrm : kFar;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      u16x8 hi, lo;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        uint16_t a, b;
        bf16_split(c[8 * h + t], a, b);
        hi[t] = a;
        lo[t] = b;
      }
      reinterpret_cast<u16x8*>(apack[h])[2 * k] = hi;
      reinterpret_cast<u16x8*>(apack[h])[2 * k + 1] = lo;
    }
    const int cell = k >> 2;
#pragma unroll
    for (int q = 0; q < 2 * H; ++q)
      cf[cell * kChunks + (((k & 3) * 2 * H + q) ^ (cell & (kChunks - 1)))] =
          f4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
  }
  __syncthreads();
  auto codeword = [&](int k, float (&c)[DM]) {
    const int cell = k >> 2;
#pragma unroll
    for (int q = 0; q < 2 * H; ++q) {
      const f4 a = cf[cell * kChunks + (((k & 3) * 2 * H + q) ^ (cell & (kChunks - 1)))];
#pragma unroll
      for (int t = 0; t < 4; ++t) c[4 * q + t] = a[t];
    }
  };
  auto distance = [&](const double (&x)[DM], const float (&c)[DM]) {
    double D = 0.0;
#pragma unroll
    for (int t = 0; t < DM; ++t) {
      if (FT != 0 || t < d) {
        const double diff = x[t] - static_cast<double>(c[t]);
        D = D + diff * diff;
      }
    }
    return D;
  };
  auto row_f32 = [&](int64_t i, float (&v)[DM]) {
    if constexpr (FT == 0) {
      if (src.type == ET_F64) {
        const int64_t off = row_offset(src, i);
#pragma unroll
        for (int t = 0; t < DM; ++t) v[t] = t < d ? static_cast<float>(row_elem(src, off, t)) : 0.0f;
      } else if (src.type == ET_F32) {
        load_f32_elems<DM>(static_cast<const float*>(src.base) + row_offset(src, i), d, true, v);
      } else {
        load_bf16_elems<DM>(static_cast<const uint16_t*>(src.base) + row_offset(src, i), d, true, v);
      }
    } else {
      packed_row<H, FT>(src.base, i, v);
    }
  };
  const bool want_dist = dist != nullptr || codes == nullptr;
  auto exact_row = [&](int64_t i, double (&x)[DM]) {
    if constexpr (FT == 0) {
      load_row_exact<DM>(src, i, true, x);
    } else {
      float v[DM];
      packed_row<H, FT>(src.base, i, v);
#pragma unroll
      for (int t = 0; t < DM; ++t) x[t] = static_cast<double>(v[t]);
    }
  };
  const int tiles = (K + 15) / 16;
  const int64_t groups = (n + 16 * CB - 1) / (16 * CB);
  for (int64_t grp = static_cast<int64_t>(blockIdx.x) * 4 + wave; grp < groups; grp += static_cast<int64_t>(gridDim.x) * 4) {
    const int64_t row0 = grp * (16 * CB);
    SplitOps::B bop[CB][H];
    {
      // every load in flight before the first split; a row past the end repeats the last one (its column
      // is never read)
      float v[CB][DM];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        int64_t i = row0 + cb * 16 + jl;
        i = i < n ? i : n - 1;
        row_f32(i, v[cb]);
      }
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int h = 0; h < H; ++h) {
          float w[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) w[t] = v[cb][8 * h + t];
          bop[cb][h] = SplitOps::make_b_vals(w, g);
        }
    }
    float m1[CB], m2[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      m1[cb] = kFar;
      m2[cb] = kFar;
    }
    for (int T = 0; T < tiles; ++T) {
      SplitOps::A a[H];
#pragma unroll
      for (int h = 0; h < H; ++h)
        a[h].v = *reinterpret_cast<const bf8*>(apack[h] + (T * 16 + jl) * 16 + (lane >> 5) * 8);
      const f4 c4 = cn4[4 * T + g];
      const uint32_t id = static_cast<uint32_t>(4 * T + g);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        f4 acc = SplitOps::mfma(a[0], bop[cb][0], c4);
        if constexpr (H == 2) acc = SplitOps::mfma(a[1], bop[cb][1], acc);
        const float cm = fminf(fminf(acc[0], acc[1]), fminf(acc[2], acc[3]));
        const float key = __uint_as_float((__float_as_uint(cm) & ~63u) | id);
        m2[cb] = __builtin_amdgcn_fmed3f(m1[cb], m2[cb], key);  // m1 <= m2 holds throughout
        m1[cb] = fminf(m1[cb], key);
      }
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      merge_groups<16>(m1[cb], m2[cb]);
      merge_groups<32>(m1[cb], m2[cb]);
    }
    // Every lane group holds the merged state of all CB blocks; group g finishes the rows of blocks g,
    // g + 4, ...
#pragma unroll
    for (int rr = 0; rr < (CB + 3) / 4; ++rr) {
      float s1 = kFar, s2 = kFar;
#pragma unroll
      for (int cb = 4 * rr; cb < 4 * rr + 4 && cb < CB; ++cb) {
        if (cb - 4 * rr == g) {
          s1 = m1[cb];
          s2 = m2[cb];
        }
      }
      const int cbm = 4 * rr + g;
      const int64_t i = row0 + cbm * 16 + jl;
      const bool live = cbm < CB && i < n;
      bool certain = true;
      double D1 = 0.0;
      int kk = 0;
      if (live) {
        // no searchable winner (a NaN row, values past fp32): the exact search takes the row
        const bool has = s1 < 1.0e38f;
        const int kc = has ? static_cast<int>(__float_as_uint(s1) & 63u) * 4 : 0;
        float xf[DM];
        row_f32(i, xf);
        float xn2 = 0.0f;
#pragma unroll
        for (int t = 0; t < DM; ++t) xn2 = __builtin_fmaf(xf[t], xf[t], xn2);
        // the cell's distances in fp32, each within 2^-19 of itself (fp32 and bf16 rows)
        float d1 = kFar, d2 = kFar;
        kk = kc;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float c[DM], D = 0.0f;
          codeword(kc + r, c);
#pragma unroll
          for (int t = 0; t < DM; ++t) {
            const float diff = xf[t] - c[t];
            D = __builtin_fmaf(diff, diff, D);
          }
          D = kc + r < K ? D : kFar;
          d2 = __builtin_amdgcn_fmed3f(d1, d2, D);
          kk = D < d1 ? kc + r : kk;
          d1 = fminf(d1, D);
        }
        if (src.type == ET_F64 || !(d2 > d1 * (1.0f + 0x1p-18f) + 1e-36f)) {  // too close in the cell: exactly
          double xd[DM];
          exact_row(i, xd);
          kk = kc;
          for (int r = 0; r < 4; ++r) {
            float c[DM];
            codeword(kc + r, c);
            const double D = distance(xd, c);
            if (r == 0) {
              D1 = D;
            } else if (kc + r < K && cless(D, kc + r, D1, kk)) {
              D1 = D;
              kk = kc + r;
            }
          }
          d1 = static_cast<float>(D1);
        } else if (want_dist) {
          double xd[DM];
          float c[DM];
#pragma unroll
          for (int t = 0; t < DM; ++t) xd[t] = static_cast<double>(xf[t]);
          codeword(kk, c);
          D1 = distance(xd, c);
        }
        // ||x||, sqrt(D) and D from above in fp32 (the hardware root within one ulp); the bound's terms in
        // (R + ||x||)^2 cover the roundings of this comparison too.  Past fp32's range R^2 is not below the
        // limit and the row goes to the exact search (a codeword whose norm overflows is screened out;
        // none can win while R^2 is far below).
        const float up = d1 * (1.0f + 0x1p-18f);
        const float xn = __builtin_amdgcn_sqrtf(xn2) * (1.0f + 0x1p-18f) + 1e-18f;
        const float R = xn + __builtin_amdgcn_sqrtf(up) * (1.0f + 0x1p-18f) + 1e-18f;
        const float delta = (acc_ulps * 0x1p-24f * (R + xn) * (R + xn) + split_coef * xn * R) * (1.0f + 0x1p-18f) +
                            0x1p-118f * (xn + R + 1.0f) + 1e-35f;
        certain = has && R * R < 1.0e38f && (s2 >= 1.0e38f || up < s2 + xn2 - delta);
      }
      uint64_t todo = __ballot(live && !certain);
      while (todo) {
        const int l = __ffsll(static_cast<long long>(todo)) - 1;
        todo &= todo - 1;
        const int64_t il = __builtin_amdgcn_readlane(static_cast<int>(i), l);  // vector counts are below 2^31
        double x[DM];
        exact_row(il, x);
        uint64_t bD = kInfBits;
        int bk = INT_MAX;
        for (int k = lane; k < K; k += 64) {
          float c[DM];
          codeword(k, c);
          const uint64_t D = order_bits(distance(x, c));
          if (D < bD || (D == bD && k < bk)) {
            bD = D;
            bk = k;
          }
        }
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
          const uint64_t oD = __shfl_xor(bD, m);
          const int ok = __shfl_xor(bk, m);
          if (oD < bD || (oD == bD && ok < bk)) {
            bD = oD;
            bk = ok;
          }
        }
        if (lane == l) {
          D1 = __builtin_bit_cast(double, bD);
          kk = bk;
        }
      }
      if (live) {
        // no codeword compared below +inf (a NaN element): code 0, distance NaN (as a bit pattern: this
        // file is compiled without NaN semantics)
        const bool none = kk == INT_MAX;
        const int k = none ? 0 : kk;
        if (codes) {
          codes[i] = k;
          if (dist) dist[i] = none ? __uint_as_float(0x7fc00000u) : static_cast<float>(D1);
        } else {
          rowD[i] = none ? __builtin_inf() : D1;
          rowK[i] = k;
        }
      }
    }
  }
}

// The packed form that applies to these rows and this codebook (0 when none does).
int packed_form(const RowSrc& src, const void* C, int ct, int d) {
  if (src.d != d || src.ld != src.vpr * d) return 0;
  const uintptr_t a = reinterpret_cast<uintptr_t>(src.base) | reinterpret_cast<uintptr_t>(C);
  if ((a & 15) != 0) return 0;
  if (src.type == ET_F32 && ct == ET_F32) return 1;
  if (src.type == ET_BF16 && ct == ET_BF16) return 2;
  return 0;
}

}  // namespace

hipError_t launch_assign_small(const RowSrc& src, const void* C, int ct, int64_t K, int32_t* codes, float* dist,
                               double* rowD, int* rowK, hipStream_t stream) {
  if (src.n <= 0) return hipSuccess;
  const int h = src.d > 8 ? 2 : 1, ft = packed_form(src, C, ct, 8 * h);
  // Rounding of the MFMA sums (96 2^-24 per 8 dimensions, measured far below), the cell number in the low
  // bits, the certificate's own fp32 roundings; the split remainder of each operand that is not bf16 already.
  const float acc_ulps = 96.0f * static_cast<float>(h) + 128.0f + 64.0f;
  const int inexact = (src.type != ET_BF16 ? 1 : 0) + (ct != ET_BF16 ? 1 : 0);
  const float split_coef = 0x1p-15f * static_cast<float>(inexact) * (1.0f + 0x1p-6f);
  // Rows per wave: 128 (64 at d > 8) when that still gives every SIMD two waves; a few rows' latency
  // decides below that.
  const int cb = src.n >= (1 << 18) ? (h == 1 ? 8 : 4) : src.n >= (1 << 15) ? 2 : 1;
  const int64_t blocks = cdiv(cdiv(src.n, 16 * cb), 4);
  const int64_t most = h == 1 ? 1280 : 1024;  // workgroups resident at once
  const dim3 grid(static_cast<unsigned>(blocks < most ? blocks : most));
#define CRVQ_SMALL(H, FT, CB)                                                                                      \
  hipLaunchKernelGGL((assign_small_kernel<H, FT, CB>), grid, dim3(256), 0, stream, src, C, ct, static_cast<int>(K), \
                     acc_ulps, split_coef, codes, dist, rowD, rowK)
#define CRVQ_SMALL_FT(H, CB)             \
  do {                                   \
    if (ft == 1)                         \
      CRVQ_SMALL(H, 1, CB);              \
    else if (ft == 2)                    \
      CRVQ_SMALL(H, 2, CB);              \
    else                                 \
      CRVQ_SMALL(H, 0, CB);              \
  } while (0)
  if (h == 1) {
    if (cb == 8)
      CRVQ_SMALL_FT(1, 8);
    else if (cb == 2)
      CRVQ_SMALL_FT(1, 2);
    else
      CRVQ_SMALL_FT(1, 1);
  } else {
    if (cb == 4)
      CRVQ_SMALL_FT(2, 4);
    else if (cb == 2)
      CRVQ_SMALL_FT(2, 2);
    else
      CRVQ_SMALL_FT(2, 1);
  }
#undef CRVQ_SMALL_FT
#undef CRVQ_SMALL
  return hipGetLastError();
}

}  // namespace crvq
