// Row and codeword access, and the split-bf16 operands of the 16 x 16 screen, shared by the search kernels.
#pragma once

#include "crvq_internal.h"

namespace crvq {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // at any element
typedef uint32_t u2u __attribute__((ext_vector_type(2), aligned(2)));  // at any bf16 element

__device__ __forceinline__ float bf16_to_f(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

__device__ __forceinline__ int64_t row_offset(const RowSrc& s, int64_t i) {
  if (s.type == ET_F64 || s.ld == s.vpr * s.d) return i * s.d;  // rows packed back to back
  // a column slab: 32-bit division (vector counts are below 2^31)
  const uint32_t r = static_cast<uint32_t>(i) / static_cast<uint32_t>(s.vpr);
  const uint32_t g = static_cast<uint32_t>(i) - r * static_cast<uint32_t>(s.vpr);
  return static_cast<int64_t>(r) * s.ld + static_cast<int64_t>(g) * s.d;
}

__device__ __forceinline__ double row_elem(const RowSrc& s, int64_t off, int t) {
  if (s.type == ET_F32) return static_cast<double>(static_cast<const float*>(s.base)[off + t]);
  if (s.type == ET_BF16) return static_cast<double>(bf16_to_f(static_cast<const uint16_t*>(s.base)[off + t]));
  return static_cast<const double*>(s.base)[off + t];
}

__device__ __forceinline__ double cb_elem(const void* C, int type, int64_t k, int d, int t) {
  if (type == ET_F32) return static_cast<double>(static_cast<const float*>(C)[k * d + t]);
  return static_cast<double>(bf16_to_f(static_cast<const uint16_t*>(C)[k * d + t]));
}

// DM fp32 / bf16 elements at p as floats, zero past d or when !ok.  Vector loads, which need no more than element
// alignment, when d fills DM, and for d = 4 .. 7 of 8: the first and the last four elements, which overlap, in one
// load each (with element loads the winners' 64 codewords, which the 32 x 32 screen scores exactly, cost more
// than its products save under 5000 codewords: d = 7, K = 3072 x 1 M rows 464 us, 300 so, 333 on 16 x 16 tiles).
// Element loads otherwise.
__device__ __forceinline__ void spread_tail(int d, const f4& b, float& v4, float& v5, float& v6, float& v7) {
  v4 = d == 5 ? b[3] : d == 6 ? b[2] : d == 7 ? b[1] : 0.0f;
  v5 = d == 6 ? b[3] : d == 7 ? b[2] : 0.0f;
  v6 = d == 7 ? b[3] : 0.0f;
  v7 = 0.0f;
}
template <int DM>
__device__ __forceinline__ void load_f32_elems(const float* p, int d, bool ok, float (&v)[DM]) {
  const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  if (DM % 4 == 0 && d == DM) {
#pragma unroll
    for (int q = 0; q < DM / 4; ++q) {
      const f4 w = ok ? reinterpret_cast<const f4u*>(p)[q] : zero;
#pragma unroll
      for (int t = 0; t < 4; ++t) v[4 * q + t] = w[t];
    }
  } else if (DM == 8 && d >= 4) {
    const f4 a = ok ? *reinterpret_cast<const f4u*>(p) : zero, b = ok ? *reinterpret_cast<const f4u*>(p + d - 4) : zero;
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = a[t];
    spread_tail(d, b, v[4 % DM], v[5 % DM], v[6 % DM], v[7 % DM]);
  } else {
#pragma unroll
    for (int t = 0; t < DM; ++t) v[t] = (DM != 8 || t < 3) && ok && t < d ? p[t] : 0.0f;
  }
}

__device__ __forceinline__ f4 widen4(const u2u& w) {
  return f4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16),
            __uint_as_float(w[1] & 0xffff0000u)};
}
template <int DM>
__device__ __forceinline__ void load_bf16_elems(const uint16_t* p, int d, bool ok, float (&v)[DM]) {
  const u2u zero = {0u, 0u};
  if (DM % 4 == 0 && d == DM) {
#pragma unroll
    for (int q = 0; q < DM / 4; ++q) {
      const f4 w = widen4(ok ? reinterpret_cast<const u2u*>(p)[q] : zero);
#pragma unroll
      for (int t = 0; t < 4; ++t) v[4 * q + t] = w[t];
    }
  } else if (DM == 8 && d >= 4) {
    const u2u a = ok ? *reinterpret_cast<const u2u*>(p) : zero, b = ok ? *reinterpret_cast<const u2u*>(p + d - 4) : zero;
    const f4 w = widen4(a);
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = w[t];
    spread_tail(d, widen4(b), v[4 % DM], v[5 % DM], v[6 % DM], v[7 % DM]);
  } else {
#pragma unroll
    for (int t = 0; t < DM; ++t) v[t] = (DM != 8 || t < 3) && ok && t < d ? bf16_to_f(p[t]) : 0.0f;
  }
}

// The first DM elements of row i in fp64 (zero past d or for an invalid row).  The type is
// dispatched once and every load is issued before any is used.
template <int DM>
__device__ __forceinline__ void load_row_exact(const RowSrc& s, int64_t i, bool valid, double (&x)[DM]) {
  const int d = s.d;
  const int64_t off = valid ? row_offset(s, i) : 0;
  if (s.type == ET_F64) {
    const double* p = static_cast<const double*>(s.base) + off;
#pragma unroll
    for (int t = 0; t < DM; ++t) x[t] = (valid && t < d) ? p[t] : 0.0;
    return;
  }
  float v[DM];
  if (s.type == ET_F32)
    load_f32_elems<DM>(static_cast<const float*>(s.base) + off, d, valid, v);
  else
    load_bf16_elems<DM>(static_cast<const uint16_t*>(s.base) + off, d, valid, v);
#pragma unroll
  for (int t = 0; t < DM; ++t) x[t] = static_cast<double>(v[t]);
}

// Codeword k as float (exact for fp32 and bf16 books), zero past d or when !ok.
template <int DM>
__device__ __forceinline__ void load_codeword(const void* C, int ct, int64_t k, int d, bool ok, float (&c)[DM]) {
  if (ct == ET_F32)
    load_f32_elems<DM>(static_cast<const float*>(C) + (ok ? k * d : 0), d, ok, c);
  else
    load_bf16_elems<DM>(static_cast<const uint16_t*>(C) + (ok ? k * d : 0), d, ok, c);
}

// A distance (never below zero) as an integer of the same order; a NaN comes after +inf, also in files
// compiled without NaN semantics.
__device__ __forceinline__ uint64_t order_bits(double D) { return __builtin_bit_cast(uint64_t, D); }
constexpr uint64_t kInfBits = 0x7ff0000000000000ull;

__device__ __forceinline__ bool cless(double Da, int ka, double Db, int kb) {
  return Da < Db || (Da == Db && ka < kb);
}

// fp32 to bf16, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t bf16_rn_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// Two-term bf16 split of v: hi = bf16(v), lo = bf16(v - hi) (v - hi is exact in fp32), so that
// |v - hi - lo| <= 2^-16 |v|.
__device__ __forceinline__ void bf16_split(float v, uint16_t& hi, uint16_t& lo) {
  hi = bf16_rn_bits(v);
  lo = bf16_rn_bits(v - __uint_as_float(static_cast<uint32_t>(hi) << 16));
}

typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));

// bf16 nearest-even of (a, b), a in the low half: one v_cvt_pk_bf16_f32, which rounds every finite
// fp32 value (subnormals included) to the same bits as bf16_rn_bits.
__device__ __forceinline__ uint32_t bf16x2_rn(float a, float b) {
  const f2v p = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(p, bf2v));
}

// The pair (a, b) of bf16_split: hi terms when !lo_term, else the lo terms.
__device__ __forceinline__ uint32_t bf16x2_split(float a, float b, bool lo_term) {
  const uint32_t h = bf16x2_rn(a, b);
  const uint32_t l = bf16x2_rn(a - __uint_as_float(h << 16), b - __uint_as_float(h & 0xffff0000u));
  return lo_term ? l : h;
}

// SplitOps (d <= 8): one v_mfma_f32_16x16x32_bf16 per tile.  Codewords and -2x are split into two
// bf16 terms (c = c1 + c2 + e_c, -2x = x1 + x2 + e_x, |e| <= 2^-16 |.|) and the four 8-element groups
// of the 32-long contraction hold c1.x1, c1.x2, c2.x1 and c2.x2: lane group g carries c1 (g < 2) or
// c2 (g >= 2) of codeword l % 16 and x1 (g even) or x2 (g odd) of row l % 16.  bf16 products are
// exact in fp32, so s is off by at most the split remainder 2^-15 sum_t |c_t| |2 x_t| plus the
// accumulation roundings; both enter the certification bound.  For bf16 rows and codebooks the split
// is exact (c2 = x2 = 0).
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct SplitOps {
  static constexpr int DM = 8;
  struct A {
    bf8 v;
  };
  struct B {
    bf8 v;
  };
  // codeword k of the packed book: 8 bf16 of c1, then 8 of c2 (32 bytes)
  __device__ static __forceinline__ A load_a(const void* apack, int64_t T, int lane) {
    A r;
    r.v = *reinterpret_cast<const bf8*>(static_cast<const uint16_t*>(apack) + (T * 16 + (lane & 15)) * 16 +
                                        (lane >> 5) * 8);
    return r;
  }
  __device__ static __forceinline__ B make_b(const RowSrc& src, int64_t i, bool ok, int g) {
    float v[8];
    if (src.type == ET_F64) {
      const int64_t off = ok ? row_offset(src, i) : 0;
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = (ok && t < src.d) ? static_cast<float>(row_elem(src, off, t)) : 0.0f;
    } else {
      const int64_t off = ok ? row_offset(src, i) : 0;
      if (src.type == ET_F32)
        load_f32_elems<8>(static_cast<const float*>(src.base) + off, src.d, ok, v);
      else
        load_bf16_elems<8>(static_cast<const uint16_t*>(src.base) + off, src.d, ok, v);
    }
    return make_b_vals(v, g);
  }
  // the B operand of lane group g from the row's first 8 elements (zero past d)
  __device__ static __forceinline__ B make_b_vals(const float (&v)[8], int g) {
    u32x4 h;
#pragma unroll
    for (int q = 0; q < 4; ++q) h[q] = bf16x2_split(-2.0f * v[2 * q], -2.0f * v[2 * q + 1], (g & 1) != 0);
    B b;
    b.v = __builtin_bit_cast(bf8, h);
    return b;
  }
  __device__ static __forceinline__ f4 mfma(const A& a, const B& b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
  }
};

}  // namespace
}  // namespace crvq
