// One step of the residual beam search against a codebook of at most 256 codewords (d <= 8, beam <= 8)
// in a single launch: screen, exact scores, selection of the children.
//
// A vector's candidates are its n_par parents' residuals against all K codewords; the n_next smallest
// keys (distance in fp64, parent rank, codeword) survive.  A wave takes 16 rows (16 / PP vectors of PP
// parent slots, PP a power of two) and keeps all their screen values in registers (SplitOps, 16 tiles of
// 16 codewords, 64 values per lane).  The screen's error for a codeword c is at most
//   a (||c|| + ||x||)^2 + b ||c|| ||x|| <= e (||c||^2 + ||x||^2),  e = 2 a + b / 2
// (a its roundings, b the split remainders).  The share of the codeword's own norm goes into the norm the
// screen starts from, ||c||^2 (1 - e), so that one long codeword does not widen the others' bounds: the
// screen value A gives
//   lower = A + (1 - e) ||x||^2 <= D <= (A + (1 + 5 e) ||x||^2) / (1 - 4 e) = upper,
// the second from D <= A + (1 + e) ||x||^2 + 2 e ||c||^2 and ||c||^2 <= 2 ||x||^2 + 2 D.  The n_next-th smallest
// upper bound U of a vector's 32 (64) groups of candidates is no less than its n_next-th smallest distance, so
// every survivor is among the candidates with lower <= U: about a dozen of 2048, which alone are scored
// exactly and ranked by their keys.  A vector with more than kCap of them (or a row the screen could not
// bound, as with a NaN) is searched exactly by its wave, in one pass over its candidates: vectors whose distances
// all tie (later books of zeros) cost about three times the others (4096 of them at width 8 81 us; 398 us with
// one pass per child).  Bound by VALU issue (about 1010 instructions per 16 rows,
// 74 % of the cycles).  The width-8 beam over three books of 256 for 286,208 vectors takes 0.66 ms; with
// per-parent top-8 lists, their re-scored tiles (40 codewords per parent row) and a merge through memory
// it took 2.27 ms.  Residuals are formed from the vector and the parent's
// codewords (the same subtractions in the same order), so a step reads and writes codes only.
#include <climits>

#include "screen_common.h"

namespace crvq {
namespace {

struct BeamBooks {
  const void* C[kMaxBooks];
  int type[kMaxBooks];
};

// Factors of the bounds above: the codewords' norms, ||x||^2 and the whole of the upper bound, ||x||^2 of the
// lower one.
struct BeamBound {
  float cn, up, up_d, low;
};

// An aligned pair of fp32 or bf16 elements as raw words: fp32 both of them, bf16 the same word twice.
struct RawPair {
  uint32_t a, b;
  __device__ __forceinline__ void load(const void* base, bool bf16, int64_t e) {
    const uint32_t* q = reinterpret_cast<const uint32_t*>(static_cast<const char*>(base) + (bf16 ? 2 * e : 4 * e));
    a = q[0];
    b = q[bf16 ? 0 : 1];
  }
  __device__ __forceinline__ double first(bool bf16) const {
    return static_cast<double>(__uint_as_float(bf16 ? a << 16 : a));
  }
  __device__ __forceinline__ double second(bool bf16) const {
    return static_cast<double>(__uint_as_float(bf16 ? b & 0xffff0000u : b));
  }
};
constexpr float kBmFar = 1.0e37f;   // ||x||^2 and distances the screen may handle
constexpr float kBmTiny = 2.0e-35f;  // products below the operands' normal range
constexpr int kBmAhead = 3;  // earlier books whose codewords are loaded one pass ahead

constexpr int kBmWaves = 4;
constexpr int kBmCand = 528;  // candidate slots per wave (16 vectors of 32, 8 or fewer of 64, each list one longer)

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The value of lane ^ MASK, by DPP or a row swap.  MASK 4: of the mirrored lane of eight, which holds the same
// list once those of lanes ^ 1 and ^ 2 are merged.
template <int MASK>
__device__ __forceinline__ float exchange(float v) {
  const int u = __float_as_int(v);
  if constexpr (MASK == 1) return __int_as_float(__builtin_amdgcn_mov_dpp(u, 0xB1, 0xf, 0xf, false));
  if constexpr (MASK == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(u, 0x4E, 0xf, 0xf, false));
  if constexpr (MASK == 4) return __int_as_float(__builtin_amdgcn_mov_dpp(u, 0x141, 0xf, 0xf, false));
  if constexpr (MASK == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(u), static_cast<uint32_t>(u), false, false);
    return __uint_as_float((threadIdx.x & 16) ? r[0] : r[1]);
  }
  if constexpr (MASK == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(u), static_cast<uint32_t>(u), false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
  }
}

__device__ __forceinline__ void order2(float& a, float& b) {
  const float lo = fminf(a, b), hi = fmaxf(a, b);
  a = lo;
  b = hi;
}
// Ascending order of a bitonic list of N.
template <int N>
__device__ __forceinline__ void sort_bitonic(float (&l)[N]) {
#pragma unroll
  for (int w = N / 2; w >= 1; w >>= 1)
#pragma unroll
    for (int j = 0; j < N; ++j)
      if ((j & w) == 0) order2(l[j], l[j + w]);
}
// The ascending union of this lane's and lane ^ MASK's ascending lists.
template <int MASK, int N>
__device__ __forceinline__ void merge_grow(const float (&l)[N], float (&out)[2 * N]) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    out[j] = l[j];
    out[2 * N - 1 - j] = exchange<MASK>(l[j]);
  }
  sort_bitonic<2 * N>(out);
}
// The eight smallest of this lane's and lane ^ MASK's ascending lists, ascending.
template <int MASK>
__device__ __forceinline__ void merge_keep(float (&l)[8]) {
  float o[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = exchange<MASK>(l[7 - j]);
#pragma unroll
  for (int j = 0; j < 8; ++j) l[j] = fminf(l[j], o[j]);
  sort_bitonic<8>(l);
}

template <int N>
__device__ __forceinline__ void sort_small(float (&l)[N]) {
  if constexpr (N == 2) {
    order2(l[0], l[1]);
  } else if constexpr (N > 2) {
    float a[N / 2], b[N / 2];
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
      a[j] = l[j];
      b[j] = l[N / 2 + j];
    }
    sort_small<N / 2>(a);
    sort_small<N / 2>(b);
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
      l[j] = a[j];
      l[N - 1 - j] = b[j];
    }
    sort_bitonic<N>(l);
  }
}

// Groups of screen values per lane: 32 per vector, 64 where a vector has eight parents (with 32, one vector
// in 700 had more than kCap candidates: its best children came from few parents).
template <int PP>
constexpr int kBmGroups = PP == 8 ? 2 : 8 / PP;

// The eight smallest upper bounds of a vector, ascending, from kBmGroups per lane over its PP parents'
// columns (lanes xor 1 .. PP / 2) and the four lane groups (xor 16, 32).
template <int PP>
__device__ __forceinline__ void vector_list(float (&u)[kBmGroups<PP>], float (&l)[8]) {
  sort_small<kBmGroups<PP>>(u);
  if constexpr (PP == 1) {
#pragma unroll
    for (int j = 0; j < 8; ++j) l[j] = u[j];
  } else if constexpr (PP == 2) {
    merge_grow<1>(u, l);
  } else {
    float a[4];
    merge_grow<1>(u, a);
    merge_grow<2>(a, l);
    if constexpr (PP == 8) merge_keep<4>(l);
  }
  merge_keep<16>(l);
  merge_keep<32>(l);
}

// The minimum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  v = min(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0xB1, 0xf, 0xf, false)));   // lane ^ 1
  v = min(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x4E, 0xf, 0xf, false)));   // lane ^ 2
  v = min(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x141, 0xf, 0xf, false)));  // other four of eight
  v = min(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x140, 0xf, 0xf, false)));  // other eight of 16
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = min(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return min(b[0], b[1]);
}

// The n_next (at most N) smallest keys (distance, parent rank, codeword) of one vector, rank r's in lane r (INT_MAX
// where no distance up to +inf is left).  Every lane walks its codewords of every parent once, in key order,
// and keeps the N smallest; the wave then takes the least head of its lists n_next times.
template <int N>
__device__ __forceinline__ void exact_children(const double (*xv)[10], const float (*cf)[8], int n_par, int K,
                                               int n_next, int lane, uint64_t& outD, int& outK) {
  uint64_t LD[N];
  int LK[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    LD[j] = kInfBits;
    LK[j] = INT_MAX;
  }
#pragma unroll 1
  for (int pp = 0; pp < n_par; ++pp) {
    double x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = xv[pp][t];
#pragma unroll N == 1 ? 4 : 1
    for (int k = lane; k < K; k += 64) {
      double D = 0.0;
#pragma unroll
      for (int t = 0; t < 8; ++t) {  // (zeros past d add nothing)
        const double diff = x[t] - static_cast<double>(cf[k][t]);
        D = D + diff * diff;
      }
      uint64_t b = order_bits(D);
      int key = (pp << 8) | k;
      // (an equal distance met later has the larger key; +inf itself still beats an empty slot)
      if (b < LD[N - 1] || (b == kInfBits && LK[N - 1] == INT_MAX)) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const bool lt = b < LD[j] || (b == LD[j] && key < LK[j]);
          const uint64_t tD = lt ? LD[j] : b;
          const int tk = lt ? LK[j] : key;
          LD[j] = lt ? b : LD[j];
          LK[j] = lt ? key : LK[j];
          b = tD;
          key = tk;
        }
      }
    }
  }
  outD = kInfBits;
  outK = INT_MAX;
#pragma unroll 1
  for (int s = 0; s < n_next; ++s) {
    const uint32_t hi = static_cast<uint32_t>(LD[0] >> 32), lo = static_cast<uint32_t>(LD[0]);
    const uint32_t mh = wave_min(hi);
    const uint32_t ml = wave_min(hi == mh ? lo : 0xffffffffu);
    const bool top = hi == mh && lo == ml;
    const uint32_t mk = wave_min(top ? static_cast<uint32_t>(LK[0]) : static_cast<uint32_t>(INT_MAX));
    if (lane == s) {
      outD = static_cast<uint64_t>(mh) << 32 | ml;
      outK = static_cast<int>(mk);
    }
    if (top && static_cast<uint32_t>(LK[0]) == mk) {  // keys are distinct: one lane (all of them when none is left)
#pragma unroll
      for (int j = 0; j + 1 < N; ++j) {
        LD[j] = LD[j + 1];
        LK[j] = LK[j + 1];
      }
      LD[N - 1] = kInfBits;
      LK[N - 1] = INT_MAX;
    }
  }
}

template <int PP, bool PAIRS>
__global__ __launch_bounds__(64 * kBmWaves, 3) void beam_small_kernel(RowSrc src, int64_t n, int n_par, int n_next,
                                                                  int step, int n_books, BeamBooks books, int K,
                                                                  BeamBound eb, const int* __restrict__ tup_in,
                                                                  int* __restrict__ tup_out, double* __restrict__ res_out,
                                                                  int last, CodePtrs outs, int64_t vpr,
                                                                  float* __restrict__ err_out) {
  constexpr int V = 16 / PP;          // vectors per wave and pass
  constexpr int GS = 4 * PP;          // lanes of a vector
  constexpr int kCap = V == 16 ? 32 : 64;
  constexpr int kCapStride = kCap + 1;  // the vectors' lists start on different banks
  static_assert(V * kCapStride <= kBmCand, "candidate lists");
  constexpr int S = kBmGroups<PP>;    // groups of screen values per lane
  __shared__ uint16_t apack[256 * 16];
  __shared__ float cn[256];
  __shared__ float cf[256][8];
  __shared__ double xr_s[kBmWaves][16][10];
  __shared__ double candD_s[kBmWaves][kBmCand];
  __shared__ int candK_s[kBmWaves][kBmCand];
  __shared__ int tup_s[kBmWaves][16][kMaxBooks];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int jl = lane & 15, g = lane >> 4, d = src.d;
  const void* C = books.C[step];
  const int ct = books.type[step];
  // the book packed by every workgroup for itself: split operands, norms, fp32 copy
  {
    const int k = tid;
    float c[8];
    load_codeword<8>(C, ct, k, d, k < K, c);
    float nrm = 0.0f;
    u16x8 hi, lo;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      nrm = nrm + c[t] * c[t];
      cf[k][t] = c[t];
      uint16_t h, l;
      bf16_split(c[t], h, l);
      hi[t] = h;
      lo[t] = l;
    }
    cn[k] = k < K ? nrm * eb.cn : __builtin_inff();
    reinterpret_cast<u16x8*>(apack)[2 * k] = hi;
    reinterpret_cast<u16x8*>(apack)[2 * k + 1] = lo;
  }
  __syncthreads();
  const int tiles = (K + 15) / 16;
  double(*xr)[10] = xr_s[wave];
  double* candD = candD_s[wave];
  int* candK = candK_s[wave];
  const int v = jl / PP, p = jl % PP, sub = p * 4 + g;
  const uint64_t vmask = (static_cast<uint64_t>((1u << PP) - 1u) << (v * PP)) * 0x0001000100010001ull;
  const uint64_t below = vmask & ((1ull << lane) - 1ull);
  double* myD = candD + v * kCapStride;
  int* myK = candK + v * kCapStride;
  const int64_t npass = (n + V - 1) / V, stride = static_cast<int64_t>(gridDim.x) * kBmWaves;
  int(*tq)[kMaxBooks] = tup_s[wave];
  // PAIRS: the rows of the next pass are loaded during this one, the parents' codes another pass ahead
  const bool xb = src.type == ET_BF16;
  const int ahead = step < kBmAhead ? step : kBmAhead;
  RawPair px, pc[kBmAhead];
  int qc[kBmAhead], qn[kBmAhead];
  auto load_codes = [&](int64_t ps, int(&q)[kBmAhead]) {
    const int64_t i = ps * V + v;
    const bool ok = i < n && p < n_par;
#pragma unroll
    for (int u = 0; u < kBmAhead; ++u) q[u] = (ok && u < ahead) ? tup_in[(i * n_par + p) * n_books + u] : 0;
  };
  auto load_pass = [&](int64_t ps, const int(&q)[kBmAhead]) {
    const int64_t i = ps * V + v;
    const int e = 2 * g < d ? 2 * g : 0;  // a pair past d is not used
    px.load(src.base, xb, (i < n && p < n_par ? row_offset(src, i) : 0) + e);
#pragma unroll
    for (int u = 0; u < kBmAhead; ++u)
      if (u < ahead) pc[u].load(books.C[u], books.type[u] == ET_BF16, static_cast<int64_t>(q[u]) * d + e);
  };
  const int64_t first = static_cast<int64_t>(blockIdx.x) * kBmWaves + wave;
  if (PAIRS && first < npass) {
    load_codes(first, qc);
    load_pass(first, qc);
    load_codes(first + stride, qn);
  }
  for (int64_t ps = first; ps < npass; ps += stride) {
    const int64_t i = ps * V + v;
    const bool row_ok = i < n && p < n_par;
    // the row: elements 2 g, 2 g + 1 by this lane, exchanged through LDS
    {
      const int* tp = tup_in + (i * n_par + p) * n_books;
      double e0, e1;
      int u = 0;
      if (PAIRS) {
        const bool in = row_ok && 2 * g < d;
        e0 = in ? px.first(xb) : 0.0;
        e1 = in ? px.second(xb) : 0.0;
#pragma unroll
        for (int w = 0; w < kBmAhead; ++w)
          if (w < ahead) {
            const bool bf = books.type[w] == ET_BF16;
            e0 = in ? e0 - pc[w].first(bf) : 0.0;
            e1 = in ? e1 - pc[w].second(bf) : 0.0;
            if (g == 0) tq[jl][w] = qc[w];
          }
        u = ahead;
      } else {
        const int64_t off = row_ok ? row_offset(src, i) : 0;
        e0 = (row_ok && 2 * g < d) ? row_elem(src, off, 2 * g) : 0.0;
        e1 = (row_ok && 2 * g + 1 < d) ? row_elem(src, off, 2 * g + 1) : 0.0;
      }
      for (; u < step; ++u) {
        const int q = row_ok ? tp[u] : 0;
        if (g == 0) tq[jl][u] = q;
        if (row_ok && 2 * g < d) e0 = e0 - cb_elem(books.C[u], books.type[u], q, d, 2 * g);
        if (row_ok && 2 * g + 1 < d) e1 = e1 - cb_elem(books.C[u], books.type[u], q, d, 2 * g + 1);
      }
      xr[jl][2 * g] = e0;
      xr[jl][2 * g + 1] = e1;
      if (PAIRS) {
        if (ps + stride < npass) load_pass(ps + stride, qn);
#pragma unroll
        for (int w = 0; w < kBmAhead; ++w) qc[w] = qn[w];
        load_codes(ps + 2 * stride, qn);
      }
    }
    wave_sync();
    float xf[8];
    double xn2 = 0.0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const double x = xr[jl][t];
      xn2 = xn2 + x * x;
      xf[t] = static_cast<float>(x);
    }
    const SplitOps::B bop = SplitOps::make_b_vals(xf, g);
    f4 acc[16];
    float tm[16];
#pragma unroll
    for (int T = 0; T < 16; ++T) {
      if (T < tiles) {
        SplitOps::A a;
        a.v = *reinterpret_cast<const bf8*>(apack + (T * 16 + jl) * 16 + (lane >> 5) * 8);
        acc[T] = SplitOps::mfma(a, bop, *reinterpret_cast<const f4*>(cn + T * 16 + 4 * g));
      } else {
        acc[T] = f4{__builtin_inff(), __builtin_inff(), __builtin_inff(), __builtin_inff()};
      }
    }
#pragma unroll
    for (int T = 0; T < 16; ++T) tm[T] = fminf(fminf(acc[T][0], acc[T][1]), fminf(acc[T][2], acc[T][3]));
    const float xn2f = static_cast<float>(xn2);
    // past this a norm or a sum of the screen may leave fp32's range: the vector is searched exactly
    const bool far = row_ok && !(xn2f < kBmFar);
    const float xu = xn2f + (eb.up * xn2f + kBmTiny), xl = (eb.low * xn2f + kBmTiny) - xn2f;
    float u[S], best[8];  // the upper bounds but for their common factor
#pragma unroll
    for (int s = 0; s < S; ++s) {
      float m = __builtin_inff();
#pragma unroll
      for (int T = s * (16 / S); T < (s + 1) * (16 / S); ++T) m = fminf(m, tm[T]);
      u[s] = row_ok ? m + xu : __builtin_inff();
    }
    vector_list<PP>(u, best);
    float U = best[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) U = j < n_next ? best[j] : U;
    U *= eb.up_d;
    // lower <= U; a padding codeword (+inf) never is
    const float thr = row_ok ? fminf(U + xl, 3.0e38f) : -3.0e38f;
    // each lane's hits as bits (value 0 of a half in the highest), then one list entry per lane and round
    int cnt = 0;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      uint32_t hits = 0;
#pragma unroll
      for (int e = 0; e < 32; ++e) hits = hits + hits + (acc[8 * half + e / 4][e % 4] <= thr ? 1u : 0u);
      for (;;) {
        const uint64_t m = __ballot(hits != 0);
        if (m == 0) break;
        const int e = __clz(static_cast<int>(hits | 1u));
        const int at = cnt + __popcll(m & below);
        if (hits != 0 && at < kCap) myK[at] = (p << 8) | (128 * half + 16 * (e >> 2) + 4 * g + (e & 3));
        hits &= 0x7fffffffu >> e;
        cnt += __popcll(m & vmask);
      }
    }
    wave_sync();
    const bool sure = U < kBmFar && (__ballot(far) & vmask) == 0;  // (U is +inf where a small book fills few groups)
    const bool fits = cnt <= kCap && cnt >= n_next && (sure || cnt == n_par * K);
    // a child: its codes, residual and error
    auto child = [&](int64_t iv, int vv, int rank, int pp, int k, double D, bool none) {
      if (last) {
        // vector counts are below 2^31
        const uint32_t r = static_cast<uint32_t>(iv) / static_cast<uint32_t>(vpr);
        const uint32_t gg = static_cast<uint32_t>(iv) - r * static_cast<uint32_t>(vpr);
        for (int t = 0; t < step; ++t) outs.q[t][r * outs.ld[t] + gg] = tq[vv * PP + pp][t];
        outs.q[step][r * outs.ld[step] + gg] = k;
        if (err_out) err_out[iv] = static_cast<float>(D);
      } else {
        int* to = tup_out + (iv * n_next + rank) * n_books;
        for (int t = 0; t < step; ++t) to[t] = tq[vv * PP + pp][t];
        to[step] = k;
        if (res_out) {
          double* ro = res_out + (iv * n_next + rank) * d;
          for (int t = 0; t < d; ++t) ro[t] = none ? 0.0 : xr[vv * PP + pp][t] - static_cast<double>(cf[k][t]);
        }
      }
    };
    auto exact = [&](int row, int k) {
      double D = 0.0;
#pragma unroll
      for (int t = 0; t < 8; ++t) {  // (zeros past d add nothing)
        const double diff = xr[row][t] - static_cast<double>(cf[k][t]);
        D = D + diff * diff;
      }
      return D;
    };
    const int mine = fits ? cnt : 0;
    for (int c = sub; c < mine; c += GS) {
      const int key = myK[c];
      myD[c] = exact(v * PP + (key >> 8), key & 255);
    }
    wave_sync();
    for (int c = sub; c < mine; c += GS) {
      const int key = myK[c];
      const double D = myD[c];
      int rank = 0;
#pragma unroll 4
      for (int j = 0; j < mine; ++j) {
        const double Dj = myD[j];
        const int kj = myK[j];
        rank += ((Dj < D) | ((Dj == D) & (kj < key))) ? 1 : 0;
      }
      if (rank < n_next) child(i, v, rank, key >> 8, key & 255, D, false);
    }
    // the other vectors one by one, all candidates by the whole wave; then their children at once
    const uint64_t slow = __ballot(i < n && !fits);
    if (slow) {
      for (uint64_t todo = slow; todo;) {
        const int vv = ((__ffsll(static_cast<long long>(todo)) - 1) & 15) / PP;
        todo &= ~((static_cast<uint64_t>((1u << PP) - 1u) << (vv * PP)) * 0x0001000100010001ull);
        uint64_t D;
        int key;
        if (n_next == 1)
          exact_children<1>(xr + vv * PP, cf, n_par, K, 1, lane, D, key);
        else
          exact_children<8>(xr + vv * PP, cf, n_par, K, n_next, lane, D, key);
        if (lane < n_next) {
          candD[vv * 8 + lane] = __builtin_bit_cast(double, D);
          candK[vv * 8 + lane] = key;
        }
      }
      wave_sync();
      for (int j = lane; j < V * 8; j += 64) {
        const int vv = j >> 3, s = j & 7, key = candK[j];
        if (s >= n_next || ((slow >> (vv * PP)) & 1) == 0) continue;
        const bool none = key == INT_MAX;  // no distance left up to +inf (a NaN row): a defined child
        child(ps * V + vv, vv, s, none ? 0 : key >> 8, none ? 0 : key & 255, candD[j], none);
      }
    }
    wave_sync();  // the next pass overwrites the rows and the candidates
  }
}

}  // namespace

bool beam_small_form(int d, int64_t K, int64_t n_par, int beam) { return d <= 8 && K <= 256 && n_par <= 8 && beam <= 8; }

hipError_t launch_beam_small(const RowSrc& src0, int n_par, int n_next, int step, int n_books, const void* const* C,
                             const int* types, int64_t K, const int* tup_in, int* tup_out, double* res_out, bool last,
                             const CodePtrs& outs, int64_t vpr, float* err_out, hipStream_t stream) {
  if (src0.n <= 0) return hipSuccess;
  BeamBooks b = {};
  for (int t = 0; t < n_books; ++t) {
    b.C[t] = C[t];
    b.type[t] = types[t];
  }
  // a = 112 roundings of the screen (screen_bound's 96 and those of the scaled norms), b the split remainder of
  // each operand that is not bf16 already
  const int inexact = (step > 0 || src0.type != ET_BF16 ? 1 : 0) + (types[step] != ET_BF16 ? 1 : 0);
  const float ec = 2.0f * 112.0f * 0x1p-24f + 0.5f * 0x1p-15f * static_cast<float>(inexact) * (1.0f + 0x1p-6f);
  const BeamBound eb = {1.0f - ec, 5.0f * ec + 0x1p-20f, 1.0f + 4.25f * ec + 0x1p-20f, ec + 0x1p-20f};
  const int pp = n_par <= 1 ? 1 : n_par <= 2 ? 2 : n_par <= 4 ? 4 : 8;
  const int64_t passes = cdiv(src0.n, 16 / pp), blocks = cdiv(passes, kBmWaves);
  const dim3 grid(static_cast<unsigned>(blocks < 768 ? blocks : 768));
  // pairs of elements at even offsets from bases aligned to a pair
  auto aligned = [](const void* q, int type) { return reinterpret_cast<uintptr_t>(q) % (type == ET_BF16 ? 4 : 8) == 0; };
  bool pairs = src0.d % 2 == 0 && src0.ld % 2 == 0 && aligned(src0.base, src0.type);
  for (int t = 0; t < step; ++t) pairs = pairs && aligned(C[t], types[t]);
#define CRVQ_BEAM2(PPV, PR)                                                                                          \
  hipLaunchKernelGGL((beam_small_kernel<PPV, PR>), grid, dim3(64 * kBmWaves), 0, stream, src0, src0.n, n_par, n_next, step, \
                     n_books, b, static_cast<int>(K), eb, tup_in, tup_out, res_out, last ? 1 : 0, outs, vpr, err_out)
#define CRVQ_BEAM(PPV)     \
  if (pairs)               \
    CRVQ_BEAM2(PPV, true); \
  else                     \
    CRVQ_BEAM2(PPV, false)
  switch (pp) {
    case 1: CRVQ_BEAM(1); break;
    case 2: CRVQ_BEAM(2); break;
    case 4: CRVQ_BEAM(4); break;
    default: CRVQ_BEAM(8); break;
  }
#undef CRVQ_BEAM
#undef CRVQ_BEAM2
  return hipGetLastError();
}

}  // namespace crvq
