// Loss-driven refinement of a quantized layer (the QuantLoss / FineTuneCodebook / BeamSearchOptimize
// loop of Alg. 1), on the layer in reordered channel order.  With H = X^T X (the paper's X X^T for
// activations stored tokens x N) and R = W - W_hat:
//   QuantLoss = ||W X^T - W_hat X^T||^2 = sum_r R_r H R_r^T,  dQuantLoss / dW_hat = -2 R H.
//
// Kernels:
//  * row_dot_kernel: the per-row loss sum_j R_rj G_rj in a fixed order.
//  * code_sum_wave_partial (K <= 256, d <= 8) or code_sum_partial, then code_sum_final: per-code sums
//    of fp64 vectors (the codebook gradient) in a fixed order -- per-wave LDS tables filled by ballot
//    peer groups, or one owner thread per code -- with the block partials folded in block order;
//    deterministic, no atomics.
//  * adam_kernel: one Adam step (moments in fp64, bias correction from the host) on an fp32 book.
//  * refine_block_kernel: the width-1 code search over a block of column groups (64 columns) for
//    every row, minimising QuantLoss with all other codes fixed; the running product S = R H is
//    updated in LDS inside the block and, for the later columns, by one product D H per block (D the
//    block's codeword changes).  One wave per row, eight rows per workgroup.
//  * refine_rows_kernel: the same for d = 8 and K <= 256, a row's state in its wave's registers.
#include "f64_tile.h"

namespace crvq {
namespace {

// out[r] = sum_{j < n} A[r * lda + j] * B[r * ldb + j]: strided per-thread sums, then a fixed tree.
__global__ __launch_bounds__(256) void row_dot_kernel(int64_t n, const double* __restrict__ A, int64_t lda,
                                                      const double* __restrict__ B, int64_t ldb,
                                                      double* __restrict__ out) {
  __shared__ double red[256];
  const int64_t r = blockIdx.x;
  double acc = 0.0;
  for (int64_t j = threadIdx.x; j < n; j += 256) acc = acc + A[r * lda + j] * B[r * ldb + j];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (static_cast<int>(threadIdx.x) < w) red[threadIdx.x] = red[threadIdx.x] + red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[r] = red[0];
}

// out[0] = sum_{i < n} x[i] (the layer's QuantLoss from its per-row terms): one block, strided
// per-thread sums in index order, then the same fixed tree.
__global__ __launch_bounds__(256) void sum_f64_kernel(int64_t n, const double* __restrict__ x,
                                                      double* __restrict__ out) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) acc = acc + x[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (static_cast<int>(threadIdx.x) < w) red[threadIdx.x] = red[threadIdx.x] + red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0];
}

// ---- per-code sums ------------------------------------------------------------------------------
constexpr int kCsVec = 256;      // vectors staged per round
constexpr int kCsMaxOwn = 4;     // codes per thread (K <= 1024)
constexpr int64_t kCsMaxK = 256 * kCsMaxOwn;  // larger books are grouped by a radix pass (k_kmeans.hip)

// Block b sums the vectors [b * per_block, ...) of a vector set over an fp64 matrix (vector
// v = r * vpr + g at element r * ld + g * d).  Thread t owns codes t, t + 256, ... and adds, in
// vector order, every staged vector whose code it owns.  part layout: [k * d + t][block].
__global__ __launch_bounds__(256) void code_sum_partial(const double* __restrict__ X, int64_t vpr, int64_t ld, int d,
                                                        int64_t n, const int32_t* __restrict__ codes, int K,
                                                        int64_t per_block, int64_t nblocks,
                                                        double* __restrict__ part, int* __restrict__ pcount) {
  __shared__ double sv[kCsVec * 16];
  __shared__ int sc[kCsVec];
  const int tid = threadIdx.x;
  const int64_t b0 = static_cast<int64_t>(blockIdx.x) * per_block;
  const int64_t b1 = b0 + per_block < n ? b0 + per_block : n;
  double acc[kCsMaxOwn][16];
  int cnt[kCsMaxOwn];
#pragma unroll
  for (int j = 0; j < kCsMaxOwn; ++j) {
    cnt[j] = 0;
#pragma unroll
    for (int t = 0; t < 16; ++t) acc[j][t] = 0.0;
  }
  for (int64_t base = b0; base < b1; base += kCsVec) {
    const int rn = static_cast<int>(b1 - base < kCsVec ? b1 - base : kCsVec);
    for (int v = tid; v < rn; v += 256) {
      const int64_t i = base + v;
      const int64_t r = i / vpr, g = i - r * vpr;
      const double* p = X + r * ld + g * d;
      for (int t = 0; t < d; ++t) sv[v * d + t] = p[t];
      const int c = codes[i];
      sc[v] = (c >= 0 && c < K) ? c : -1;
    }
    __syncthreads();
    for (int v = 0; v < rn; ++v) {
      const int c = sc[v];
      if (c >= 0 && (c & 255) == tid) {
        const int j = c >> 8;
#pragma unroll
        for (int jj = 0; jj < kCsMaxOwn; ++jj) {
          if (jj == j) {
            ++cnt[jj];
#pragma unroll
            for (int t = 0; t < 16; ++t)
              if (t < d) acc[jj][t] = acc[jj][t] + sv[v * d + t];
          }
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < kCsMaxOwn; ++j) {
    const int k = tid + 256 * j;
    if (k >= K) continue;
#pragma unroll
    for (int t = 0; t < 16; ++t)
      if (t < d) part[(static_cast<int64_t>(k) * d + t) * nblocks + blockIdx.x] = acc[j][t];
    pcount[static_cast<int64_t>(k) * nblocks + blockIdx.x] = cnt[j];
  }
}

// K <= 256, d <= 8: per-wave tables.  Every wave owns a private fp64 table of K x 8 sums in LDS and the
// batches of 64 vectors wave, wave + W, ... (W waves in the grid).  Within a batch the lanes that share
// a code find each other with eight ballots, and the lowest of them adds its peers' vectors (staged in
// LDS) in ascending lane order to that code's entry, so every entry is a fixed-order sum over the
// wave's batches; the block then folds its wave tables in wave order (layout [k * d + t][block]).
constexpr int kCwWaves = 6;   // waves per block: 6 tables of 21 KiB fit one CU's LDS
constexpr int kCwDepth = 2;   // batches in flight per wave

struct CwTable {
  double acc[256 * 8];
  int cnt[256];
  double stage[64][8];
};

__device__ __forceinline__ uint64_t code_peers(bool valid, int c) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const bool bit = (c >> b) & 1;
    const uint64_t m = __ballot(bit);
    peers &= bit ? m : ~m;
  }
  return valid ? peers : 0ull;
}

__device__ __forceinline__ void cw_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// vector i of the set as 8 doubles (zero past d); a lane outside the set reads vector 0
__device__ __forceinline__ void cw_load(const double* X, int64_t vpr, int64_t ld, int d, int64_t i, bool ok,
                                        double (&v)[8]) {
  const int64_t j = ok ? i : 0;
  const int64_t r = j / vpr, g = j - r * vpr;
  const double* p = X + r * ld + g * d;
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t] = t < d ? p[t] : 0.0;
}

__global__ __launch_bounds__(64 * kCwWaves) void code_sum_wave_partial(const double* __restrict__ X, int64_t vpr,
                                                                       int64_t ld, int d, int64_t n,
                                                                       const int32_t* __restrict__ codes, int K,
                                                                       int64_t nblocks, double* __restrict__ part,
                                                                       int* __restrict__ pcount) {
  __shared__ CwTable tab[kCwWaves];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  CwTable& T = tab[w];
  for (int e = lane; e < 256 * 8; e += 64) T.acc[e] = 0.0;
  for (int e = lane; e < 256; e += 64) T.cnt[e] = 0;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kCwWaves * 64;
  const int64_t w0 = (static_cast<int64_t>(blockIdx.x) * kCwWaves + w) * 64;
  double v[kCwDepth][8];
  int cq[kCwDepth];
#pragma unroll
  for (int s = 0; s < kCwDepth; ++s) {
    const int64_t i = w0 + stride * s + lane;
    const bool ok = i < n;
    cw_load(X, vpr, ld, d, i, ok, v[s]);
    cq[s] = codes[ok ? i : 0];
  }
  for (int64_t base = w0; base < n; base += stride * kCwDepth) {
#pragma unroll
    for (int s = 0; s < kCwDepth; ++s) {
      const int64_t bb = base + stride * s;
      if (bb < n) {  // uniform across the wave
        const int c = (bb + lane < n) ? cq[s] : -1;
        const bool valid = c >= 0 && c < K;
#pragma unroll
        for (int t = 0; t < 8; ++t) T.stage[lane][t] = v[s][t];
        cw_sync();
        const uint64_t peers = code_peers(valid, valid ? c : 0);
        if (valid && (__ffsll(static_cast<long long>(peers)) - 1) == lane) {
          double acc[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) acc[t] = T.acc[c * 8 + t];
          uint64_t m = peers;
          while (m) {
            const int sl = __ffsll(static_cast<long long>(m)) - 1;
            m &= m - 1;
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] = acc[t] + T.stage[sl][t];
          }
#pragma unroll
          for (int t = 0; t < 8; ++t) T.acc[c * 8 + t] = acc[t];
          T.cnt[c] += __popcll(peers);
        }
        cw_sync();
      }
      const int64_t i = bb + stride * kCwDepth + lane;
      const bool ok = i < n;
      cw_load(X, vpr, ld, d, i, ok, v[s]);
      cq[s] = codes[ok ? i : 0];
    }
  }
  __syncthreads();
  for (int e = tid; e < K * d; e += 64 * kCwWaves) {
    const int k = e / d, t = e - k * d;
    double acc = 0.0;
#pragma unroll
    for (int ww = 0; ww < kCwWaves; ++ww) acc = acc + tab[ww].acc[k * 8 + t];
    part[static_cast<int64_t>(e) * nblocks + blockIdx.x] = acc;
    if (t == 0) {
      int cnt = 0;
#pragma unroll
      for (int ww = 0; ww < kCwWaves; ++ww) cnt += tab[ww].cnt[k];
      pcount[static_cast<int64_t>(k) * nblocks + blockIdx.x] = cnt;
    }
  }
}

// One wave per sum element: lanes fold blocks lane, lane + 64, ... in order, then a fixed butterfly.
__global__ __launch_bounds__(256) void code_sum_final(const double* __restrict__ part, const int* __restrict__ pcount,
                                                      int64_t nblocks, int64_t K, int d, double* __restrict__ sums,
                                                      int32_t* __restrict__ counts) {
  const int lane = threadIdx.x & 63;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (e >= K * d) return;
  const int64_t k = e / d;
  const int t = static_cast<int>(e - k * d);
  double acc = 0.0;
  int cnt = 0;
  for (int64_t b = lane; b < nblocks; b += 64) {
    acc = acc + part[e * nblocks + b];
    cnt += pcount[k * nblocks + b];
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    acc = acc + __shfl_xor(acc, m);
    cnt += __shfl_xor(cnt, m);
  }
  if (lane == 0) {
    sums[e] = acc;
    if (counts && t == 0) counts[k] = cnt;
  }
}

// ---- Adam ---------------------------------------------------------------------------------------
// g = scale * grad; m = b1 m + (1 - b1) g; v = b2 v + (1 - b2) g^2; C -= lr * (m / bc1) / (sqrt(v / bc2) + eps)
// with the bias corrections bc1 = 1 - b1^t, bc2 = 1 - b2^t from the host; fp64 throughout, the
// codeword rounded once to fp32.  Each operation is rounded on its own (no contraction).
__global__ __launch_bounds__(256) void adam_kernel(int64_t n, float* __restrict__ C, const double* __restrict__ grad,
                                                   double scale, double* __restrict__ m, double* __restrict__ v,
                                                   double lr, double b1, double b2, double bc1, double bc2,
                                                   double eps) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  const double g = scale * grad[i];
  const double mi = b1 * m[i] + (1.0 - b1) * g;
  const double vi = b2 * v[i] + (1.0 - b2) * (g * g);
  m[i] = mi;
  v[i] = vi;
  const double mh = mi / bc1;
  const double vh = vi / bc2;
  C[i] = static_cast<float>(static_cast<double>(C[i]) - lr * mh / (sqrt(vh) + eps));
}

// The same step on an fp32 master of a bf16 codebook (set from the book at step 1), then the book as
// the master rounded to bf16, nearest-even (the master is finite here: rounding on its bits).
__global__ __launch_bounds__(256) void adam_bf16_kernel(int64_t n, uint16_t* __restrict__ C, float* __restrict__ master,
                                                        const double* __restrict__ grad, double scale,
                                                        double* __restrict__ m, double* __restrict__ v, double lr,
                                                        double b1, double b2, double bc1, double bc2, double eps,
                                                        int first) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  const float x0 = first ? __uint_as_float(static_cast<uint32_t>(C[i]) << 16) : master[i];
  const double g = scale * grad[i];
  const double mi = b1 * m[i] + (1.0 - b1) * g;
  const double vi = b2 * v[i] + (1.0 - b2) * (g * g);
  m[i] = mi;
  v[i] = vi;
  const double mh = mi / bc1;
  const double vh = vi / bc2;
  const float x = static_cast<float>(static_cast<double>(x0) - lr * mh / (sqrt(vh) + eps));
  master[i] = x;
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) != 0x7f800000u) u += 0x7fffu + ((u >> 16) & 1u);  // inf and NaN keep their bits
  C[i] = static_cast<uint16_t>(u >> 16);
}

// ---- width-1 code search, one block of column groups per launch ----------------------------------
constexpr int kRfRows = 8;      // rows per workgroup, one wave each
constexpr int kRfThreads = 64 * kRfRows;
constexpr int kRbCols = 64;     // columns per block (whole groups: 64 / d of them)

__device__ __forceinline__ double book_elem(const void* C, int type, int64_t i) {
  if (type == ET_F32) return static_cast<double>(static_cast<const float*>(C)[i]);
  return static_cast<double>(__uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t*>(C)[i]) << 16));
}

// The groups of columns [c0, c0 + bw) in order, for rows blockIdx.x * 8 + wave.  With s = (R H)_g, the
// loss change of moving a group's code from c0 to c_k is
//   c_k^T Hgg c_k - 2 c_k . (s + Hgg c_cur) - (the same at c_cur),
// so the row takes the k minimising f(k) = a_k - 2 c_k . b with a_k = c_k^T Hgg c_k and
// b = s + Hgg c_cur (lowest k on ties).  The block's H and the rows' (R H) on the block's columns are
// held in LDS; a moved row subtracts delta = c_k - c_cur from its residual and delta^T H[g rows, c] from
// its (R H) on the block's later columns, and writes delta (zero if unmoved) to D, from which one
// product D H updates the columns after the block.  A code outside [0, K) leaves the group unchanged.
template <int DMAX>
__global__ __launch_bounds__(kRfThreads) void refine_block_kernel(int64_t M, int d, int64_t c0, int bw,
                                                                 double* __restrict__ R, int64_t ldr,
                                                                 const double* __restrict__ S, int64_t lds,
                                                                 const double* __restrict__ H, int64_t ldh,
                                                                 const void* __restrict__ Cb, int c_type, int K,
                                                                 int32_t* __restrict__ codes, int64_t ldq,
                                                                 double* __restrict__ D, int64_t ldd) {
  extern __shared__ double sm[];
  double* Cs = sm;                      // K * d
  double* Ak = Cs + K * d;              // K
  double* Hb = Ak + K;                  // kRbCols x kRbCols
  double* sS = Hb + kRbCols * kRbCols;  // kRfRows x kRbCols
  __shared__ double s_b[kRfRows][16];
  __shared__ double s_delta[kRfRows][16];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kRfRows;
  const int64_t r = r0 + w;
  for (int e = tid; e < K * d; e += kRfThreads) Cs[e] = book_elem(Cb, c_type, e);
  for (int e = tid; e < bw * bw; e += kRfThreads) {
    const int i = e / bw, j = e - i * bw;
    Hb[i * kRbCols + j] = H[(c0 + i) * ldh + c0 + j];
  }
  for (int e = tid; e < kRfRows * bw; e += kRfThreads) {
    const int rr = e / bw, c = e - rr * bw;
    sS[rr * kRbCols + c] = (r0 + rr < M) ? S[(r0 + rr) * lds + c0 + c] : 0.0;
  }
  __syncthreads();
  const int ng = bw / d;
  for (int gi = 0; gi < ng; ++gi) {
    const int cg = gi * d;
    for (int k = tid; k < K; k += kRfThreads) {
      double a = 0.0;
      for (int t = 0; t < d; ++t) {
        double h = 0.0;
        for (int u = 0; u < d; ++u) h = h + Hb[(cg + t) * kRbCols + cg + u] * Cs[k * d + u];
        a = a + Cs[k * d + t] * h;
      }
      Ak[k] = a;
    }
    const int64_t gq = c0 / d + gi;
    const int cur = r < M ? codes[r * ldq + gq] : -1;
    const bool active = cur >= 0 && cur < K;
    if (active && lane < d) {  // b = s + Hgg c_cur, one lane per element
      double h = 0.0;
      for (int u = 0; u < d; ++u) h = h + Hb[(cg + lane) * kRbCols + cg + u] * Cs[cur * d + u];
      s_b[w][lane] = sS[w * kRbCols + cg + lane] + h;
    }
    __syncthreads();
    int moved = 0;
    if (active) {
      double b[DMAX];
#pragma unroll
      for (int t = 0; t < DMAX; ++t) b[t] = t < d ? s_b[w][t] : 0.0;
      double best = __builtin_inf();
      int bk = K;
#pragma unroll 1
      for (int k = lane; k < K; k += 64) {
        double dot = 0.0;
#pragma unroll
        for (int t = 0; t < DMAX; ++t)
          if (t < d) dot = dot + Cs[k * d + t] * b[t];
        const double f = Ak[k] - 2.0 * dot;
        if (f < best) {
          best = f;
          bk = k;
        }
      }
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) {
        const double ob = __shfl_xor(best, m);
        const int ok = __shfl_xor(bk, m);
        if (ob < best || (ob == best && ok < bk)) {
          best = ob;
          bk = ok;
        }
      }
      if (bk < K && bk != cur) {
        moved = 1;
        if (lane < d) {
          const double delta = Cs[bk * d + lane] - Cs[cur * d + lane];
          s_delta[w][lane] = delta;
          R[r * ldr + c0 + cg + lane] = R[r * ldr + c0 + cg + lane] - delta;
          D[r * ldd + cg + lane] = delta;
        }
        if (lane == 0) codes[r * ldq + gq] = bk;
      }
    }
    if (!moved && r < M && lane < d) D[r * ldd + cg + lane] = 0.0;
    __syncthreads();
    if (moved) {
      for (int c = cg + d + lane; c < bw; c += 64) {
        double acc = 0.0;
        for (int t = 0; t < d; ++t) acc = acc + s_delta[w][t] * Hb[(cg + t) * kRbCols + c];
        sS[w * kRbCols + c] = sS[w * kRbCols + c] - acc;
      }
    }
    __syncthreads();
  }
}

// ---- width-1 code search for d = 8 and K <= 256 ----------------------------------------------------
// The same search with the state of a row in one wave's registers, kRwCols columns per launch.  A lane
// keeps codewords lane, lane + 64, ... (K <= 256) and columns lane, lane + 64 of the row's R, S = R H and
// D; the block of H lies in LDS and a_k = c_k^T Hgg c_k comes from a table formed once per call, so a
// group costs a wave its scores (32 fused multiply-adds per row), an argmin on fp32-rounded keys (the
// exact values only where several codewords share the least key) and the update of its columns of S,
// with no barrier.  refine_block_kernel, which forms a_k in every workgroup and meets four barriers
// per group, took 93 us for 64 columns of 4096 rows; this one takes 40 us for 128: about 10 us until
// the block of H is in LDS and 2 us per group, where the fp64 issue of the four rows of a SIMD is half.
// RPW rows per wave share the codewords and the H reads and cover each other's latency.
constexpr int kRwCols = 128;            // columns per launch
constexpr int kRwOuter = 512;           // columns between two updates of all later columns of S
constexpr int kRwStride = kRwCols + 2;  // LDS row stride of H's block: 8 rows of a group on distinct banks
constexpr int kRwWaves = 8;
constexpr int kRwK = 256;
constexpr size_t kRwLds = (kRwCols * kRwStride + kRwK * 8) * sizeof(double);

bool refine_rows_form(int64_t K, int d) { return d == 8 && K <= kRwK; }

// a_k of every group (blockIdx.x) against every codeword; +inf past K, so that a padding codeword is
// never the minimum.
__global__ __launch_bounds__(kRwK) void refine_self_kernel(const double* __restrict__ H, int64_t ldh,
                                                           const void* __restrict__ Cb, int c_type, int K,
                                                           double* __restrict__ Aself) {
  __shared__ double Hg[64];
  const int k = threadIdx.x;
  const int64_t g = blockIdx.x;
  if (k < 64) Hg[k] = H[(g * 8 + k / 8) * ldh + g * 8 + k % 8];
  __syncthreads();
  double a = __builtin_inf();
  if (k < K) {
    double c[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) c[t] = book_elem(Cb, c_type, static_cast<int64_t>(k) * 8 + t);
    a = 0.0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      double h = 0.0;
#pragma unroll
      for (int u = 0; u < 8; ++u) h = h + Hg[t * 8 + u] * c[u];
      a = a + c[t] * h;
    }
  }
  Aself[g * kRwK + k] = a;
}

template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
// The minimum over the wave, in every lane.
__device__ __forceinline__ int wave_min_i32(int v) {
  v = min(v, dpp_i32<0xB1>(v));   // lane ^ 1
  v = min(v, dpp_i32<0x4E>(v));   // lane ^ 2
  v = min(v, dpp_i32<0x141>(v));  // the other four of eight
  v = min(v, dpp_i32<0x140>(v));  // the other eight of sixteen
  const auto a = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(v), static_cast<uint32_t>(v), false, false);
  v = min(static_cast<int>(a[0]), static_cast<int>(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(v), static_cast<uint32_t>(v), false, false);
  return min(static_cast<int>(b[0]), static_cast<int>(b[1]));
}
constexpr int kNoKey = 0x7fffffff;
constexpr int kMany = 9;  // equal rounded scores from which a wave reduces the exact ones instead of walking them
// f rounded to fp32, as an integer of the same order; kNoKey when that is +inf or NaN.
__device__ __forceinline__ int order_key(double f) {
  const float x = static_cast<float>(f);
  const int u = __float_as_int(x);
  const int key = u ^ ((u >> 31) & 0x7fffffff);
  return x < __builtin_inff() ? key : kNoKey;
}
template <int RPW>
__global__ __launch_bounds__(64 * kRwWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void refine_rows_kernel(int64_t M, int64_t c0, int bw, double* __restrict__ R,
                                                                   int64_t ldr, const double* __restrict__ S, int64_t lds,
                                                                   const double* __restrict__ H, int64_t ldh, int vec,
                                                                   const void* __restrict__ Cb, int c_type, int K,
                                                                   int32_t* __restrict__ codes, int64_t ldq,
                                                                   const double* __restrict__ Aself,
                                                                   double* __restrict__ D, int64_t ldd) {
  extern __shared__ double sm[];
  double* Hb = sm;                         // kRwCols x kRwStride
  double* Cs = Hb + kRwCols * kRwStride;   // kRwK x 8
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, ng = bw / 8;
  const int64_t r0 = (static_cast<int64_t>(blockIdx.x) * kRwWaves + w) * RPW, g0 = c0 / 8;
  // H's block on and right of the diagonal groups; the rest as zeros (those columns take no part, but
  // every lane updates its columns of S)
  if (vec && bw == kRwCols) {
    constexpr int kN = kRwCols * kRwCols / 2 / (64 * kRwWaves);
    const double2* src = reinterpret_cast<const double2*>(H + c0 * ldh + c0);
    double2 v[kN];
#pragma unroll
    for (int n = 0; n < kN; ++n) {
      const int i = (tid >> 6) + n * kRwWaves;
      v[n] = make_double2(0.0, 0.0);
      if (2 * lane >= (i & ~7)) v[n] = src[i * (ldh / 2) + lane];
    }
#pragma unroll
    for (int n = 0; n < kN; ++n)
      *reinterpret_cast<double2*>(&Hb[((tid >> 6) + n * kRwWaves) * kRwStride + 2 * lane]) = v[n];
  } else {
    for (int e = tid; e < kRwCols * kRwCols; e += 64 * kRwWaves) {
      const int i = e / kRwCols, j = e % kRwCols;
      Hb[i * kRwStride + j] = (i < bw && j < bw && j >= (i & ~7)) ? H[(c0 + i) * ldh + c0 + j] : 0.0;
    }
  }
  for (int e = tid; e < kRwK * 8; e += 64 * kRwWaves) Cs[e] = e < K * 8 ? book_elem(Cb, c_type, e) : 0.0;
  double s[RPW][2], rr[RPW][2], dd[RPW][2];
  int code[RPW];  // lane g: the code of group g
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int64_t r = r0 + i;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = lane + 64 * h;
      const bool in = r < M && c < bw;
      s[i][h] = in ? S[r * lds + c0 + c] : 0.0;
      rr[i][h] = in ? R[r * ldr + c0 + c] : 0.0;
      dd[i][h] = 0.0;
    }
    code[i] = (r < M && lane < ng) ? codes[r * ldq + g0 + lane] : -1;
  }
  __syncthreads();
  double c[4][8];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int t = 0; t < 8; ++t) c[j][t] = Cs[(lane + 64 * j) * 8 + t];
  const double* ap = Aself + g0 * kRwK + lane;
  const int t0 = lane & 7;
  double an[4];  // a_k of the next group
#pragma unroll
  for (int j = 0; j < 4; ++j) an[j] = ap[64 * j];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll 1
    for (int gi = 0; gi < 8; ++gi) {
      const int g = 8 * h + gi;
      if (g >= ng) break;
      double a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = an[j];
      const int gn = g + 1 < ng ? g + 1 : g;
#pragma unroll
      for (int j = 0; j < 4; ++j) an[j] = ap[gn * kRwK + 64 * j];
      __builtin_amdgcn_sched_barrier(0);
      // the rows go through every stage together, so that one's latency covers the other's
      int cur[RPW], now[RPW], key[RPW][4], best[RPW];
      bool valid[RPW];
      double cc[RPW][8], bt[RPW], b[RPW][8], f[RPW][4];
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        const int q = __builtin_amdgcn_readlane(code[i], g);
        valid[i] = static_cast<unsigned>(q) < static_cast<unsigned>(K);
        cur[i] = valid[i] ? q : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) cc[i][u] = Cs[cur[i] * 8 + u];
        bt[i] = s[i][h];
      }
      // b = s + Hgg c_cur, element t0 in the group's lane
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double hg = Hb[(8 * g + t0) * kRwStride + 8 * g + u];
#pragma unroll
        for (int i = 0; i < RPW; ++i) bt[i] = __builtin_fma(hg, cc[i][u], bt[i]);
      }
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int t = 0; t < 8; ++t) b[i][t] = lane_f64(bt[i], 8 * gi + t);
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) f[i][j] = c[j][0] * b[i][0];
#pragma unroll
      for (int t = 1; t < 8; ++t)
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) f[i][j] = __builtin_fma(c[j][t], b[i][t], f[i][j]);
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f[i][j] = __builtin_fma(-2.0, f[i][j], a[j]);  // a - 2 dot: the doubling is exact
          key[i][j] = order_key(f[i][j]);
        }
#pragma unroll
      for (int i = 0; i < RPW; ++i) best[i] = wave_min_i32(min(min(key[i][0], key[i][1]), min(key[i][2], key[i][3])));
      bool moved = false;
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        // the codewords whose rounded f is the least (rounding keeps the order, so the minimum is among
        // them); slot j holds 64 j .. 64 j + 63
        const int bi = __builtin_amdgcn_readfirstlane(best[i]);
        uint64_t m[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j] = __ballot(key[i][j] == bi);
        int bk = cur[i];
        const int least = bi == kNoKey ? kMany : __popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]);
        if (least == 1) {
#pragma unroll
          for (int j = 0; j < 4; ++j) bk = m[j] ? 64 * j + __ffsll(static_cast<long long>(m[j])) - 1 : bk;
        } else if (least >= kMany) {
          // many (a book of equal codewords), or f beyond fp32: every lane's own least, then the wave's, the
          // lowest codeword of equal ones; +inf and NaN never win
          double v = __builtin_inf();
          int k = kNoKey;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bool better = (bi == kNoKey || key[i][j] == bi) && f[i][j] < v;
            v = better ? f[i][j] : v;
            k = better ? 64 * j + lane : k;
          }
          int64_t o = __builtin_bit_cast(int64_t, v + 0.0);  // (no -0)
          o ^= (o >> 63) & 0x7fffffffffffffffll;
          const int hi = static_cast<int>(o >> 32), lo = static_cast<int>(static_cast<uint32_t>(o) ^ 0x80000000u);
          const int mh = wave_min_i32(hi), ml = wave_min_i32(hi == mh ? lo : kNoKey);
          const int mk = wave_min_i32(hi == mh && lo == ml ? k : kNoKey);
          bk = mk == kNoKey ? bk : mk;
        } else {
          // a few: the exact values in ascending codeword order
          double fb = __builtin_inf();
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            uint64_t mj = m[j];
            while (mj) {
              const int l = __ffsll(static_cast<long long>(mj)) - 1;
              mj &= mj - 1;
              const double v = lane_f64(f[i][j], l);
              if (v < fb) {
                fb = v;
                bk = 64 * j + l;
              }
            }
          }
        }
        now[i] = valid[i] ? __builtin_amdgcn_readfirstlane(bk) : cur[i];
        moved = moved || now[i] != cur[i];
      }
      if (!moved) continue;
      double de[RPW][8];
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        const double* cn = Cs + now[i] * 8;
#pragma unroll
        for (int u = 0; u < 8; ++u) de[i][u] = cn[u] - cc[i][u];
        const double dl = cn[t0] - Cs[cur[i] * 8 + t0];
        const bool mine = (lane >> 3) == gi;
        rr[i][h] = mine ? rr[i][h] - dl : rr[i][h];
        dd[i][h] = mine ? dl : dd[i][h];
        code[i] = (lane == g && valid[i]) ? now[i] : code[i];
      }
      // S of the columns after the group (those up to it are not read again)
#pragma unroll
      for (int hh = h; hh < 2; ++hh)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const double hb = Hb[(8 * g + u) * kRwStride + lane + 64 * hh];
#pragma unroll
          for (int i = 0; i < RPW; ++i) s[i][hh] = __builtin_fma(-de[i][u], hb, s[i][hh]);
        }
    }
  }
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int64_t r = r0 + i;
    if (r >= M) continue;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int cl = lane + 64 * h;
      if (cl < bw) {
        R[r * ldr + c0 + cl] = rr[i][h];
        D[r * ldd + cl] = dd[i][h];
      }
    }
    if (lane < ng) codes[r * ldq + g0 + lane] = code[i];
  }
}

// ---- the same search for books too large for one CU's LDS ------------------------------------------
// One group at a time over all rows: refine_scan_kernel finds, for 64 rows per workgroup and one slice
// of the codebook per grid row y, the k minimising f(k) = a_k - 2 c_k . b (the formulas and orders of
// refine_block_kernel, so the same values); refine_apply_kernel merges the slices (lowest k among equal
// values) and moves the rows' codes, updating R, D and the block's later columns of S = R H in memory.
constexpr int kRsRows = 64;      // rows per workgroup of the scan
constexpr int kRsTile = 256;     // codewords staged in LDS per round
constexpr int kRsMaxSlices = 8;  // codebook slices (grid y) at most

// Thread (rg, ks) = (tid % 16, tid / 16) scores rows 4 rg .. 4 rg + 3 against every sixteenth
// codeword of each staged round (so a codeword read from LDS serves four rows); the next round's
// codewords are loaded into registers while the current one is scored.
template <int DMAX>
__global__ __launch_bounds__(256) void refine_scan_kernel(int64_t M, int d, int64_t col, int64_t gq,
                                                          const double* __restrict__ S, int64_t lds,
                                                          const double* __restrict__ H, int64_t ldh,
                                                          const void* __restrict__ Cb, int c_type, int K, int slice,
                                                          const int32_t* __restrict__ codes, int64_t ldq,
                                                          double* __restrict__ bestF, int* __restrict__ bestK) {
  constexpr int kPer = kRsTile * DMAX / 256;  // staged elements per thread and round
  __shared__ double Hg[16 * 16];
  __shared__ double sb[kRsRows][16];
  __shared__ double Cs[kRsTile * DMAX];
  __shared__ double Ak[kRsTile];
  __shared__ double rf[16][kRsRows];
  __shared__ int rk[16][kRsRows];
  const int tid = threadIdx.x, rg = tid & 15, ks = tid >> 4;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kRsRows;
  const int k0 = static_cast<int>(blockIdx.y) * slice;
  const int k1 = k0 + slice < K ? k0 + slice : K;
  for (int e = tid; e < d * d; e += 256) Hg[e] = H[(col + e / d) * ldh + col + e % d];
  __syncthreads();
  // b = s + Hgg c_cur per row (a row with a code outside [0, K) takes no part)
  for (int e = tid; e < kRsRows * d; e += 256) {
    const int rr = e / d, t = e - rr * d;
    const int64_t r = r0 + rr;
    const int cur = r < M ? codes[r * ldq + gq] : -1;
    double v = 0.0;
    if (cur >= 0 && cur < K) {
      double h = 0.0;
      for (int u = 0; u < d; ++u) h = h + Hg[t * d + u] * book_elem(Cb, c_type, static_cast<int64_t>(cur) * d + u);
      v = S[r * lds + col + t] + h;
    }
    sb[rr][t] = v;
  }
  __syncthreads();
  double b[4][DMAX];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int t = 0; t < DMAX; ++t) b[q][t] = t < d ? sb[4 * rg + q][t] : 0.0;
  double best[4];
  int bk[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    best[q] = __builtin_inf();
    bk[q] = K;
  }
  // round kt's codewords as kPer elements per thread (element e = tid + 256 i of the round)
  double pf[kPer];
  auto fetch = [&](int kt) {
    const int64_t base = static_cast<int64_t>(kt) * d, lim = static_cast<int64_t>(k1) * d;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int64_t e = base + tid + 256 * i;
      pf[i] = e < lim ? book_elem(Cb, c_type, e) : 0.0;
    }
  };
  if (k0 < k1) fetch(k0);
  for (int kt = k0; kt < k1; kt += kRsTile) {
    const int tn = k1 - kt < kRsTile ? k1 - kt : kRsTile;
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (tid + 256 * i < tn * d) Cs[tid + 256 * i] = pf[i];
    __syncthreads();
    if (kt + kRsTile < k1) fetch(kt + kRsTile);  // in flight while this round is scored
    if (tid < tn) {  // a_k = c_k^T Hgg c_k
      double a = 0.0;
      for (int t = 0; t < d; ++t) {
        double h = 0.0;
        for (int u = 0; u < d; ++u) h = h + Hg[t * d + u] * Cs[tid * d + u];
        a = a + Cs[tid * d + t] * h;
      }
      Ak[tid] = a;
    }
    __syncthreads();
    for (int jj = ks; jj < tn; jj += 16) {
      double c[DMAX];
#pragma unroll
      for (int t = 0; t < DMAX; ++t) c[t] = t < d ? Cs[jj * d + t] : 0.0;
      const double a = Ak[jj];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double dot = 0.0;
#pragma unroll
        for (int t = 0; t < DMAX; ++t)
          if (t < d) dot = dot + c[t] * b[q][t];
        const double f = a - 2.0 * dot;
        if (f < best[q]) {
          best[q] = f;
          bk[q] = kt + jj;
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    rf[ks][4 * rg + q] = best[q];
    rk[ks][4 * rg + q] = bk[q];
  }
  __syncthreads();
  if (tid < kRsRows && r0 + tid < M) {
    double f0 = rf[0][tid];
    int k = rk[0][tid];
    for (int q = 1; q < 16; ++q)
      if (rf[q][tid] < f0 || (rf[q][tid] == f0 && rk[q][tid] < k)) {
        f0 = rf[q][tid];
        k = rk[q][tid];
      }
    bestF[static_cast<int64_t>(blockIdx.y) * M + r0 + tid] = f0;
    bestK[static_cast<int64_t>(blockIdx.y) * M + r0 + tid] = k;
  }
}

template <int DMAX>
__global__ __launch_bounds__(256) void refine_apply_kernel(int64_t M, int d, int64_t c0, int cg, int bw, int64_t gq,
                                                           double* __restrict__ R, int64_t ldr, double* __restrict__ S,
                                                           int64_t lds, const double* __restrict__ H, int64_t ldh,
                                                           const void* __restrict__ Cb, int c_type, int K,
                                                           int32_t* __restrict__ codes, int64_t ldq,
                                                           double* __restrict__ D, int64_t ldd, int nslice,
                                                           const double* __restrict__ bestF,
                                                           const int* __restrict__ bestK) {
  const int64_t r = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (r >= M) return;
  const int cur = codes[r * ldq + gq];
  double best = __builtin_inf();
  int bk = K;
  for (int sl = 0; sl < nslice; ++sl) {
    const double f = bestF[static_cast<int64_t>(sl) * M + r];
    const int k = bestK[static_cast<int64_t>(sl) * M + r];
    if (f < best || (f == best && k < bk)) {
      best = f;
      bk = k;
    }
  }
  const bool moved = cur >= 0 && cur < K && bk < K && bk != cur;
  double delta[DMAX];
#pragma unroll
  for (int t = 0; t < DMAX; ++t) {
    delta[t] = 0.0;
    if (t < d && moved)
      delta[t] = book_elem(Cb, c_type, static_cast<int64_t>(bk) * d + t) -
                 book_elem(Cb, c_type, static_cast<int64_t>(cur) * d + t);
  }
#pragma unroll
  for (int t = 0; t < DMAX; ++t)
    if (t < d) D[r * ldd + cg + t] = delta[t];
  if (!moved) return;
  codes[r * ldq + gq] = bk;
#pragma unroll
  for (int t = 0; t < DMAX; ++t)
    if (t < d) R[r * ldr + c0 + cg + t] = R[r * ldr + c0 + cg + t] - delta[t];
  for (int c = cg + d; c < bw; ++c) {
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < DMAX; ++t)
      if (t < d) acc = acc + delta[t] * H[(c0 + cg + t) * ldh + c0 + c];
    S[r * lds + c0 + c] = S[r * lds + c0 + c] - acc;
  }
}

}  // namespace

// ---- launchers -----------------------------------------------------------------------------------
hipError_t launch_row_dot(int64_t M, int64_t n, const double* A, int64_t lda, const double* B, int64_t ldb,
                          double* out, hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  hipLaunchKernelGGL(row_dot_kernel, dim3(static_cast<unsigned>(M)), dim3(256), 0, stream, n, A, lda, B, ldb, out);
  return hipGetLastError();
}

hipError_t launch_sum_f64(int64_t n, const double* x, double* out, hipStream_t stream) {
  hipLaunchKernelGGL(sum_f64_kernel, dim3(1), dim3(256), 0, stream, n, x, out);
  return hipGetLastError();
}

static int64_t code_sum_blocks(int64_t n) {
  const int64_t rounds = cdiv(n > 0 ? n : 1, kCsVec);
  return rounds < 1024 ? rounds : 1024;
}

// blocks of the per-wave scheme: at most one wave per batch of 64 vectors, 256 CUs' worth of waves
static int64_t code_sum_wave_blocks(int64_t n) {
  const int64_t batches = cdiv(n > 0 ? n : 1, 64);
  const int64_t waves = batches < 256 * kCwWaves ? batches : 256 * kCwWaves;
  return cdiv(waves, kCwWaves);
}

size_t code_sums_ws_bytes(int64_t n, int64_t K, int d) {
  if (K > kCsMaxK) return code_sums_large_ws_bytes(n, K);
  WsCursor c(nullptr);
  const int64_t nb = code_sum_blocks(n) > code_sum_wave_blocks(n) ? code_sum_blocks(n) : code_sum_wave_blocks(n);
  c.take<double>(static_cast<size_t>(nb * K * d));
  c.take<int>(static_cast<size_t>(nb * K));
  return c.used;
}

hipError_t launch_code_sums(const double* X, int64_t vpr, int64_t ld, int d, int64_t n, const int32_t* codes,
                            int64_t K, double* sums, int32_t* counts, void* ws, hipStream_t stream) {
  if (K > kCsMaxK) {
    RowSrc src;
    src.base = X;
    src.type = ET_F64;
    src.d = d;
    src.vpr = vpr;
    src.ld = ld;
    src.n = n;
    return launch_code_sums_large(src, codes, K, sums, counts, ws, stream);
  }
  if (K <= 256 && d <= 8 && n > 0) {
    WsCursor cw(ws);
    const int64_t nbw = code_sum_wave_blocks(n);
    const int64_t nbmax = code_sum_blocks(n) > nbw ? code_sum_blocks(n) : nbw;
    double* part = cw.take<double>(static_cast<size_t>(nbmax * K * d));
    int* pcount = cw.take<int>(static_cast<size_t>(nbmax * K));
    hipLaunchKernelGGL(code_sum_wave_partial, dim3(static_cast<unsigned>(nbw)), dim3(64 * kCwWaves), 0, stream, X, vpr,
                       ld, d, n, codes, static_cast<int>(K), nbw, part, pcount);
    hipLaunchKernelGGL(code_sum_final, dim3(static_cast<unsigned>(cdiv(K * d, 4))), dim3(256), 0, stream, part, pcount,
                       nbw, K, d, sums, counts);
    return hipGetLastError();
  }
  WsCursor cur(ws);
  int64_t nb = code_sum_blocks(n);
  const int64_t per_block = cdiv(cdiv(n > 0 ? n : 1, nb), kCsVec) * kCsVec;
  nb = cdiv(n > 0 ? n : 1, per_block);
  const int64_t nbmax = code_sum_blocks(n) > code_sum_wave_blocks(n) ? code_sum_blocks(n) : code_sum_wave_blocks(n);
  double* part = cur.take<double>(static_cast<size_t>(nbmax * K * d));
  int* pcount = cur.take<int>(static_cast<size_t>(nbmax * K));
  hipLaunchKernelGGL(code_sum_partial, dim3(static_cast<unsigned>(nb)), dim3(256), 0, stream, X, vpr, ld, d, n, codes,
                     static_cast<int>(K), per_block, nb, part, pcount);
  hipLaunchKernelGGL(code_sum_final, dim3(static_cast<unsigned>(cdiv(K * d, 4))), dim3(256), 0, stream, part, pcount,
                     nb, K, d, sums, counts);
  return hipGetLastError();
}

hipError_t launch_adam_bf16(int64_t n, uint16_t* C, float* master, const double* grad, double scale, double* m,
                            double* v, double lr, double b1, double b2, double bc1, double bc2, double eps, bool first,
                            hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(adam_bf16_kernel, dim3(static_cast<unsigned>(cdiv(n, 256))), dim3(256), 0, stream, n, C, master,
                     grad, scale, m, v, lr, b1, b2, bc1, bc2, eps, first ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_adam(int64_t n, float* C, const double* grad, double scale, double* m, double* v, double lr,
                       double b1, double b2, double bc1, double bc2, double eps, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(adam_kernel, dim3(static_cast<unsigned>(cdiv(n, 256))), dim3(256), 0, stream, n, C, grad, scale, m,
                     v, lr, b1, b2, bc1, bc2, eps);
  return hipGetLastError();
}

size_t refine_lds_bytes(int64_t K, int d) {
  return static_cast<size_t>(K * d + K + kRbCols * kRbCols + kRfRows * kRbCols) * sizeof(double);
}

namespace {
struct RefineWs {
  double* S;      // M x n_cols: R H on the book's columns
  double* D;      // M x (columns of an outer block): its codeword changes
  double* parts;  // the split parts of S
  double* bestF;  // large books: the slices' minima and codewords
  int* bestK;
  double* self;   // d = 8, K <= 256: a_k of every group
};
RefineWs carve_refine(WsCursor& c, int64_t M, int64_t n_cols, int64_t N) {
  RefineWs w;
  const size_t out = static_cast<size_t>(M) * static_cast<size_t>(n_cols);
  w.S = c.take<double>(out);
  w.D = c.take<double>(static_cast<size_t>(M) * kRwOuter);
  w.parts = c.take<double>(static_cast<size_t>(gemm_split_parts(M, n_cols, N)) * out);
  w.bestF = c.take<double>(static_cast<size_t>(kRsMaxSlices) * static_cast<size_t>(M));
  w.bestK = c.take<int>(static_cast<size_t>(kRsMaxSlices) * static_cast<size_t>(M));
  w.self = c.take<double>(static_cast<size_t>(n_cols / 8) * kRwK);
  return w;
}
}  // namespace

size_t refine_ws_bytes(int64_t M, int64_t n_cols, int64_t N) {
  WsCursor c(nullptr);
  (void)carve_refine(c, M, n_cols, N);
  return c.used;
}

// The codebook fits the block kernel's LDS (with H's block and the rows' S).
bool refine_book_in_lds(int64_t K, int d) { return K * d <= 8192 && refine_lds_bytes(K, d) + 4096 <= 160 * 1024; }

hipError_t launch_refine_book(int64_t M, int64_t N, int d, int64_t n_cols, double* R, int64_t ldr, const double* H,
                              int64_t ldh, const void* Cb, int c_type, int64_t K, int32_t* codes, int64_t ldq,
                              void* ws, hipStream_t stream) {
  if (M <= 0 || n_cols <= 0) return hipSuccess;
  WsCursor cur(ws);
  const RefineWs w = carve_refine(cur, M, n_cols, N);
  double *S = w.S, *D = w.D, *bestF = w.bestF;
  int* bestK = w.bestK;
  // S = R H[:, 0:n_cols]
  hipError_t e = launch_gemm_f64_split(M, n_cols, N, R, ldr, H, ldh, S, n_cols, w.parts, stream);
  if (e != hipSuccess) return e;
  const size_t lds = refine_lds_bytes(K, d);
  const dim3 grid(static_cast<unsigned>(cdiv(M, kRfRows)));
  // d = 8 against K <= 256 keeps the rows in registers (a 4096 x 4096 layer's basic book 10.6 -> 4.85 ms
  // with the products); other books that fit a CU's LDS are searched from it
  const bool rows_form = refine_rows_form(K, d);
  if (rows_form) {
    hipLaunchKernelGGL(refine_self_kernel, dim3(static_cast<unsigned>(n_cols / 8)), dim3(kRwK), 0, stream, H, ldh, Cb,
                       c_type, static_cast<int>(K), w.self);
  }
  const int rpw = M > 8 * 256 ? 2 : 1;  // two rows per wave once one per wave gives every CU its workgroup
  const dim3 grid_rows(static_cast<unsigned>(cdiv(M, kRwWaves * rpw)));
  const int64_t bw_max = rows_form ? kRwCols : (kRbCols / d) * d;
  const bool in_lds = refine_book_in_lds(K, d);
  // large books: enough codebook slices to give the scan about 512 workgroups
  const int64_t row_tiles = cdiv(M, kRsRows);
  int64_t nslice = cdiv(512, row_tiles);
  nslice = nslice < kRsMaxSlices ? nslice : kRsMaxSlices;
  nslice = nslice < cdiv(K, kRsTile) ? nslice : cdiv(K, kRsTile);
  const int slice = static_cast<int>(cdiv(cdiv(K, nslice), kRsTile) * kRsTile);
  nslice = cdiv(K, slice);
  // S takes a block's code changes D in two steps: right after the block on the columns of its outer
  // block, S[:, c0 + bw : o1] -= D_block H[block, c0 + bw : o1], and at the outer block's end on all later
  // columns, S[:, o1 :] -= D H[o0 : o1, o1 :], so that most of S moves once per outer block.
  const int64_t outer = rows_form ? kRwOuter : bw_max;
  const int vec = (ldh % 2 == 0 && reinterpret_cast<uintptr_t>(H) % 16 == 0) ? 1 : 0;
  for (int64_t c0 = 0; c0 < n_cols; c0 += bw_max) {
    const int bw = static_cast<int>(n_cols - c0 < bw_max ? n_cols - c0 : bw_max);
    const int64_t o0 = c0 / outer * outer, o1 = o0 + outer < n_cols ? o0 + outer : n_cols;
    double* Db = D + (c0 - o0);
    if (rows_form) {
      if (rpw == 2)
        hipLaunchKernelGGL(refine_rows_kernel<2>, grid_rows, dim3(64 * kRwWaves), kRwLds, stream, M, c0, bw, R, ldr, S,
                           n_cols, H, ldh, vec, Cb, c_type, static_cast<int>(K), codes, ldq, w.self, Db, outer);
      else
        hipLaunchKernelGGL(refine_rows_kernel<1>, grid_rows, dim3(64 * kRwWaves), kRwLds, stream, M, c0, bw, R, ldr, S,
                           n_cols, H, ldh, vec, Cb, c_type, static_cast<int>(K), codes, ldq, w.self, Db, outer);
    } else if (!in_lds) {
      for (int cg = 0; cg < bw; cg += d) {
        const int64_t gq = c0 / d + cg / d;
        const dim3 gs(static_cast<unsigned>(row_tiles), static_cast<unsigned>(nslice));
        const unsigned ga = static_cast<unsigned>(cdiv(M, 256));
        if (d <= 8) {
          hipLaunchKernelGGL(refine_scan_kernel<8>, gs, dim3(256), 0, stream, M, d, c0 + cg, gq, S, n_cols, H, ldh, Cb,
                             c_type, static_cast<int>(K), slice, codes, ldq, bestF, bestK);
          hipLaunchKernelGGL(refine_apply_kernel<8>, dim3(ga), dim3(256), 0, stream, M, d, c0, cg, bw, gq, R, ldr, S,
                             n_cols, H, ldh, Cb, c_type, static_cast<int>(K), codes, ldq, D, bw_max,
                             static_cast<int>(nslice), bestF, bestK);
        } else {
          hipLaunchKernelGGL(refine_scan_kernel<16>, gs, dim3(256), 0, stream, M, d, c0 + cg, gq, S, n_cols, H, ldh,
                             Cb, c_type, static_cast<int>(K), slice, codes, ldq, bestF, bestK);
          hipLaunchKernelGGL(refine_apply_kernel<16>, dim3(ga), dim3(256), 0, stream, M, d, c0, cg, bw, gq, R, ldr, S,
                             n_cols, H, ldh, Cb, c_type, static_cast<int>(K), codes, ldq, D, bw_max,
                             static_cast<int>(nslice), bestF, bestK);
        }
      }
    } else if (d <= 8)
      hipLaunchKernelGGL(refine_block_kernel<8>, grid, dim3(kRfThreads), lds, stream, M, d, c0, bw, R, ldr, S, n_cols,
                         H, ldh, Cb, c_type, static_cast<int>(K), codes, ldq, D, bw_max);
    else
      hipLaunchKernelGGL(refine_block_kernel<16>, grid, dim3(kRfThreads), lds, stream, M, d, c0, bw, R, ldr, S, n_cols,
                         H, ldh, Cb, c_type, static_cast<int>(K), codes, ldq, D, bw_max);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int64_t c1 = c0 + bw;
    if (c1 < o1)
      e = launch_gemm_f64(M, o1 - c1, bw, Db, outer, H + c0 * ldh + c1, ldh, S + c1, n_cols, true, stream);
    else if (c1 < n_cols)
      e = launch_gemm_f64(M, n_cols - c1, c1 - o0, D, outer, H + o0 * ldh + c1, ldh, S + c1, n_cols, true, stream);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace crvq
