// Stacked right-hand sides solved together by the enlarged-CG recurrences (Alg. 2, Orthomin
// variant) applied to t right-hand sides that share P and N^-1:
//
//   R = B, Z = M R;  repeat:  W = A Z (one multi-column product), G = Z^T W, H1 = Z^T R,
//   X += Z G^+ H1,  R -= W G^+ H1,  stop columns with ||R_j|| < eps ||B_j||,
//   Z <- M R - Z G^+ (W^T M R)
//
// (P_k = Z G^-1/2 folds into G^+ = G^-1/2 G^-1/2).  G^+ is an FP64 eigen pseudo-inverse that
// drops directions below 1e-12 of the largest eigenvalue, a safeguard against the rank loss of
// the search block (the paper's Cholesky square root has none).  Converged columns leave the
// block (their X is final).  The t x t algebra runs on the host in FP64; the tall-skinny Gram
// products, updates and the block-Jacobi apply run in the kernels below, in FP64.  An iteration
// meets the host once: G and H1 come back (with the outcome of the previous iteration's stop
// tests, which the device has already applied to Z), a1 and G^+ go out; on FP64 plans the outcome
// comes back on its own, ahead of the product.
//
// Block size: opts->block >= 2 fixes t; opts->block < 0 tunes it: the first column groups are
// solved with t = 1 (8 columns, each alone by Alg. 1), 8, 16, 32 in turn (real work, not a
// rehearsal); the candidate with the lowest time per right-hand side then solves the remaining
// columns and is kept in the plan and, for the life of the process, for plans of the same
// shape, so later tuned solves start with it.  When
// the stacked recurrences do not shorten the iteration enough to pay for their extra
// tall-skinny work, t = 1 wins.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <initializer_list>
#include <map>
#include <mutex>
#include <numeric>
#include <tuple>

#include "mm_internal.h"

namespace mm {

namespace {

constexpr int kThreads = 256;
constexpr int kMaxT = 32;

// Gram partials of U^T V1 (tu x tv1) and U^T V2 (tu x tv2; tv2 = 0: one product), summed over
// workgroup x's rows, on the FP64 matrix cores: workgroup (x, y) takes block y of 16 columns of U
// by 16 columns of [V1 | V2] and a grid-stride share of the rows, each wavefront 32 rows a step.
// A lane loads 8 consecutive rows of one column of each operand (64 contiguous bytes) and feeds
// them to eight 16 x 16 x 4 products: which four rows meet in one product does not matter as long
// as both operands agree.  The four wavefronts' blocks are added in LDS in a fixed order.
// partial[x] holds the tu x tv1 entries, then the tu x tv2 entries.
//
// The kernel is bound by its latency (3 MB a column at 16,384 pixels): a form with 64 sums per
// thread needed 384 shuffles to reduce them, so it could only afford 12 workgroups there, 30 us
// for eight columns against 5 us with a workgroup per 128 rows.
constexpr int kGB = 16;        // block of column pairs
constexpr int kGRows = 8;      // consecutive rows per lane and step
constexpr int kGStep = 4 * kGRows;  // rows per wavefront and step
constexpr int kWaves = kThreads / 64;

typedef double v4d __attribute__((ext_vector_type(4)));

// Rows [r, r + kGRows) of a column (null: zeros), zero past its end.
__device__ __forceinline__ void gram_rows(const double* __restrict__ col, int64_t r, int64_t n,
                                          double (&a)[kGRows]) {
#pragma unroll
  for (int k = 0; k < kGRows; ++k) a[k] = 0.0;
  if (col == nullptr) return;
  if (r + kGRows <= n) {
#pragma unroll
    for (int k = 0; k < kGRows; ++k) a[k] = col[r + k];
  } else {
#pragma unroll
    for (int k = 0; k < kGRows; ++k)
      if (r + k < n) a[k] = col[r + k];
  }
}

__global__ __launch_bounds__(kThreads) void k_gram(const double* __restrict__ U, int tu,
                                                   const double* __restrict__ V1, int tv1,
                                                   const double* __restrict__ V2, int tv2,
                                                   int64_t n, double* __restrict__ partial) {
  __shared__ double red[kWaves][kGB * kGB];
  const int tv = tv1 + tv2, nbv = (tv + kGB - 1) / kGB;
  const int i0 = (static_cast<int>(blockIdx.y) / nbv) * kGB;
  const int j0 = (static_cast<int>(blockIdx.y) % nbv) * kGB;
  const int lane = static_cast<int>(threadIdx.x & 63u);
  const int wave = static_cast<int>(threadIdx.x >> 6);
  const int c = lane & 15, q = lane >> 4;
  const int i = i0 + c, j = j0 + c;
  const double* u = i < tu ? U + static_cast<int64_t>(i) * n : nullptr;
  const double* v = j < tv1   ? V1 + static_cast<int64_t>(j) * n
                    : j < tv ? V2 + static_cast<int64_t>(j - tv1) * n
                             : nullptr;
  v4d acc = {0.0, 0.0, 0.0, 0.0};
  for (int64_t r0 = (static_cast<int64_t>(blockIdx.x) * kWaves + wave) * kGStep; r0 < n;
       r0 += static_cast<int64_t>(gridDim.x) * kWaves * kGStep) {
    const int64_t r = r0 + kGRows * q;
    double a[kGRows], b[kGRows];
    gram_rows(u, r, n, a);
    gram_rows(v, r, n, b);
#pragma unroll
    for (int k = 0; k < kGRows; ++k)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k], b[k], acc, 0, 0, 0);
  }
  // lane (q, c) holds entries (q + 4 k, c) of the block
#pragma unroll
  for (int k = 0; k < 4; ++k) red[wave][(q + 4 * k) * kGB + c] = acc[k];
  __syncthreads();
  const int bi = i0 + static_cast<int>(threadIdx.x) / kGB;
  const int bj = j0 + static_cast<int>(threadIdx.x) % kGB;
  if (bi < tu && bj < tv) {
    double x = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) x += red[w][threadIdx.x];
    const int at = bj < tv1 ? bi * tv1 + bj : tu * tv1 + bi * tv2 + (bj - tv1);
    partial[static_cast<int64_t>(blockIdx.x) * tu * tv + at] = x;
  }
}

// out[e] = sum_w partial[w][e] in a fixed order: kRedEntries entries per workgroup, 16 threads
// per entry each summing every 16th partial, then a fixed tree over the 16 sums (one thread per
// entry walking all partials serially took ~150 us for 512 partials).  Entries from count on come
// from a second array (partial2, nwg2 rows of count2) and go to out2.
constexpr int kRedEntries = kThreads / 16;

__global__ __launch_bounds__(kThreads) void k_gram_reduce(const double* __restrict__ partial,
                                                          int nwg, int count,
                                                          double* __restrict__ out,
                                                          const double* __restrict__ partial2,
                                                          int nwg2, int count2,
                                                          double* __restrict__ out2) {
  __shared__ double red[kThreads];
  const int le = threadIdx.x >> 4, lw = threadIdx.x & 15;
  int e = blockIdx.x * kRedEntries + le;
  const bool second = e >= count;
  if (second) {
    e -= count;
    partial = partial2;
    nwg = nwg2;
    out = out2;
  }
  const int stride = second ? count2 : count;
  double s = 0.0;
  if (e < stride)
    for (int w = lw; w < nwg; w += 16) s += partial[static_cast<int64_t>(w) * stride + e];
  red[threadIdx.x] = s;
  __syncthreads();
#pragma unroll
  for (int h = 8; h > 0; h >>= 1) {
    if (lw < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (lw == 0 && e < stride) out[e] = red[threadIdx.x];
}

inline unsigned reduce_grid(int count) {
  return static_cast<unsigned>((count + kRedEntries - 1) / kRedEntries);
}

// The coefficient table's address, opaque to the optimiser: read inside the row loop (broadcast
// LDS reads) instead of hoisting up to t x t coefficients into registers across all rows.
__device__ __forceinline__ const double* row_coefs(const double* p) {
  asm volatile("" : "+v"(p));
  return p;
}

// X_cols[j] += sum_i Z_i a1[i][j];  R_j -= sum_i W_i a1[i][j];  rr partial of ||R_j||^2, for the
// t columns of the block (TM >= t).  The rows of X (and of R) are loaded eight columns at a time
// ahead of their stores: the compiler cannot tell the columns apart, and would wait for each
// column's load behind the previous column's store (16 us against 12 us for eight columns at
// 16,384 pixels).
template <int TM>
__global__ __launch_bounds__(kThreads) void k_block_update(
    const double* __restrict__ Z, const double* __restrict__ W, double* __restrict__ R, int t,
    int64_t nu, double* __restrict__ x, const int32_t* __restrict__ cols,
    const double* __restrict__ a1, double* __restrict__ rr_partial) {
  constexpr int kBatch = 8;
  __shared__ double sa[kMaxT * kMaxT];
  __shared__ double red[kThreads / 64][TM];
  for (int e = threadIdx.x; e < t * t; e += kThreads) sa[e] = a1[e];
  __syncthreads();
  double rr[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) rr[j] = 0.0;
  for (int64_t r = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; r < nu;
       r += static_cast<int64_t>(gridDim.x) * kThreads) {
    {  // X += Z a1 (one row of Z live at a time)
      double z[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) z[i] = i < t ? Z[i * nu + r] : 0.0;
      const double* c = row_coefs(sa);
#pragma unroll
      for (int j0 = 0; j0 < TM; j0 += kBatch) {
        double xv[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
          xv[j] = j0 + j < t ? x[static_cast<int64_t>(cols[j0 + j]) * nu + r] : 0.0;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
          if (j0 + j < t) {
            double dx = 0.0;
#pragma unroll
            for (int i = 0; i < TM; ++i)
              if (i < t) dx += z[i] * c[i * t + j0 + j];
            x[static_cast<int64_t>(cols[j0 + j]) * nu + r] = xv[j] + dx;
          }
        }
      }
    }
    {  // R -= W a1, with the norms
      double w[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) w[i] = i < t ? W[i * nu + r] : 0.0;
      const double* c = row_coefs(sa);
#pragma unroll
      for (int j0 = 0; j0 < TM; j0 += kBatch) {
        double rv[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) rv[j] = j0 + j < t ? R[(j0 + j) * nu + r] : 0.0;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
          if (j0 + j < t) {
            double dr = 0.0;
#pragma unroll
            for (int i = 0; i < TM; ++i)
              if (i < t) dr += w[i] * c[i * t + j0 + j];
            const double rn = rv[j] - dr;
            R[(j0 + j) * nu + r] = rn;
            rr[j0 + j] += rn * rn;
          }
        }
      }
    }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    double v = rr[j];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if (lane == 0) red[wv][j] = v;
  }
  __syncthreads();
  if (threadIdx.x < t) {
    double s = 0.0;
    for (int q = 0; q < kThreads / 64; ++q) s += red[q][threadIdx.x];
    rr_partial[static_cast<int64_t>(blockIdx.x) * t + threadIdx.x] = s;
  }
}

// After an update: act[j] = 1 while column j's ||R_j||^2 has not passed under its limit, *done
// once none is left, and a2 = G^+ H2 (t x t).  One workgroup.
__global__ __launch_bounds__(kThreads) void k_block_coef(int t, const double* __restrict__ rr,
                                                         const double* __restrict__ limit,
                                                         const double* __restrict__ gi,
                                                         const double* __restrict__ h2,
                                                         double* __restrict__ a2,
                                                         double* __restrict__ act,
                                                         int32_t* __restrict__ done) {
  const int j = threadIdx.x;
  const bool live = j < t && !(rr[j] < limit[j]);
  if (j < t) act[j] = live ? 1.0 : 0.0;
  const int left = __syncthreads_count(live);
  if (threadIdx.x == 0 && left == 0) *done = 1;
  for (int e = threadIdx.x; e < t * t; e += kThreads) {
    const int row = e / t, col = e % t;
    double s = 0.0;
    for (int k = 0; k < t; ++k) s += gi[row * t + k] * h2[k * t + col];
    a2[e] = s;
  }
}

// Z_j <- MR_j - sum_i Z_i a2[i][j]  for the columns still in the block, 0 for those that have
// left it (in place: each row reads all old Z first)
template <int TM>
__global__ __launch_bounds__(kThreads) void k_block_direction(double* __restrict__ Z, int t,
                                                              const double* __restrict__ MR,
                                                              int64_t nu,
                                                              const double* __restrict__ a2,
                                                              const double* __restrict__ act) {
  constexpr int kBatch = 8;
  __shared__ double sa[kMaxT * kMaxT];
  for (int e = threadIdx.x; e < t * t; e += kThreads) sa[e] = a2[e];
  __syncthreads();
  for (int64_t r = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; r < nu;
       r += static_cast<int64_t>(gridDim.x) * kThreads) {
    double z[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) z[i] = i < t ? Z[i * nu + r] : 0.0;
    const double* c = row_coefs(sa);
#pragma unroll
    for (int j0 = 0; j0 < TM; j0 += kBatch) {
      double mr[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) mr[j] = j0 + j < t ? MR[(j0 + j) * nu + r] : 0.0;
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        if (j0 + j < t) {
          double s = mr[j];
#pragma unroll
          for (int i = 0; i < TM; ++i)
            if (i < t) s -= z[i] * c[i * t + j0 + j];
          Z[(j0 + j) * nu + r] = act[j0 + j] != 0.0 ? s : 0.0;
        }
      }
    }
  }
}

// rr_partial[wg][j] = partial sum of (B_j - Y_j)^2 (or B_j^2 when Y is null)
template <int TM>
__global__ __launch_bounds__(kThreads) void k_col_norms(const double* __restrict__ B, int t,
                                                        const double* __restrict__ Y, int64_t nu,
                                                        double* __restrict__ partial) {
  __shared__ double red[kThreads / 64][TM];
  double acc[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) acc[j] = 0.0;
  for (int64_t r = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; r < nu;
       r += static_cast<int64_t>(gridDim.x) * kThreads) {
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      if (j < t) {
        const double v = B[j * nu + r] - (Y ? Y[j * nu + r] : 0.0);
        acc[j] += v * v;
      }
    }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    double v = acc[j];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if (lane == 0) red[wv][j] = v;
  }
  __syncthreads();
  if (threadIdx.x < t) {
    double s = 0.0;
    for (int q = 0; q < kThreads / 64; ++q) s += red[q][threadIdx.x];
    partial[static_cast<int64_t>(blockIdx.x) * t + threadIdx.x] = s;
  }
}

__global__ void k_zero_cols(double* __restrict__ x, const int32_t* __restrict__ cols, int t,
                            int64_t nu) {
  for (int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; e < t * nu;
       e += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int j = static_cast<int>(e / nu);
    x[static_cast<int64_t>(cols[j]) * nu + (e % nu)] = 0.0;
  }
}

#define MM_TM_DISPATCH(KERNEL, t, grid, s, ...)                                             \
  do {                                                                                      \
    if ((t) <= 8)                                                                           \
      hipLaunchKernelGGL(KERNEL<8>, dim3(grid), dim3(kThreads), 0, s, __VA_ARGS__);         \
    else if ((t) <= 16)                                                                     \
      hipLaunchKernelGGL(KERNEL<16>, dim3(grid), dim3(kThreads), 0, s, __VA_ARGS__);        \
    else                                                                                    \
      hipLaunchKernelGGL(KERNEL<32>, dim3(grid), dim3(kThreads), 0, s, __VA_ARGS__);        \
  } while (0)

// ---- host-side t x t algebra (FP64) ---------------------------------------------------------

// C (n x m) = A (n x n) B (n x m), row-major
void matmul(const std::vector<double>& A, const std::vector<double>& B, int n, int m,
            std::vector<double>& C) {
  C.assign(static_cast<size_t>(n) * m, 0.0);
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < n; ++k) {
      const double aik = A[i * n + k];
      for (int j = 0; j < m; ++j) C[i * m + j] += aik * B[k * m + j];
    }
}

struct BlockWs {
  double* R = nullptr;
  double* Z = nullptr;
  double* W = nullptr;
  double* MR = nullptr;
  double* small = nullptr;    // scalars and t x t matrices (k* offsets below)
  double* partial = nullptr;  // Gram partials
  double* rr_partial = nullptr;
  int32_t* cols = nullptr;    // user column of each slot, then the done flag
  int cap = 0;
};

// Layout of BlockWs::small (doubles).  An iteration reads [0, kG + 2 t^2) back in one copy: the
// last update's norms and activity and the new Gram matrices; and writes [kA1, kA1 + 2 t^2).
constexpr int kMat = kMaxT * kMaxT;
constexpr int kRr = 0, kAct = kMaxT, kG = 2 * kMaxT;           // G, then H1
constexpr int kA1 = kG + 2 * kMat;                             // a1, then G^+
constexpr int kH2 = kA1 + 2 * kMat, kA2 = kH2 + kMat, kLimit = kA2 + kMat;
constexpr int kSmall = kLimit + kMaxT;
static_assert(kSmall + kMaxT <= kBlockHost, "pinned transfer area");

// Workgroups of the Gram kernel: one step of each wavefront, at most one workgroup per CU and
// column block (more partials would cost the reduction what they hide).
int gram_grid(int64_t nu) {
  const int64_t g = (nu + kWaves * kGStep - 1) / (kWaves * kGStep);
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(g, 256)));
}

int rows_grid(int64_t nu) {
  int64_t g = (nu + kThreads - 1) / kThreads;
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(g, 1024)));
}

mm_status ensure_ws(Plan* P, Work& Wk, BlockWs& ws, int t) {
  if (ws.cap >= t) return MM_OK;
  const int64_t nu = 3 * P->n_kept;
  for (void* p : {static_cast<void*>(ws.R), static_cast<void*>(ws.Z), static_cast<void*>(ws.W),
                  static_cast<void*>(ws.MR), static_cast<void*>(ws.small),
                  static_cast<void*>(ws.partial), static_cast<void*>(ws.rr_partial),
                  static_cast<void*>(ws.cols)})
    dev_free(p);
  ws = BlockWs{};
  auto alloc = [&](void** p, size_t bytes) -> mm_status {
    if (dev_malloc(p, std::max<size_t>(bytes, 8)) != hipSuccess) {
      *p = nullptr;
      return fail(MM_ERR_OOM, "hipMalloc (block workspace) failed");
    }
    return MM_OK;
  };
  const size_t vec = sizeof(double) * static_cast<size_t>(t) * nu;
  MM_TRY(alloc(reinterpret_cast<void**>(&ws.R), vec));
  MM_TRY(alloc(reinterpret_cast<void**>(&ws.Z), vec));
  MM_TRY(alloc(reinterpret_cast<void**>(&ws.W), vec));
  MM_TRY(alloc(reinterpret_cast<void**>(&ws.MR), vec));
  MM_TRY(alloc(reinterpret_cast<void**>(&ws.small), sizeof(double) * kSmall));
  MM_TRY(alloc(reinterpret_cast<void**>(&ws.partial),
               sizeof(double) * static_cast<size_t>(gram_grid(nu)) * 2 * kMat));
  MM_TRY(alloc(reinterpret_cast<void**>(&ws.rr_partial),
               sizeof(double) * static_cast<size_t>(rows_grid(nu)) * kMaxT));
  MM_TRY(alloc(reinterpret_cast<void**>(&ws.cols), sizeof(int32_t) * (kMaxT + 1)));
  if (Wk.h_block == nullptr) {
    std::unique_lock<std::shared_mutex> lock(alloc_gate());
    MM_HIP_TRY(hipHostMalloc(reinterpret_cast<void**>(&Wk.h_block), sizeof(double) * kBlockHost,
                             hipHostMallocDefault));
  }
  ws.cap = t;
  return MM_OK;
}

void free_ws(BlockWs& ws) {
  for (void* p : {static_cast<void*>(ws.R), static_cast<void*>(ws.Z), static_cast<void*>(ws.W),
                  static_cast<void*>(ws.MR), static_cast<void*>(ws.small),
                  static_cast<void*>(ws.partial), static_cast<void*>(ws.rr_partial),
                  static_cast<void*>(ws.cols)})
    dev_free(p);
  ws = BlockWs{};
}

// Gram partials of U^T V1 and U^T V2 (tv2 = 0: one product); returns their number.
int launch_gram(const double* U, int tu, const double* V1, int tv1, const double* V2, int tv2,
                int64_t nu, double* partial, hipStream_t s) {
  const int g = gram_grid(nu);
  const int nb = ((tu + kGB - 1) / kGB) * ((tv1 + tv2 + kGB - 1) / kGB);
  hipLaunchKernelGGL(k_gram, dim3(static_cast<unsigned>(g), static_cast<unsigned>(nb)),
                     dim3(kThreads), 0, s, U, tu, V1, tv1, V2, tv2, nu, partial);
  return g;
}

void launch_reduce(const double* partial, int nwg, int count, double* out, const double* partial2,
                   int nwg2, int count2, double* out2, hipStream_t s) {
  hipLaunchKernelGGL(k_gram_reduce, dim3(reduce_grid(count + count2)), dim3(kThreads), 0, s,
                     partial, nwg, count, out, partial2, nwg2, count2, out2);
}

// Per-column ||B_j - Y_j||^2 (Y may be null) to the host.
mm_status col_norms(const double* B, const double* Y, int t, int64_t nu, BlockWs& ws,
                    double* host, std::vector<double>& out, hipStream_t s) {
  const int g = rows_grid(nu);
  MM_TM_DISPATCH(k_col_norms, t, g, s, B, t, Y, nu, ws.rr_partial);
  launch_reduce(ws.rr_partial, g, t, ws.small + kRr, nullptr, 0, 0, nullptr, s);
  MM_HIP_TRY(hipGetLastError());
  MM_HIP_TRY(hipMemcpyAsync(host, ws.small + kRr, sizeof(double) * t, hipMemcpyDeviceToHost, s));
  MM_HIP_TRY(hipStreamSynchronize(s));
  out.assign(host, host + t);
  return MM_OK;
}

// Solve the columns `cols` (at most kMaxT) together.
mm_status solve_group(Plan* P, Work& Wk, const float* d, int64_t ld_d, double* x,
                      const std::vector<int32_t>& cols, double tol, int max_iter,
                      mm_solve_info* info, int block_used, BlockWs& ws, hipStream_t s) {
  const int t = static_cast<int>(cols.size());
  const int64_t nu = 3 * P->n_kept;
  MM_TRY(ensure_ws(P, Wk, ws, t));
  double* const host = Wk.h_block;
  auto ev = std::chrono::steady_clock::now();

  // R_j = b_j = P^T N^-1 d_j, X_j = 0
  MM_HIP_TRY(hipMemcpyAsync(ws.cols, cols.data(), sizeof(int32_t) * t, hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(k_zero_cols, dim3(rows_grid(t * nu)), dim3(kThreads), 0, s, x, ws.cols, t, nu);
  for (int j = 0; j < t; ++j) MM_TRY(compute_rhs(P, Wk, d + cols[j] * ld_d, ws.R + j * nu, s));
  std::vector<double> bb;
  MM_TRY(col_norms(ws.R, nullptr, t, nu, ws, host, bb, s));
  std::vector<double> bnorm(t);
  for (int j = 0; j < t; ++j) bnorm[j] = std::sqrt(bb[j]);

  // active slots: columns with b != 0 (others are solved by x = 0)
  std::vector<int32_t> act;           // user column of each active slot
  std::vector<int> slot_of;           // original position of each active slot
  std::vector<int> iters(t, 0), conv(t, 0);
  std::vector<double> relres(t, 0.0);
  for (int j = 0; j < t; ++j) {
    if (bnorm[j] > 0.0) {
      if (static_cast<int>(act.size()) != j)
        MM_HIP_TRY(hipMemcpyAsync(ws.R + act.size() * nu, ws.R + j * nu, sizeof(double) * nu,
                                  hipMemcpyDeviceToDevice, s));
      act.push_back(cols[j]);
      slot_of.push_back(j);
    } else {
      conv[j] = 1;
    }
  }
  int ta = static_cast<int>(act.size());
  int32_t* const done = ws.cols + kMaxT;
  // Slot tables (user columns, limits of ||R_j||^2, the done flag cleared): at the start and
  // whenever columns have left.  They travel through their own part of the pinned area, which
  // is read before the stream is next synchronized.
  auto upload_slots = [&]() -> mm_status {
    double* lim = host + kLimit;
    int32_t* tab = reinterpret_cast<int32_t*>(host + kSmall);
    for (int i = 0; i < ta; ++i) {
      const double l = tol * bnorm[slot_of[i]];
      lim[i] = l * l;
      tab[i] = act[i];
    }
    tab[kMaxT] = 0;
    MM_HIP_TRY(hipMemcpyAsync(ws.small + kLimit, lim, sizeof(double) * ta, hipMemcpyHostToDevice, s));
    MM_HIP_TRY(hipMemcpyAsync(ws.cols, tab, sizeof(int32_t) * (kMaxT + 1), hipMemcpyHostToDevice, s));
    return MM_OK;
  };
  // The last update's outcome, already on the host: norms, and the slots still in the block.
  std::vector<int> keep;
  auto settle = [&](int k) {
    keep.clear();
    for (int i = 0; i < ta; ++i) {
      const int j = slot_of[i];
      relres[j] = std::sqrt(std::max(host[kRr + i], 0.0)) / bnorm[j];
      iters[j] = k;
      if (host[kAct + i] != 0.0)
        keep.push_back(i);
      else
        conv[j] = 1;
    }
  };
  // Drops the columns that have left from the block's vectors and slot tables.
  auto compact = [&](std::initializer_list<double*> vecs) -> mm_status {
    const int tn = static_cast<int>(keep.size());
    for (int i = 0; i < tn; ++i) {
      if (keep[i] != i)
        for (double* v : vecs)
          MM_HIP_TRY(hipMemcpyAsync(v + i * nu, v + keep[i] * nu, sizeof(double) * nu,
                                    hipMemcpyDeviceToDevice, s));
      act[i] = act[keep[i]];
      slot_of[i] = slot_of[keep[i]];
    }
    ta = tn;
    act.resize(ta);
    slot_of.resize(ta);
    return ta > 0 ? upload_slots() : MM_OK;
  };
  // The stop flag gates every product but the FP64 one: there the host reads an update's outcome
  // ahead of the next product, not with its Gram matrices, so that no column takes a product after
  // its last update (a second read-back per iteration, against a product per column).
  const bool gated = P->precision != MM_PRECISION_FP64 || P->lambda_max == 0;
  auto read_outcome = [&](int k) -> mm_status {
    MM_HIP_TRY(hipMemcpyAsync(host, ws.small, sizeof(double) * kG, hipMemcpyDeviceToHost, s));
    MM_HIP_TRY(hipStreamSynchronize(s));
    settle(k);
    return MM_OK;
  };
  std::vector<double> G, H, Gi, A;
  if (ta > 0) {
    MM_TRY(upload_slots());
    MM_TRY(launch_precond_multi(P, ws.R, ws.Z, ta, s));  // Z = M R
  }
  int k = 0;
  while (ta > 0 && k < max_iter) {
    // W = A Z; G = Z^T W, H1 = Z^T R.  With the outcome of the last update still on the device,
    // columns that left in it have Z = 0 (and rows and columns of zeros in G); with none left the
    // product exits at once.
    MM_TRY(apply_A_multi(P, Wk, ws.Z, nu, ws.W, nu, ta, s, done));
    const int ng = launch_gram(ws.Z, ta, ws.W, ta, ws.R, ta, nu, ws.partial, s);
    launch_reduce(ws.partial, ng, 2 * ta * ta, ws.small + kG, nullptr, 0, 0, nullptr, s);
    MM_HIP_TRY(hipGetLastError());
    MM_HIP_TRY(hipMemcpyAsync(host, ws.small, sizeof(double) * (kG + 2 * ta * ta),
                              hipMemcpyDeviceToHost, s));
    MM_HIP_TRY(hipStreamSynchronize(s));
    const int told = ta;
    keep.resize(ta);
    std::iota(keep.begin(), keep.end(), 0);
    if (k > 0 && gated) {
      settle(k);
      if (keep.empty()) {
        ta = 0;
        break;
      }
      if (static_cast<int>(keep.size()) < told) MM_TRY(compact({ws.Z, ws.W, ws.R}));
    }
    G.resize(static_cast<size_t>(ta) * ta);
    H.resize(static_cast<size_t>(ta) * ta);
    for (int i = 0; i < ta; ++i)
      for (int j = 0; j < ta; ++j) {
        G[i * ta + j] = host[kG + keep[i] * told + keep[j]];
        H[i * ta + j] = host[kG + told * told + keep[i] * told + keep[j]];
      }
    sym_pinv(G, ta, 1e-12, Gi);
    matmul(Gi, H, ta, ta, A);  // a1 = G^+ H1
    std::copy(A.begin(), A.end(), host + kA1);
    std::copy(Gi.begin(), Gi.end(), host + kA1 + ta * ta);
    MM_HIP_TRY(hipMemcpyAsync(ws.small + kA1, host + kA1, sizeof(double) * 2 * ta * ta,
                              hipMemcpyHostToDevice, s));
    const int g = rows_grid(nu);
    MM_TM_DISPATCH(k_block_update, ta, g, s, ws.Z, ws.W, ws.R, ta, nu, x, ws.cols,
                   ws.small + kA1, ws.rr_partial);
    // MR = M R, H2 = W^T MR and ||R_j||^2; a2 = G^+ H2 and the stop tests; Z <- MR - Z a2.  The
    // host reads the norms with the next iteration's Gram matrices.
    MM_TRY(launch_precond_multi(P, ws.R, ws.MR, ta, s));
    const int nh = launch_gram(ws.W, ta, ws.MR, ta, nullptr, 0, nu, ws.partial, s);
    launch_reduce(ws.partial, nh, ta * ta, ws.small + kH2, ws.rr_partial, g, ta, ws.small + kRr, s);
    hipLaunchKernelGGL(k_block_coef, dim3(1), dim3(kThreads), 0, s, ta, ws.small + kRr,
                       ws.small + kLimit, ws.small + kA1 + ta * ta, ws.small + kH2,
                       ws.small + kA2, ws.small + kAct, done);
    MM_TM_DISPATCH(k_block_direction, ta, g, s, ws.Z, ta, ws.MR, nu, ws.small + kA2,
                   ws.small + kAct);
    MM_HIP_TRY(hipGetLastError());
    ++k;
    if (!gated) {
      MM_TRY(read_outcome(k));
      if (static_cast<int>(keep.size()) < ta) MM_TRY(compact({ws.Z, ws.R}));
    }
  }
  if (ta > 0 && gated) MM_TRY(read_outcome(k));  // stopped by max_iter

  // true residuals ||b - A x|| (W = A X, R = b)
  std::vector<double> tr(t, 0.0);
  MM_HIP_TRY(hipMemcpyAsync(ws.cols, cols.data(), sizeof(int32_t) * t, hipMemcpyHostToDevice, s));
  for (int j = 0; j < t; ++j) {
    MM_TRY(compute_rhs(P, Wk, d + cols[j] * ld_d, ws.R + j * nu, s));
    MM_TRY(apply_A(P, Wk, x + static_cast<int64_t>(cols[j]) * nu, ws.W + j * nu, nullptr, s));
  }
  MM_TRY(col_norms(ws.R, ws.W, t, nu, ws, host, tr, s));
  const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - ev).count();
  for (int j = 0; j < t; ++j) {
    mm_solve_info& in = info[cols[j]];
    in.iterations = iters[j];
    in.converged = conv[j];
    in.relres = relres[j];
    in.bnorm = bnorm[j];
    in.true_relres = bnorm[j] > 0 ? std::sqrt(tr[j]) / bnorm[j] : 0.0;
    in.ms = ms;
    in.block = block_used;
    in.refine_steps = 0;
    in.true_relres64 = -1.0;
    in.inner_iterations = 0;
    in.pad0 = 0;
  }
  return MM_OK;
}

}  // namespace

// Pseudo-inverse of a symmetric positive semi-definite n x n matrix (row-major) by cyclic
// Jacobi eigen-decomposition; eigenvalues below rtol * largest are dropped.
void sym_pinv(const std::vector<double>& G, int n, double rtol, std::vector<double>& out,
              SymPinvInfo* info) {
  std::vector<double> a(G), v(static_cast<size_t>(n) * n, 0.0);
  for (int i = 0; i < n; ++i) v[i * n + i] = 1.0;
  // The rotations annihilate the upper triangle.  G = Z^T A Z of a single-precision operator is
  // symmetric to ~1e-8 only, and what asymmetry it has stays below the diagonal: the upper
  // triangle alone says when the sweeps are done (one more follows, to full precision).
  bool last = false;
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0, tot = 0.0;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) {
        tot += a[i * n + j] * a[i * n + j];
        if (i < j) off += a[i * n + j] * a[i * n + j];
      }
    if (last || tot == 0.0) break;
    last = off <= 1e-30 * tot;
    for (int p = 0; p < n - 1; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = a[p * n + q];
        if (apq == 0.0) continue;
        const double theta = (a[q * n + q] - a[p * n + p]) / (2.0 * apq);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
        const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
        for (int k = 0; k < n; ++k) {  // columns p, q
          const double akp = a[k * n + p], akq = a[k * n + q];
          a[k * n + p] = c * akp - s * akq;
          a[k * n + q] = s * akp + c * akq;
        }
        for (int k = 0; k < n; ++k) {  // rows p, q
          const double apk = a[p * n + k], aqk = a[q * n + k];
          a[p * n + k] = c * apk - s * aqk;
          a[q * n + k] = s * apk + c * aqk;
        }
        for (int k = 0; k < n; ++k) {  // eigenvectors
          const double vkp = v[k * n + p], vkq = v[k * n + q];
          v[k * n + p] = c * vkp - s * vkq;
          v[k * n + q] = s * vkp + c * vkq;
        }
      }
  }
  double wmax = 0.0;
  for (int i = 0; i < n; ++i) wmax = std::max(wmax, a[i * n + i]);
  out.assign(static_cast<size_t>(n) * n, 0.0);
  if (info) *info = SymPinvInfo{0, INFINITY, wmax};
  for (int e = 0; e < n; ++e) {
    const double w = a[e * n + e];
    if (!(w > rtol * wmax) || w <= 0.0) continue;
    if (info) {
      info->rank += 1;
      info->wmin = std::min(info->wmin, w);
    }
    const double inv = 1.0 / w;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) out[i * n + j] += v[i * n + e] * inv * v[j * n + e];
  }
}


// Tuned block sizes by problem shape, kept for the life of the process: a plan rebuilt for the
// same geometry starts with the size an earlier plan found.
namespace {
struct ShapeKey {
  int64_t n_samples, n_kept;
  int32_t lambda_max, fft_n, algo, fused;
  bool operator<(const ShapeKey& o) const {
    return std::tie(n_samples, n_kept, lambda_max, fft_n, algo, fused) <
           std::tie(o.n_samples, o.n_kept, o.lambda_max, o.fft_n, o.algo, o.fused);
  }
};
std::mutex g_tuned_mu;
std::map<ShapeKey, int32_t> g_tuned;

ShapeKey shape_of(const Plan* P) {
  return ShapeKey{P->n_samples, P->n_kept, P->lambda_max, P->fft_n, P->algo, P->fused ? 1 : 0};
}
}  // namespace

mm_status block_solve(Plan* P, Work& Wk, const float* d, int32_t k, int64_t ld_d, double* x,
                      const mm_solve_opts* o, mm_solve_info* info, hipStream_t s) {
  if (o->block < 0 && P->tuned_block.load() == 0) {
    std::lock_guard<std::mutex> lock(g_tuned_mu);
    auto it = g_tuned.find(shape_of(P));
    if (it != g_tuned.end()) P->tuned_block = it->second;
  }
  const double tol = o->tol > 0 ? o->tol : 1e-8;
  const int max_iter = o->max_iter > 0 ? o->max_iter : 10000;
  std::vector<mm_solve_info> local(static_cast<size_t>(k));
  mm_solve_info* inf = info ? info : local.data();
  BlockWs ws;
  struct Guard {
    BlockWs& w;
    ~Guard() { free_ws(w); }
  } guard{ws};
  std::vector<int> candidates;
  int best = 0;
  if (o->block < 0 && P->tuned_block.load() > 0) {
    best = P->tuned_block.load();  // chosen by an earlier tuned solve on this plan
  } else if (o->block < 0) {
    candidates = {1, 8, 16, 32};  // 1: each column alone by Alg. 1
    best = candidates[0];
  } else {
    best = std::min(std::max(2, static_cast<int>(o->block)), kMaxT);
  }
  int32_t next = 0;
  size_t ci = 0;
  double best_cost = INFINITY;
  mm_solve_opts alone = *o;  // the t = 1 candidate: Alg. 1 per column
  alone.block = 0;
  alone.use_x0 = 0;
  alone.precond = 0;
  while (next < k) {
    const bool tuning = ci < candidates.size();
    const int t = tuning ? candidates[ci] : best;
    const int group = t == 1 ? kMaxT / 4 : t;  // columns per group (8 for the t = 1 candidate)
    const int n = std::min<int32_t>(group, k - next);
    std::vector<int32_t> cols(n);
    std::iota(cols.begin(), cols.end(), next);
    const auto t0 = std::chrono::steady_clock::now();
    if (t == 1) {
      for (int32_t j : cols) {
        const mm_status st = pcg_solve(P, Wk, d + j * ld_d, x + static_cast<int64_t>(j) * 3 * P->n_kept,
                                       &alone, &inf[j], s);
        if (st != MM_OK && st != MM_ERR_NO_CONV && st != MM_ERR_NOT_SPD) return st;
      }
    } else {
      MM_TRY(solve_group(P, Wk, d, ld_d, x, cols, tol, max_iter, inf, t, ws, s));
    }
    const double cost = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() / n;
    if (tuning) {
      if (n == group && cost < best_cost) {
        best_cost = cost;
        best = t;
      }
      ++ci;
      if (ci == candidates.size() && best_cost < INFINITY) {
        P->tuned_block = best;
        std::lock_guard<std::mutex> lock(g_tuned_mu);
        g_tuned[shape_of(P)] = best;
      }
    }
    next += n;
  }
  for (int j = 0; j < k; ++j) {
    if (inf[j].converged != 1) return fail(MM_ERR_NO_CONV, "block solve reached max_iter");
  }
  return MM_OK;
}

}  // namespace mm
