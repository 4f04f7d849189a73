// Pointing products on the GPU: un-pointing t = P x and pointing y = P^T u (MAPMAT core
// operations), plus the data mask used for the right-hand side.
//
// Layout: per-sample arrays are separate coalesced streams (local pixel int32, cos/sin FP32);
// each thread owns 8 consecutive samples, read with two 16-byte loads per stream (at any 4-byte
// alignment).  Pixel-domain vectors are FP64 [n_kept][3] and stay cache-resident while the time
// streams go by; the un-pointing loads the pixels of a thread's first and last samples together and
// a third pixel only when one occurs (scan runs make that rare), since these kernels are bound by the
// count and the latency of vector memory instructions rather than by bytes.  P^T accumulates in
// FP64: samples of one pixel arrive in runs (the scan dwells on a pixel for several samples), so each
// thread first sums its own run pieces, then a wavefront segmented scan merges runs that continue
// across lanes, and the completed runs are listed and added by one FP64 atomic per lane.
#include "mm_internal.h"
#include "segment_io.h"
#include "wave_runs.h"

namespace mm {

namespace {

constexpr int kThreads = 256;
constexpr int kLane = 8;
constexpr int kLaneBlock = kThreads * kLane;
constexpr int kListed = 128;                // listed runs per wavefront in the scatter

inline int grid_for(int64_t n, int per_block) {
  int64_t g = (n + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > 65536) g = 65536;
  return static_cast<int>(g);
}

// (Six wavefronts per SIMD: with the compiler's choice of 84 registers for flags and short runs it
// has five, and 2^23 unflagged samples take 21.7 us instead of 21.2; eight spill, 38 us.)
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_unpoint(
    const int32_t* __restrict__ lpix, const float* __restrict__ wq, const float* __restrict__ wu,
    const double* __restrict__ x, float* __restrict__ t, int64_t n,
    const int32_t* __restrict__ done) {
  if (done != nullptr && *done) return;
  const int i = static_cast<int>(threadIdx.x) * kLane;
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * kLaneBlock; base < n;
       base += static_cast<int64_t>(gridDim.x) * kLaneBlock) {
    const int len = n - base < kLaneBlock ? static_cast<int>(n - base) : kLaneBlock;
    float out[kLane];
    gather_lane<kLane, false>(segment_streams(lpix, wq, wu, nullptr, base), x, i, 0, len, out);
    if (i + kLane <= len) {
#pragma unroll
      for (int c = 0; c < kLane; c += 4)
        store4u(t + base + i + c, out[c], out[c + 1], out[c + 2], out[c + 3]);
    } else {
#pragma unroll
      for (int j = 0; j < kLane; ++j)
        if (i + j < len) t[base + i + j] = out[j];
    }
  }
}

// t = d at kept samples, 0 at gap samples (flagged or excised: zero rows of P).
__global__ __launch_bounds__(kThreads) void k_mask_data(const int32_t* __restrict__ lpix,
                                                        const float* __restrict__ d,
                                                        float* __restrict__ t, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * kThreads) {
    t[i] = lpix[i] >= 0 ? d[i] : 0.0f;
  }
}

__global__ __launch_bounds__(kThreads) void k_point(const int32_t* __restrict__ lpix,
                                                    const float* __restrict__ wq,
                                                    const float* __restrict__ wu,
                                                    const float* __restrict__ u,
                                                    double* __restrict__ y, int64_t n,
                                                    const int32_t* __restrict__ done) {
  if (done != nullptr && *done) return;
  const AtomicFlush flush{y};
  // per wavefront: the runs it completes, listed before the atomics
  __shared__ double list[kThreads / 64][run_list_bytes<3, kListed>() / sizeof(double)];
  const int wave = static_cast<int>(threadIdx.x >> 6);
  // Every lane of the block runs the same number of iterations (wavefront-collective scan).
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * kLaneBlock; base < n;
       base += static_cast<int64_t>(gridDim.x) * kLaneBlock) {
    const int i = static_cast<int>(threadIdx.x) * kLane;
    const int len = n - base < kLaneBlock ? static_cast<int>(n - base) : kLaneBlock;
    LanePointing<kLane, false> lane;
    float tv[kLane];
    lane.load(segment_streams(lpix, wq, wu, nullptr, base), i, 0, len);
    if (i + kLane <= len) {
#pragma unroll
      for (int c = 0; c < kLane; c += 4) load4u(u + base + i + c, tv + c);
    } else {
#pragma unroll
      for (int j = 0; j < kLane; ++j) tv[j] = i + j < len ? u[base + i + j] : 0.0f;
    }
    lane.bridge_flags(tv);
    double v[kLane][3];
#pragma unroll
    for (int j = 0; j < kLane; ++j) {
      v[j][0] = tv[j];
      v[j][1] = static_cast<double>(lane.qq[j]) * tv[j];
      v[j][2] = static_cast<double>(lane.uu[j]) * tv[j];
    }
    wave_merge_runs_listed<kLane, 3, kListed>(lane.kk, v, flush, list[wave]);
  }
}

// Diagonal weights: per tile of samples with one weight c_0, y += P^T (c_0 (P x)) or
// y += P^T (c_0 d) with every product in FP64 (no FP32 time-domain intermediate).  Bound by the
// pointing streams: 64 detectors x 2^19 samples 95 us (4.2 TB/s), with 2 % flags 108 us; with
// 4 samples per lane, scalar loads and one round of atomics per lane position 190 and 258 us.
template <bool kFromData>
__global__ __launch_bounds__(kThreads) void k_diag_apply(const int32_t* __restrict__ lpix,
                                                         const float* __restrict__ wq,
                                                         const float* __restrict__ wu,
                                                         const Tile* __restrict__ tiles,
                                                         const double* __restrict__ x,
                                                         const float* __restrict__ d,
                                                         double* __restrict__ y,
                                                         const int32_t* __restrict__ done) {
  if (done != nullptr && *done) return;
  __shared__ double list[kThreads / 64][run_list_bytes<3, kListed>() / sizeof(double)];
  const int wave = static_cast<int>(threadIdx.x >> 6);
  const Tile tl = tiles[blockIdx.x];
  const SegmentStreams tile = segment_streams(lpix, wq, wu, d, tl.start);
  const double c0 = tl.c0;
  for (int i = static_cast<int>(threadIdx.x) * kLane; i - kLane * static_cast<int>(threadIdx.x & 63u) < tl.len;
       i += kLaneBlock) {  // wavefront-uniform
    LanePointing<kLane, false> lane;
    double t[kLane];
    lane.load(tile, i, 0, tl.len);
    if constexpr (kFromData)
      gather_lane<kLane, true>(tile, x, i, 0, tl.len, t);
    else
      lane.resolve(x, t);
    lane.bridge_flags(t);
    double v[kLane][3];
#pragma unroll
    for (int j = 0; j < kLane; ++j) {
      const double tv = t[j] * c0;
      v[j][0] = tv;
      v[j][1] = static_cast<double>(lane.qq[j]) * tv;
      v[j][2] = static_cast<double>(lane.uu[j]) * tv;
    }
    wave_merge_runs_listed<kLane, 3, kListed>(lane.kk, v, AtomicFlush{y}, list[wave]);
  }
}

__global__ void k_zero(double* __restrict__ y, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    y[i] = 0.0;
}

}  // namespace

mm_status launch_diag_tiles(Plan* P, const Tile* tiles, int32_t n_tiles, const double* x,
                            const float* d, double* y, const int32_t* done, hipStream_t s) {
  if (n_tiles == 0 || P->n_kept == 0) return MM_OK;
  TimedLaunch tl(P, K_POINT, s);
  if (x != nullptr)
    hipLaunchKernelGGL(k_diag_apply<false>, dim3(n_tiles), dim3(kThreads), 0, s, P->lpix, P->wq,
                       P->wu, tiles, x, d, y, done);
  else
    hipLaunchKernelGGL(k_diag_apply<true>, dim3(n_tiles), dim3(kThreads), 0, s, P->lpix, P->wq,
                       P->wu, tiles, x, d, y, done);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

mm_status launch_diag_apply(Plan* P, const double* x, const float* d, double* y,
                            const int32_t* done, hipStream_t s) {
  return launch_diag_tiles(P, P->tiles, P->n_tiles, x, d, y, done, s);
}

mm_status launch_zero(double* y, int64_t n, hipStream_t s) {
  if (n <= 0) return MM_OK;
  int64_t g = (n + 255) / 256;
  if (g > 16384) g = 16384;
  hipLaunchKernelGGL(k_zero, dim3(static_cast<unsigned>(g)), dim3(256), 0, s, y, n);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

mm_status launch_unpoint(Plan* P, const double* x, float* t, const int32_t* done,
                         hipStream_t s) {
  const int64_t n = P->n_samples;
  if (n == 0) return MM_OK;
  TimedLaunch tl(P, K_UNPOINT, s);
  hipLaunchKernelGGL(k_unpoint, dim3(grid_for(n, kLaneBlock)), dim3(kThreads), 0, s, P->lpix,
                     P->wq, P->wu, x, t, n, done);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

mm_status launch_mask_data(Plan* P, const float* d, float* t, hipStream_t s) {
  const int64_t n = P->n_samples;
  if (n == 0) return MM_OK;
  int64_t g = (n + kThreads - 1) / kThreads;
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(k_mask_data, dim3(static_cast<unsigned>(g)), dim3(kThreads), 0, s, P->lpix,
                     d, t, n);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

mm_status launch_point(Plan* P, const float* u, double* y, bool zero_first, const int32_t* done,
                       hipStream_t s) {
  if (zero_first) MM_TRY(launch_zero(y, 3 * P->n_kept, s));
  const int64_t n = P->n_samples;
  if (n == 0 || P->n_kept == 0) return MM_OK;
  TimedLaunch tl(P, K_POINT, s);
  hipLaunchKernelGGL(k_point, dim3(grid_for(n, kLaneBlock)), dim3(kThreads), 0, s, P->lpix,
                     P->wq, P->wu, u, y, n, done);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

}  // namespace mm
