// Direct banded Toeplitz products for short bands, in two forms:
//
//   plain  u = N^-1 t for FP32 time-domain vectors in HBM (the stand-alone N^-1 t product)
//   fused  y += P^T N^-1 (P x) or y += P^T N^-1 d, one workgroup per tile of 1,024 outputs: the
//          gather fills the tile's window in LDS and the run-merged FP64 scatter drains the sums,
//          so the time-domain vectors never go to HBM
//
// y_i = c_0 x_i + sum_k c_k (x_{i-k} + x_{i+k}) in FP32, k ascending.  A thread forms 8
// consecutive outputs (the scatter's lane): for eight values of k the left and the right window
// are 15 samples each, of which 8 are new per eight k, so a sample read from LDS serves 8 outputs
// (one output per thread and k read two samples for every multiply-add).  The window is padded
// by one slot per 8 samples: lanes 8 samples apart then hit different banks.  Samples outside
// every block are tiles with band -1 (identity rows, c_0 = 1).
//
// FP64 plans take the fused form with window, sums and map products in FP64: 64 detectors x 2^20
// samples, lambda = 32, 2,097 us with 4 outputs per thread, two window samples read per
// multiply-add, and one load at a time in the gather; 396 us here (lambda = 8: 740 and 284).
//
// Bound by the pointing's bytes at short bands (lambda = 16: 12 B against 50 multiply-adds a
// sample).  64 detectors x 2^18 samples, lambda = 16: 188 us for the three kernels (un-pointing
// 44, direct product 95, pointing 47) before, 73 us fused.
#include <algorithm>

#include "mm_internal.h"
#include "segment_io.h"
#include "wave_runs.h"

namespace mm {

namespace {

constexpr int kTile = 1024;     // outputs per workgroup
constexpr int kLane = 8;        // consecutive samples per thread
constexpr int kThreads = kTile / kLane;
constexpr int kWaves = kThreads / 64;
constexpr int kListed = 64;     // runs listed per wavefront
constexpr int kMaxLambda = 4096;

enum DirectIo { kIoPlain = 0, kIoApply = 1, kIoRhs = 2 };

struct DirectArgs {
  const float* t;  // plain: input and output vectors
  float* u;
  const int32_t* lpix;  // fused: pointing, map(s) or data, accumulated output map(s)
  const float* wq;
  const float* wu;
  const double* x0;
  const float* d0;
  double* y0;
  int64_t ldx, ldy;
  int ncol;
  const Chunk* tiles;
  const float* coef;
  const int64_t* off;
  const int32_t* ncoef;
  const int32_t* done;
};

__device__ __forceinline__ int slot(int i) { return i + (i >> 3); }

// LDS bytes: the window of a tile with 8 samples before and after it (the last round of sums reads
// up to 7 past either end), or the run lists that replace it.
template <class T>
inline size_t lds_bytes(int lambda) {
  const int window = (kTile + 2 * lambda + kLane - 1) / kLane + 2;
  return std::max<size_t>(sizeof(T) * static_cast<size_t>(window * (kLane + 1)),
                          kWaves * run_list_bytes<3, kListed>());
}

__device__ __forceinline__ float mul_add(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double mul_add(double a, double b, double c) { return fma(a, b, c); }

template <int IO, class T>
__global__ __launch_bounds__(kThreads) void k_direct(const DirectArgs a) {
  extern __shared__ __align__(16) char lds[];
  T* xs = reinterpret_cast<T*>(lds);
  if (a.done != nullptr && *a.done) return;
  const int tid = threadIdx.x;
  const int col = static_cast<int>(blockIdx.x) % a.ncol;
  const Chunk c = a.tiles[static_cast<int>(blockIdx.x) / a.ncol];
  const int lam = c.band < 0 ? 0 : a.ncoef[c.band] - 1;
  const float* __restrict__ coef = c.band < 0 ? nullptr : a.coef + a.off[c.band];
  const double* __restrict__ x = IO == kIoApply ? a.x0 + col * a.ldx : nullptr;
  const float* __restrict__ d = IO == kIoRhs ? a.d0 + col * a.ldx : nullptr;
  const SegmentStreams win =
      segment_streams(a.lpix, a.wq, a.wu, IO == kIoPlain ? a.t : d, c.out0 - lam);
  const int nin = c.out_len + 2 * lam;
  int lo, hi;
  window_range(c, lam, nin, lo, hi);

  // ---- window: sample out0 - lam + i at slot(i + 8), zero outside the block -----------------
  for (int i = tid * kLane; i < nin; i += kTile) {
    T v[kLane];
    if constexpr (IO == kIoPlain) {
      if (i >= lo && i + kLane <= hi) {
        load4u(win.d + static_cast<uint32_t>(i), v);
        load4u(win.d + static_cast<uint32_t>(i + 4), v + 4);
      } else {
#pragma unroll
        for (int j = 0; j < kLane; ++j) v[j] = i + j >= lo && i + j < hi ? win.d[i + j] : 0.0f;
      }
    } else {
      gather_lane<kLane, IO == kIoRhs>(win, x, i, lo, hi, v);
    }
#pragma unroll
    for (int j = 0; j < kLane; ++j) xs[slot(i + kLane) + j] = v[j];
  }
  __syncthreads();

  // ---- sums: outputs o .. o + 7 of the tile ---------------------------------------------------
  // at(i) is window sample o + i; i is uniform, so lanes sit 9 slots apart.  Samples before the
  // window's first or past its last are read (slots of the padding, or whatever a shorter tile
  // left there) only into sums that no output uses.
  const int o = tid * kLane;
  const T* mine = xs + (kLane + 1) * tid;
  auto at = [&](int i) { return mine[slot(i + kLane)]; };
  const T c0 = coef != nullptr ? coef[0] : 1.0f;
  T acc[kLane];
#pragma unroll
  for (int j = 0; j < kLane; ++j) acc[j] = c0 * at(lam + j);
  // a round's k0 .. k0 + 7: left[i] = at(lam - k0 - 7 + i), right[i] = at(lam + k0 + i), i < 15
  T left[2 * kLane - 1], right[2 * kLane - 1];
#pragma unroll
  for (int j = 0; j < kLane - 1; ++j) {
    left[kLane + j] = at(lam + j);
    right[j] = at(lam + 1 + j);
  }
  for (int k0 = 1; k0 <= lam; k0 += kLane) {
#pragma unroll
    for (int j = 0; j < kLane; ++j) {
      left[j] = at(lam - k0 - (kLane - 1) + j);
      right[kLane - 1 + j] = at(lam + k0 + (kLane - 1) + j);
    }
#pragma unroll
    for (int m = 0; m < kLane; ++m) {
      if (k0 + m <= lam) {
        const T ck = coef[k0 + m];
#pragma unroll
        for (int j = 0; j < kLane; ++j)
          acc[j] = mul_add(ck, left[kLane - 1 + j - m] + right[j + m], acc[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < kLane - 1; ++j) {
      left[kLane + j] = left[j];
      right[j] = right[kLane + j];
    }
  }

  if constexpr (IO == kIoPlain) {
    if (o + kLane <= c.out_len) {
      store4u(a.u + c.out0 + o, acc[0], acc[1], acc[2], acc[3]);
      store4u(a.u + c.out0 + o + 4, acc[4], acc[5], acc[6], acc[7]);
    } else {
#pragma unroll
      for (int j = 0; j < kLane; ++j)
        if (o + j < c.out_len) a.u[c.out0 + o + j] = acc[j];
    }
  } else {
    LanePointing<kLane, false> lane;
    lane.load(win, lam + o, lam, lam + c.out_len);
    lane.bridge_flags(acc);
    double val[kLane][3];
#pragma unroll
    for (int j = 0; j < kLane; ++j) {
      const double tv = acc[j];
      val[j][0] = tv;
      val[j][1] = static_cast<double>(lane.qq[j]) * tv;
      val[j][2] = static_cast<double>(lane.uu[j]) * tv;
    }
    __syncthreads();  // the window has been read: its LDS holds the run lists
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    wave_merge_runs_listed<kLane, 3, kListed>(
        lane.kk, val, AtomicFlush{a.y0 + col * a.ldy},
        lds + wave * run_list_bytes<3, kListed>());
  }
}

template <int IO, class T>
mm_status launch(Plan* P, const DirectArgs& a, int64_t n_tiles, hipStream_t s) {
  const int64_t grid = n_tiles * a.ncol;
  if (grid > INT32_MAX) return fail(MM_ERR_UNSUPPORTED, "too many tile x column workgroups");
  const size_t lds = lds_bytes<T>(P->lambda_max);
  if (lds > 64 * 1024)  // FP64 windows of lambda > 3,000
    MM_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_direct<IO, T>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                   static_cast<int>(lds)));
  hipLaunchKernelGGL((k_direct<IO, T>), dim3(static_cast<unsigned>(grid)), dim3(kThreads), lds, s,
                     a);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

DirectArgs base_args(Plan* P, const int32_t* done) {
  DirectArgs a{};
  a.lpix = P->lpix;
  a.wq = P->wq;
  a.wu = P->wu;
  a.coef = P->band_coef;
  a.off = P->band_off;
  a.ncoef = P->band_ncoef;
  a.tiles = P->chunks;
  a.done = done;
  a.ncol = 1;
  return a;
}

}  // namespace

int32_t max_direct_lambda() { return kMaxLambda; }

int32_t direct_tile() { return kTile; }

mm_status launch_toeplitz_direct(Plan* P, const float* t, float* u, const int32_t* done,
                                 hipStream_t s) {
  DirectArgs a = base_args(P, done);
  a.t = t;
  a.u = u;
  return launch<kIoPlain, float>(P, a, P->n_chunks, s);
}

mm_status launch_apply_direct(Plan* P, const double* x, const float* d, double* y,
                              const int32_t* done, hipStream_t s, int32_t ncol, int64_t ldx,
                              int64_t ldy, bool fp64) {
  const int64_t n_tiles = static_cast<int64_t>(P->n_chunks) + P->n_id_chunks;
  if (P->n_kept == 0 || ncol <= 0 || n_tiles == 0) return MM_OK;
  TimedLaunch tl(P, K_TOEPLITZ, s);
  DirectArgs a = base_args(P, done);
  a.x0 = x;
  a.d0 = d;
  a.y0 = y;
  a.ldx = ldx != 0 ? ldx : (d != nullptr ? P->n_samples : 3 * P->n_kept);
  a.ldy = ldy != 0 ? ldy : 3 * P->n_kept;
  a.ncol = ncol;
  if (fp64)
    return d != nullptr ? launch<kIoRhs, double>(P, a, n_tiles, s)
                        : launch<kIoApply, double>(P, a, n_tiles, s);
  return d != nullptr ? launch<kIoRhs, float>(P, a, n_tiles, s)
                      : launch<kIoApply, float>(P, a, n_tiles, s);
}

}  // namespace mm
