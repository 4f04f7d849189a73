// Fused system product for the FFT path: one workgroup per overlap-save segment does
//
//   gather   t = P x (FP64 sums rounded to FP32) or t = d at kept samples, straight into LDS
//   Toeplitz u = N^-1 t by the LDS real FFT (shift-and-overlap segment, Toeplitz package)
//   scatter  y += P^T u for the segment's outputs, FP64, run-merged atomics
//
// so the time-domain vectors never go to HBM: per output sample the kernel reads the pointing
// of its input window (12 B per window sample, the lambda halo included) and again for its
// outputs, and issues the run-merged atomics.  Samples outside every block (identity rows of
// stbmm) are handled by the diagonal kernel over identity tiles.
//
// The gather is bound by the number of vector memory instructions, not by bytes: a lane takes
// 8 consecutive samples (two 16-byte loads per pointing array) and loads a pixel's three values
// only when the pixel changes, which scan runs make rare.  On small problems, with one or two
// wavefronts to a segment and a segment to a CU, its waits count: two rounds are in flight.
// Rates: 64 detectors x 2^19 samples on 16-sample runs, lambda = 1000 (N = 4096) 222 us; 61
// detectors x 200,003 samples on 7-sample runs with 2 % flags, lambda = 2047, 94 us (254 us with
// scalar loads where windows start unaligned and runs flushed where they end).
#include "fft_lds.h"
#include "mm_internal.h"
#include "segment_io.h"
#include "wave_runs.h"

namespace mm {

namespace {

using namespace fft;

// Consecutive samples per lane in the gather and in the scatter.  Wider lanes issue fewer,
// wider memory instructions and load a pixel's values once per run; 8 is the widest that
// 1,024-thread workgroups (128 registers per lane) hold without spilling.
constexpr int kGatherLane = 8;
constexpr int kScatterLane = 8;

// Runs listed per wavefront and scatter round.  The list lives in the wavefront's own outputs, which
// it has read by then: from the complex point after its slice's first (with odd lambda the first
// and last are shared with the neighbouring wavefronts) on.  A slice that starts within 256
// samples of the window's end may reach past it: at most kListSlack points.
constexpr int kListed = 64;
constexpr int kListSlack = 96;
constexpr int kReadSlack = 8;  // points that the last output's lane reads past the window
constexpr int kListPoints = run_list_bytes<3, kListed>() / static_cast<int>(sizeof(float2));
static_assert(run_list_bytes<3, kListed>() <= 254 * sizeof(float2),
              "run list must fit between the shared points of a slice");

template <int LOG, bool kFromData>
__global__ __launch_bounds__(FftCfg<LOG>::T) void k_apply_fused(
    const int32_t* __restrict__ lpix, const float* __restrict__ wq, const float* __restrict__ wu,
    const double* __restrict__ x0, const float* __restrict__ d0, double* __restrict__ y0,
    int ncol, int64_t ldx, int64_t ldy, const Chunk* __restrict__ chunks,
    const float* __restrict__ spec,
    const float2* __restrict__ tw0g, const float2* __restrict__ tw1g, int lam,
    const int32_t* __restrict__ done) {
  using C = FftCfg<LOG>;
  constexpr int NC = C::NC, N = C::N, T = C::T;
  constexpr int kBuf = C::LDS + (T > 64 ? kListSlack : kReadSlack);
  __shared__ float2 buf[kBuf];
  __shared__ float2 tw0[128];
  __shared__ float2 tw1[N / 128];
  if (done != nullptr && *done) return;
  const int tid = threadIdx.x;
  for (int i = tid; i < 128; i += T) tw0[i] = tw0g[i];
  for (int i = tid; i < N / 128; i += T) tw1[i] = tw1g[i];

  // workgroup -> (segment, column), columns fastest: an XCD runs all columns of a segment
  // back to back, so the pointing re-reads of the later columns hit its L2
  const int wg = xcd_ordered(blockIdx.x, gridDim.x);
  const int col = wg % ncol;
  const Chunk c = chunks[wg / ncol];
  const double* __restrict__ x = kFromData ? x0 : x0 + col * ldx;
  const float* __restrict__ d = kFromData ? d0 + col * ldx : d0;
  double* __restrict__ y = y0 + col * ldy;
  const SegmentStreams win = segment_streams(lpix, wq, wu, d, c.out0 - lam);
  int lo, hi;
  window_range(c, lam, N, lo, hi);

  // ---- gather the N-sample window (zero outside the block) ---------------------------------
  // Four rounds of T SG samples, one window quarter each.  With N = 4 lambda the right half of
  // the window is the left half of the next segment's, and neighbouring segments run at the
  // same time on one XCD: even segments gather their right half first, odd ones their left
  // half first, so both readers of a shared half fetch it together and the second finds it in
  // L2.
  constexpr int SG = kGatherLane;
  // Two rounds' loads in flight where registers allow (LOG = 14 has 128 and uses them all): at
  // lambda = 512, 18 detectors x 2^17 samples, a solve takes 1,236 us against 1,264 with one; all
  // four at once take 208 registers and 1,477 us.
  constexpr int kDeep = LOG <= 13 ? 2 : 1;
  // Scans aligned to the lanes (one pixel a lane) have one sum per sample instead of two, where the
  // branch costs no registers that matter: in 1,024-thread workgroups, which are capped at 128 and,
  // one to a CU, bound by vector instructions.  256 detectors x 2^20 samples on 16-sample runs,
  // lambda = 8000 2,172 -> 2,078 us, 6000 2,279 -> 2,195 us; smaller workgroups would pass 128
  // registers and lose a wavefront per SIMD (lambda = 4000 1,746 -> 2,577 us).  In the scatter it
  // costs none anywhere (lambda = 2000 1,524 -> 1,486 us, 500 1,517 -> 1,475 us).
  constexpr bool kOnePixel = LOG == 14;
  static_assert(N == 4 * T * SG, "four gather rounds");
  const int rot = ((wg / ncol) & 1) == 0 ? 2 : 0;
  for (int rr = 0; rr < 4; rr += kDeep) {
    LanePointing<SG, kFromData> lane[kDeep];
    typename LanePointing<SG, kFromData>::Pixels px[kDeep];
    int n[kDeep];
#pragma unroll
    for (int e = 0; e < kDeep; ++e) {
      n[e] = ((rr + e + rot) & 3) * (T * SG) + tid * SG;
      lane[e].load(win, n[e], lo, hi);
    }
#pragma unroll
    for (int e = 0; e < kDeep; ++e) lane[e].fetch(x, px[e]);
#pragma unroll
    for (int e = 0; e < kDeep; ++e) {
      float v[SG];
      lane[e].template finish<kOnePixel>(x, px[e], v);
      // samples n..n+SG-1 are complex points n/2.. (n/2 even: contiguous pairs after padding)
      float2* dst = buf + pad(n[e] >> 1);
#pragma unroll
      for (int j = 0; j < SG / 2; ++j) dst[j] = make_float2(v[2 * j], v[2 * j + 1]);
    }
  }
  __syncthreads();

  // ---- Toeplitz product in LDS ----------------------------------------------------------------
  fft_forward<LOG, T>(buf, tw0, tw1);
  symbol_multiply<LOG, T>(buf, spec + static_cast<int64_t>(c.band) * (NC + 1), tw0, tw1);
  fft_forward<LOG, T>(buf, tw0, tw1);

  // ---- scatter the segment's outputs ----------------------------------------------------------
  constexpr int SS = kScatterLane;
  const AtomicFlush flush{y};
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (wavefronts past the last output have nothing to do in the last round)
  for (int base = 0; base + 64 * SS * wave < c.out_len; base += T * SS) {
    const int i0 = base + tid * SS;
    LanePointing<SS, false> lane;
    lane.load(win, lam + i0, lam, lam + c.out_len);
    // the lane's outputs: window samples lam + i0 on, two to a point (samples past the last output
    // have no pixel, and bridge_flags clears their values)
    float2 z[SS / 2 + 1];
#pragma unroll
    for (int q = 0; q <= SS / 2; ++q) z[q] = make_float2(0.0f, 0.0f);
    if (i0 < c.out_len) {
#pragma unroll
      for (int q = 0; q <= SS / 2; ++q) z[q] = buf[pad(((lam + i0) >> 1) + q)];
    }
    float u[SS];
    if (lam & 1) {  // uniform
#pragma unroll
      for (int q = 0; q < SS / 2; ++q) {
        u[2 * q] = -z[q].y;
        u[2 * q + 1] = z[q + 1].x;
      }
    } else {
#pragma unroll
      for (int q = 0; q < SS / 2; ++q) {
        u[2 * q] = z[q].x;
        u[2 * q + 1] = -z[q].y;
      }
    }
    lane.bridge_flags(u);
    int at = pad(((lam + base + 64 * SS * wave) >> 1) + 1);
    if constexpr (T == 64) at = min(at, kBuf - kListPoints);
    wave_point_runs<SS, kListed, true>(lane.kk, lane.qq, lane.uu, u, flush, buf + at);
  }
}

template <int LOG>
mm_status launch(Plan* P, const double* x, const float* d, int64_t ldx, double* y, int64_t ldy,
                 int ncol, const int32_t* done, hipStream_t s) {
  using C = FftCfg<LOG>;
  const int64_t grid = static_cast<int64_t>(P->n_chunks) * ncol;
  if (grid > INT32_MAX) return fail(MM_ERR_UNSUPPORTED, "too many segment x column workgroups");
  if (d != nullptr) {
    hipLaunchKernelGGL((k_apply_fused<LOG, true>), dim3(static_cast<unsigned>(grid)), dim3(C::T), 0,
                       s, P->lpix, P->wq, P->wu, x, d, y, ncol, ldx, ldy, P->chunks,
                       P->spec, P->tw0, P->tw1, P->lambda_max, done);
  } else {
    hipLaunchKernelGGL((k_apply_fused<LOG, false>), dim3(static_cast<unsigned>(grid)), dim3(C::T), 0,
                       s, P->lpix, P->wq, P->wu, x, d, y, ncol, ldx, ldy, P->chunks,
                       P->spec, P->tw0, P->tw1, P->lambda_max, done);
  }
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

}  // namespace

mm_status launch_apply_fused(Plan* P, const double* x, const float* d, double* y,
                             const int32_t* done, hipStream_t s, float2* tiles, int32_t ncol,
                             int64_t ldx, int64_t ldy) {
  if (P->n_kept == 0 || ncol <= 0) return MM_OK;
  if (ldx == 0) ldx = d != nullptr ? P->n_samples : 3 * P->n_kept;
  if (ldy == 0) ldy = 3 * P->n_kept;
  if (P->n_chunks > 0 && long_fft_size(P->fft_n)) {
    TimedLaunch tl(P, K_TOEPLITZ, s);
    MM_TRY(launch_apply_long(P, x, d, ldx, y, ldy, ncol, tiles, done, s));
  } else if (P->n_chunks > 0 && P->reg_fft) {
    TimedLaunch tl(P, K_TOEPLITZ, s);
    MM_TRY(launch_apply_reg(P, x, d, ldx, y, ldy, ncol, done, s));
  } else if (P->n_chunks > 0) {
    TimedLaunch tl(P, K_TOEPLITZ, s);
    switch (P->fft_n) {
      case 1 << 11: MM_TRY(launch<10>(P, x, d, ldx, y, ldy, ncol, done, s)); break;
      case 1 << 12: MM_TRY(launch<11>(P, x, d, ldx, y, ldy, ncol, done, s)); break;
      case 1 << 13: MM_TRY(launch<12>(P, x, d, ldx, y, ldy, ncol, done, s)); break;
      case 1 << 14: MM_TRY(launch<13>(P, x, d, ldx, y, ldy, ncol, done, s)); break;
      case 1 << 15: MM_TRY(launch<14>(P, x, d, ldx, y, ldy, ncol, done, s)); break;
      default: return fail(MM_ERR_UNSUPPORTED, "FFT size not supported");
    }
  }
  if (P->n_id_tiles > 0) {
    for (int32_t j = 0; j < ncol; ++j)
      MM_TRY(launch_diag_tiles(P, P->id_tiles, P->n_id_tiles, d ? nullptr : x + j * ldx,
                               d ? d + j * ldx : nullptr, y + j * ldy, done, s));
  }
  return MM_OK;
}

}  // namespace mm
