// Block-diagonal banded Toeplitz product u = N^-1 t (Toeplitz algebra package: stbmm).
//
// FFT path (shift-and-overlap, Toeplitz product paragraph): each workgroup owns one segment of
// one stationary interval: N real inputs [out0 - lambda, out0 - lambda + N), zero outside the
// interval (truncation at block edges), producing N - 2 lambda outputs.  The N real samples
// are packed as N/2 complex points (even samples real, odd imaginary) and transformed in LDS
// by a radix-16/8/4/2 Stockham FFT; the half-length spectrum is unpacked into the real
// spectrum, multiplied by the band's symbol (real because the band is symmetric), repacked,
// and transformed back (inverse = conjugate of the forward transform of the conjugate).  All
// arithmetic is FP32; twiddles come from a two-level table (exp(-2 pi i m / N) =
// coarse[m >> 7] * fine[m & 127]) computed in FP64 on the host.  The symbol is precomputed per
// band at plan time with the 1/(2N) normalisation folded in.
//
// Segments of 2^15 samples with at most 2^14 outputs take the register-resident transform
// (apply_reg.hip), short bands the direct product (direct.hip), segments of 2^16 and 2^17 the
// four-step one (toeplitz_long.hip).
#include "fft_lds.h"
#include "mm_internal.h"
#include "segment_io.h"

namespace mm {

namespace {

using namespace fft;

template <int LOG>
__global__ __launch_bounds__(FftCfg<LOG>::T) void k_toeplitz_fft(
    const float* __restrict__ t, float* __restrict__ u, const Chunk* __restrict__ chunks,
    const float* __restrict__ spec, const float2* __restrict__ tw0g,
    const float2* __restrict__ tw1g, int lam, const int32_t* __restrict__ done) {
  using C = FftCfg<LOG>;
  constexpr int NC = C::NC, N = C::N, T = C::T;
  __shared__ float2 buf[C::LDS];
  __shared__ float2 tw0[128];
  __shared__ float2 tw1[N / 128];
  if (done != nullptr && *done) return;
  const int tid = threadIdx.x;
  for (int i = tid; i < 128; i += T) tw0[i] = tw0g[i];
  for (int i = tid; i < N / 128; i += T) tw1[i] = tw1g[i];

  const Chunk c = chunks[xcd_ordered(blockIdx.x, gridDim.x)];
  const float* __restrict__ in = t + (c.out0 - lam);
  int lo, hi;
  window_range(c, lam, N, lo, hi);
  for (int p = tid; p < NC; p += T) {  // sample pairs: complex points
    const int i = 2 * p;
    if (i >= lo && i + 2 <= hi)
      buf[pad(p)] = load2u(in + static_cast<uint32_t>(i));
    else
      buf[pad(p)] = make_float2(i >= lo && i < hi ? in[i] : 0.0f,
                                i + 1 >= lo && i + 1 < hi ? in[i + 1] : 0.0f);
  }
  __syncthreads();
  fft_forward<LOG, T>(buf, tw0, tw1);
  symbol_multiply<LOG, T>(buf, spec + static_cast<int64_t>(c.band) * (NC + 1), tw0, tw1);
  fft_forward<LOG, T>(buf, tw0, tw1);
  // outputs are y[lam .. lam + out_len)
  float* __restrict__ out = u + c.out0;
  for (int o = 2 * tid; o < c.out_len; o += 2 * T) {
    if (o + 1 < c.out_len)
      store2u(out + static_cast<uint32_t>(o), real_out(buf, lam + o), real_out(buf, lam + o + 1));
    else
      out[o] = real_out(buf, lam + o);
  }
}

// Identity rows (samples outside every block): u = t.
__global__ __launch_bounds__(256) void k_copy_segments(const float* __restrict__ t,
                                                       float* __restrict__ u,
                                                       const int64_t* __restrict__ seg,
                                                       const int32_t* __restrict__ done) {
  if (done != nullptr && *done) return;
  const int64_t s0 = seg[2 * blockIdx.x], len = seg[2 * blockIdx.x + 1];
  for (int64_t i = threadIdx.x; i < len; i += 256) u[s0 + i] = t[s0 + i];
}

template <int LOG>
mm_status launch_fft(Plan* P, const float* t, float* u, const int32_t* done, hipStream_t s) {
  using C = FftCfg<LOG>;
  hipLaunchKernelGGL(k_toeplitz_fft<LOG>, dim3(P->n_chunks), dim3(C::T), 0, s, t, u, P->chunks,
                     P->spec, P->tw0, P->tw1, P->lambda_max, done);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

}  // namespace

bool fft_size_supported(int32_t n) {
  return n == (1 << 11) || n == (1 << 12) || n == (1 << 13) || n == (1 << 14) ||
         n == (1 << 15) || long_fft_size(n);
}

int32_t choose_fft_size(int32_t lambda_max) {
  // Smallest power of two >= 4 lambda (at least half of every segment is output).  Up to 2^15
  // the segment fits one CU's LDS; bands a little longer still use 2^15 while at least 8,192
  // outputs per segment remain; longer bands go to the four-step kernel (up to 2^17).
  int64_t n = 1 << 11;
  while (n < 4 * static_cast<int64_t>(lambda_max)) n *= 2;
  if (n <= (1 << 15)) return static_cast<int32_t>(n);
  if ((1 << 15) - 2 * static_cast<int64_t>(lambda_max) >= 8192) return 1 << 15;
  if (n <= (1 << 17)) return static_cast<int32_t>(n);
  if ((1 << 17) - 2 * static_cast<int64_t>(lambda_max) >= 16384) return 1 << 17;
  return 0;
}

mm_status launch_noise_weight(Plan* P, const float* t, float* u, float2* scratch,
                              const int32_t* done, hipStream_t s) {
  if (P->n_samples == 0) return MM_OK;
  TimedLaunch tl(P, K_TOEPLITZ, s);
  if (P->n_chunks > 0) {
    if (P->algo == MM_TOEPLITZ_FFT && long_fft_size(P->fft_n)) {
      MM_TRY(launch_toeplitz_long(P, t, u, scratch, done, s));
    } else if (P->algo == MM_TOEPLITZ_FFT && P->reg_fft) {
      MM_TRY(launch_toeplitz_reg(P, t, u, done, s));
    } else if (P->algo == MM_TOEPLITZ_FFT) {
      switch (P->fft_n) {
        case 1 << 11: MM_TRY(launch_fft<10>(P, t, u, done, s)); break;
        case 1 << 12: MM_TRY(launch_fft<11>(P, t, u, done, s)); break;
        case 1 << 13: MM_TRY(launch_fft<12>(P, t, u, done, s)); break;
        case 1 << 14: MM_TRY(launch_fft<13>(P, t, u, done, s)); break;
        case 1 << 15: MM_TRY(launch_fft<14>(P, t, u, done, s)); break;
        default: return fail(MM_ERR_UNSUPPORTED, "FFT size not supported");
      }
    } else {
      MM_TRY(launch_toeplitz_direct(P, t, u, done, s));
    }
  }
  if (P->n_id_seg > 0) {
    hipLaunchKernelGGL(k_copy_segments, dim3(P->n_id_seg), dim3(256), 0, s, t, u, P->id_seg, done);
    MM_HIP_TRY(hipGetLastError());
  }
  return MM_OK;
}

}  // namespace mm
