// Fused system product for 2^15-sample overlap-save segments with a register-resident FFT.
//
// Same operation as the LDS-resident fused kernel (gather t = P x, Toeplitz u = N^-1 t by the
// real FFT of the segment, scatter y += P^T u over the segment's outputs), laid out so that
// two workgroups share a CU: 512 threads each hold 32 of the 16,384 complex points in
// registers, and LDS (about 77 KB per workgroup) only stages the gather, the transposes between
// the three radix steps and the outputs.  While one workgroup waits on its gather or scatter
// the other keeps the vector ALUs busy with its transforms, which a single 142 KB workgroup
// per CU cannot do.
//
// Transform (NC = 16384 points z[n] = t[2n] + i t[2n+1], n = n1 + 16 n2 + 512 j,
// k = k3 + 32 k2 + 1024 k1):
//   A  thread t = n1 + 16 n2 holds z[t + 512 j], j < 32: radix-32 over j, twiddle W_NC^(t k3)
//   B  thread (k3, n1) holds slot n2:                  radix-32 over n2, twiddle W_512^(n1 k2)
//   C  thread holds two tasks (k3, k2), slot n1:       radix-16 over n1 -> Z[k], k1 < 16
// The two tasks of a thread are chosen so that the partner bin NC - k of each of its bins is
// also in the thread, so the real-spectrum step (unpack, band symbol, repack) stays in
// registers.  The inverse runs the same steps transposed (C, B, A with the same twiddles):
// the transposed factorisation of the symmetric DFT matrix is the DFT again, so it maps the
// repacked spectrum back to the natural order that the first step read.
#include "fft_lds.h"
#include "mm_internal.h"
#include "segment_io.h"
#include "wave_runs.h"

namespace mm {

namespace {

using namespace fft;

constexpr int kT = 512;            // threads per workgroup
constexpr int kNC = 16384;         // complex points per segment
constexpr int kN = 2 * kNC;        // real samples per segment
constexpr int kHalf = kNC;         // window samples staged per gather half; outputs at most
constexpr int kRowA = 528;         // LDS stride of a k3 row in the A <-> B transposes
constexpr int kRowB = 560;         // LDS stride of a k3 plane in the B <-> C transposes (measured:
                                   // 39 % fewer bank conflicts than 544)
constexpr int kLdsF = 32 * kRowB;  // floats of staging LDS
constexpr int kLane = 8;           // consecutive samples per lane in the gather and scatter
constexpr int kListed = 64;        // runs listed per wavefront and scatter round
constexpr int kTab = 16 * kT + 8;  // symbol pairs per band in the kernel's read order
constexpr int kW2 = 33;            // row stride of the W_512 table

typedef __attribute__((address_space(1))) const void* global_ptr;
typedef __attribute__((address_space(3))) void* lds_ptr;

// Direct load of 16 B per lane from global memory into LDS at (wave-uniform) wave_base +
// 16 B x lane, without passing through registers.
__device__ __forceinline__ void load_to_lds16(const void* src, void* wave_base) {
  __builtin_amdgcn_global_load_lds((global_ptr)src, (lds_ptr)wave_base, 16, 0, 0);
}

// Tasks of a thread in the C layout: (a3, a2) and its mirror (b3, b2).
__device__ __forceinline__ void reg_tasks(int tid, int& a3, int& a2, int& b3, int& b2) {
  if (tid >= 32) {
    a3 = tid >> 5;
    a2 = tid & 31;
    b3 = 32 - a3;
    b2 = 31 - a2;
  } else if (tid >= 16) {
    a3 = 16;
    a2 = tid - 16;
    b3 = 16;
    b2 = 47 - tid;
  } else {
    a3 = 0;
    a2 = tid;
    b3 = 0;
    b2 = tid == 0 ? 16 : 32 - tid;
  }
}

// cos and sin of 2 pi k / 32, k < 16
__device__ constexpr float kCos32[16] = {
    1.0f, 0.98078528040323043f, 0.92387953251128674f, 0.83146961230254524f,
    0.70710678118654752f, 0.55557023301960218f, 0.38268343236508978f, 0.19509032201612827f,
    0.0f, -0.19509032201612827f, -0.38268343236508978f, -0.55557023301960218f,
    -0.70710678118654752f, -0.83146961230254524f, -0.92387953251128674f, -0.98078528040323043f};
__device__ constexpr float kSin32[16] = {
    0.0f, 0.19509032201612827f, 0.38268343236508978f, 0.55557023301960218f,
    0.70710678118654752f, 0.83146961230254524f, 0.92387953251128674f, 0.98078528040323043f,
    1.0f, 0.98078528040323043f, 0.92387953251128674f, 0.83146961230254524f,
    0.70710678118654752f, 0.55557023301960218f, 0.38268343236508978f, 0.19509032201612827f};

// Radix-32 DFT on v[0..32) in natural order: two radix-16 DFTs (even and odd points) and a
// radix-2 step with W_32^k.
__device__ __forceinline__ void dft32(float2 (&v)[32]) {
  float2 e[16], o[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    e[i] = v[2 * i];
    o[i] = v[2 * i + 1];
  }
  dft<16>(e);
  dft<16>(o);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const float2 E = e[out_slot<16>(k)];
    float2 O = o[out_slot<16>(k)];
    if (k == 8)
      O = mul_mi(O);
    else if (k != 0)
      O = cmul(O, make_float2(kCos32[k], -kSin32[k]));
    v[k] = cadd(E, O);
    v[k + 16] = csub(E, O);
  }
}

// The middle half (outputs 8..23) of the radix-32 DFT of v, into v[8..24).  The last step of the
// inverse needs no more: outputs start lambda >= 2^13 samples into the window, end as far before
// its end, and slot j holds the window's points t + 512 j.
__device__ __forceinline__ void dft32_middle(float2 (&v)[32]) {
  float2 e[16], o[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    e[i] = v[2 * i];
    o[i] = v[2 * i + 1];
  }
  dft<16>(e);
  dft<16>(o);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const float2 E = e[out_slot<16>(k)];
    float2 O = o[out_slot<16>(k)];
    if (k == 8)
      O = mul_mi(O);
    else if (k != 0)
      O = cmul(O, make_float2(kCos32[k], -kSin32[k]));
    // O is rounded before the sum, as in the full transform (where it has two uses): with one use
    // the compiler would fold the sum into O's own multiply-adds and change its last bits.
    asm("" : "+v"(O.x), "+v"(O.y));
    if (k >= 8)
      v[k] = cadd(E, O);
    else
      v[k + 16] = csub(E, O);
  }
}

// Radix-16 DFT on v[off..off+16) in natural order.
template <int OFF>
__device__ __forceinline__ void dft16_at(float2 (&v)[32]) {
  float2 u[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) u[i] = v[OFF + i];
  dft<16>(u);
#pragma unroll
  for (int k = 0; k < 16; ++k) v[OFF + k] = u[out_slot<16>(k)];
}

// v[k] *= W_NC^(t k) = W_N^(2 t k), k < 32, from table twiddles and their products (2 t k < 2^15 for
// t < 512: no reduction of the angle index).  The fused products form all from five; kSeven takes
// k = 7 and 24 from the table too, so that no twiddle has more than three table factors.  u = N^-1 t
// is then no further from FP64 than with the LDS transform (relative L2 error at lambda = 8192
// 2.185e-7 against 2.190e-7; 2.210e-7 from five), at the same speed.
template <bool kSeven>
__device__ __forceinline__ void twiddle_a(float2 (&v)[32], int t, const float2* tw0,
                                          const float2* tw1) {
  auto table = [&](int k) { return twiddle(tw0, tw1, 2 * t * k); };
  const float2 w1 = table(1), w2 = table(2), w4 = table(4), w8 = table(8), w16 = table(16);
  float2 lo[8];
  lo[0] = make_float2(1.0f, 0.0f);
  lo[1] = w1;
  lo[2] = w2;
  lo[3] = cmul(w1, w2);
  lo[4] = w4;
  lo[5] = cmul(w1, w4);
  lo[6] = cmul(w2, w4);
  lo[7] = kSeven ? table(7) : cmul(lo[3], w4);
  const float2 hi[4] = {make_float2(1.0f, 0.0f), w8, w16, kSeven ? table(24) : cmul(w8, w16)};
#pragma unroll
  for (int h = 0; h < 4; ++h) {
#pragma unroll
    for (int l = 0; l < 8; ++l) {
      const int k = 8 * h + l;
      if (k == 0) continue;
      const float2 w = h == 0 ? lo[l] : (l == 0 ? hi[h] : cmul(hi[h], lo[l]));
      v[k] = cmul(v[k], w);
    }
  }
}

template <int C>
__device__ __forceinline__ float& part(float2& z) {
  if constexpr (C == 0) return z.x;
  else return z.y;
}

// A layout (thread t, slot k3) -> B layout (thread (k3, n1), slot n2), one component.
template <int C>
__device__ __forceinline__ void transpose_ab(float2 (&v)[32], float* lds, int tid, int k3b,
                                            int n1b) {
#pragma unroll
  for (int k = 0; k < 32; ++k) lds[k * kRowA + tid] = part<C>(v[k]);
  __syncthreads();
#pragma unroll
  for (int n2 = 0; n2 < 32; ++n2) part<C>(v[n2]) = lds[k3b * kRowA + n1b + 16 * n2];
  __syncthreads();
}

// B layout -> A layout.
template <int C>
__device__ __forceinline__ void transpose_ba(float2 (&v)[32], float* lds, int tid, int k3b,
                                            int n1b) {
#pragma unroll
  for (int n2 = 0; n2 < 32; ++n2) lds[k3b * kRowA + n1b + 16 * n2] = part<C>(v[n2]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 32; ++k) part<C>(v[k]) = lds[k * kRowA + tid];
  __syncthreads();
}

// Task slots of the B <-> C transposes: plane k3, row k2 of 17 floats, column n1.
struct Tasks {
  int a, b;  // k3 * kRowB + 17 * k2 of the two tasks
};

// B layout (thread (k3, n1), slot k2) -> C layout (tasks a, b; slots n1 and 16 + n1).
template <int C>
__device__ __forceinline__ void transpose_bc(float2 (&v)[32], float* lds, Tasks tk, int k3b,
                                            int n1b) {
#pragma unroll
  for (int k2 = 0; k2 < 32; ++k2) lds[k3b * kRowB + 17 * k2 + n1b] = part<C>(v[k2]);
  __syncthreads();
#pragma unroll
  for (int n1 = 0; n1 < 16; ++n1) {
    part<C>(v[n1]) = lds[tk.a + n1];
    part<C>(v[16 + n1]) = lds[tk.b + n1];
  }
  __syncthreads();
}

// C layout -> B layout.
template <int C>
__device__ __forceinline__ void transpose_cb(float2 (&v)[32], float* lds, Tasks tk, int k3b,
                                            int n1b) {
#pragma unroll
  for (int n1 = 0; n1 < 16; ++n1) {
    lds[tk.a + n1] = part<C>(v[n1]);
    lds[tk.b + n1] = part<C>(v[16 + n1]);
  }
  __syncthreads();
#pragma unroll
  for (int k2 = 0; k2 < 32; ++k2) part<C>(v[k2]) = lds[k3b * kRowB + 17 * k2 + n1b];
  __syncthreads();
}

// Real-spectrum step for one bin pair: X1 = Z[k], X2 = Z[NC - k] (indices mod NC), sa = S[k],
// sb = S[NC - k], W = W_N^k; the repacked, conjugated inverse input replaces both (see
// symbol_multiply in the LDS kernels for the derivation).
__device__ __forceinline__ void spectrum_pair(float2& X1, float2& X2, float sa, float sb,
                                              float2 W) {
  const float a = 2.0f * sa, b = 2.0f * sb;
  const float sig = a + b, del = a - b;
  const float ds = del * W.y;
  const float p = sig + ds, p2 = sig - ds, q = del * W.x;
  const float2 y1 = make_float2(p * X1.x + q * X2.y, -(p * X1.y + q * X2.x));
  const float2 y2 = make_float2(p2 * X2.x + q * X1.y, -(p2 * X2.y + q * X1.x));
  X1 = y1;
  X2 = y2;
}

// A bin that is its own partner (k = 0 or NC/2).
__device__ __forceinline__ void spectrum_self(float2& X, float sa, float sb, float2 W) {
  const float a = 2.0f * sa, b = 2.0f * sb;
  const float sig = a + b, del = a - b;
  const float p = sig + del * W.y, q = del * W.x;
  X = make_float2(p * X.x + q * X.y, -(p * X.y + q * X.x));
}

// Window samples [H kHalf, (H + 1) kHalf) (zero outside the block's [lo, hi)) through LDS into
// the A layout: z[t + 512 j] = (t[2m], t[2m+1]), m = t + 512 j, j in [16 H, 16 H + 16).
template <int H, bool kFromData>
__device__ __forceinline__ void gather_half(float2 (&v)[32], float* lds, int tid,
                                            const SegmentStreams& win,
                                            const double* __restrict__ x, int lo, int hi) {
  for (int n = tid * kLane; n < kHalf; n += kT * kLane) {
    float s[kLane];
    gather_lane<kLane, kFromData>(win, x, H * kHalf + n, lo, hi, s);
    *reinterpret_cast<float4*>(lds + n) = make_float4(s[0], s[1], s[2], s[3]);
    *reinterpret_cast<float4*>(lds + n + 4) = make_float4(s[4], s[5], s[6], s[7]);
  }
  __syncthreads();
#pragma unroll
  for (int jj = 0; jj < 16; ++jj)
    v[16 * H + jj] = *reinterpret_cast<const float2*>(lds + 2 * (tid + kT * jj));
  __syncthreads();
}

// What a segment's transform is fed with and drained into: the pointing products of a map or of
// data, or FP32 time-domain vectors in HBM (the stand-alone N^-1 t product).
enum RegIo { kIoApply = 0, kIoRhs = 1, kIoPlain = 2 };

// The plain form has neither gather nor scatter: slot j of thread t is the sample pair
// 2 (t + 512 j), so a wavefront's loads and stores are runs of 512 bytes straight between registers
// and memory, with no staging.  64 detectors x 2^20 samples, lambda = 8192: 540 us with the
// LDS-resident transform (one 1,024-thread workgroup per CU), 238 us here, bound by the
// transform's VALU issue.  (One kernel for all three, not a shared function: the rounding of the
// fused products then stays what it is.)
template <int IO>
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(4))) void k_apply_reg(
    const int32_t* __restrict__ lpix, const float* __restrict__ wq, const float* __restrict__ wu,
    const double* __restrict__ x0, const float* __restrict__ d0, double* __restrict__ y0,
    float* __restrict__ u0, int ncol, int64_t ldx, int64_t ldy, const Chunk* __restrict__ chunks,
    const float2* __restrict__ tab, const float2* __restrict__ tw0g,
    const float2* __restrict__ tw1g, int lam, const int32_t* __restrict__ done) {
  constexpr bool kFromData = IO == kIoRhs;
  __shared__ __align__(16) float lds[kLdsF + 64];
  __shared__ float2 tw0[128];
  __shared__ float2 tw1[kN / 128];
  // W_512^(n1 k2) = W_N^(64 n1 k2) at [n1 * kW2 + k2], n1 < 16, k2 < 32: rows of 33 so that
  // both the step-B reads (lanes across n1, slot k2 fixed) and the inverse reads (lanes across
  // k2, n1 fixed) hit distinct banks
  __shared__ float2 w512[16 * kW2];
  if (done != nullptr && *done) return;
  const int tid = threadIdx.x;
  if (tid < 128) tw0[tid] = tw0g[tid];
  if (tid < kN / 128) tw1[tid] = tw1g[tid];
  {
    const int e = (tid >> 5) * (tid & 31);  // < 512
    w512[(tid >> 5) * kW2 + (tid & 31)] = cmul(tw1g[e >> 1], tw0g[(e & 1) * 64]);
  }

  const int wg = xcd_ordered(blockIdx.x, gridDim.x);
  const int col = wg % ncol;
  const Chunk c = chunks[wg / ncol];
  const double* __restrict__ x = IO == kIoApply ? x0 + col * ldx : x0;
  const float* __restrict__ d = kFromData ? d0 + col * ldx : d0;
  double* __restrict__ y = y0 + col * ldy;
  const SegmentStreams win = segment_streams(lpix, wq, wu, d, c.out0 - lam);
  int lo, hi;
  window_range(c, lam, kN, lo, hi);

  // thread roles: A layout t = tid; B layout (k3, n1); C layout two mirror tasks
  const int k3b = tid >> 4, n1b = tid & 15;
  int a3, a2, b3, b2;
  reg_tasks(tid, a3, a2, b3, b2);
  const Tasks tk{a3 * kRowB + 17 * a2, b3 * kRowB + 17 * b2};

  float2 v[32];

  if constexpr (IO == kIoPlain) {
    if (lo == 0 && hi == kN) {
#pragma unroll
      for (int j = 0; j < 32; ++j)
        v[j] = load2u(win.d + static_cast<uint32_t>(2 * (tid + kT * j)));
    } else {
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        const int i = 2 * (tid + kT * j);
        v[j] = make_float2(i >= lo && i < hi ? win.d[i] : 0.0f,
                           i + 1 >= lo && i + 1 < hi ? win.d[i + 1] : 0.0f);
      }
    }
    __syncthreads();  // the twiddles are in LDS
  } else {
    // ---- gather the window in two halves of 16,384 samples through LDS ----------------------
    // The gather runs at raised wave priority: its waves issue their loads and finish their FP64
    // sums ahead of the other workgroup's transform, which has VALU work to fill the wait
    // (measured: -4 % per solve on the ground workload; the same for the scatter gave nothing).
    __builtin_amdgcn_s_setprio(3);
    // The right half of a segment's window is the left half of the next segment's (lambda = 2^13;
    // nearly so otherwise), and neighbouring segments run at the same time on one XCD: even
    // segments gather their right half first and odd ones their left half first, so that both
    // readers of a shared half fetch it together and the second finds it in L2.
    if (((wg / ncol) & 1) == 0) {
      gather_half<1, kFromData>(v, lds, tid, win, x, lo, hi);
      gather_half<0, kFromData>(v, lds, tid, win, x, lo, hi);
    } else {
      gather_half<0, kFromData>(v, lds, tid, win, x, lo, hi);
      gather_half<1, kFromData>(v, lds, tid, win, x, lo, hi);
    }
  }

  // ---- forward transform --------------------------------------------------------------------
  __builtin_amdgcn_s_setprio(0);
  dft32(v);
  twiddle_a<IO == kIoPlain>(v, tid, tw0, tw1);
  transpose_ab<0>(v, lds, tid, k3b, n1b);
  transpose_ab<1>(v, lds, tid, k3b, n1b);
  dft32(v);
#pragma unroll
  for (int k2 = 1; k2 < 32; ++k2) v[k2] = cmul(v[k2], w512[n1b * kW2 + k2]);
  transpose_bc<0>(v, lds, tk, k3b, n1b);
  transpose_bc<1>(v, lds, tk, k3b, n1b);
  // The band's symbol pairs (kTab float2, in this kernel's read order) go straight from global
  // memory into the idle staging LDS while the radix-16 steps run: each wave's direct load of
  // 16 B per lane lands at its wave base + 16 B x lane.
  {
    const float4* __restrict__ tg = reinterpret_cast<const float4*>(tab + c.band * kTab);
    const int wbase = tid & ~63;
#pragma unroll
    for (int r = 0; r < 8; ++r)
      load_to_lds16(tg + r * kT + tid, lds + 4 * (r * kT + wbase));
    if (tid < (2 * kTab) / 4 - 8 * kT)
      load_to_lds16(tg + 8 * kT + tid, lds + 4 * 8 * kT);
  }
  dft16_at<0>(v);
  dft16_at<16>(v);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // ---- real spectrum x band symbol, in registers --------------------------------------------
  // Slot k1 of task a is bin k = a3 + 32 a2 + 1024 k1 and its partner NC - k is slot 15 - k1 of
  // task b, for every thread but the first, whose tasks (0, 0) and (0, 16) are their own
  // partners.  All threads run the common pairing; thread 0 keeps its spectrum in a private LDS
  // slot, where lanes 0..16 of its wave redo its 17 bin pairs (two of them single bins) side by
  // side, and reloads it after the common pairing.  That keeps the common path free of a second
  // register pairing.  The slot is written and read by one wave only; wavefront-scope fences
  // order the hand-offs between its lanes.  (The side work comes before the common pairing: placed after it, the
  // compiler's schedule no longer fits the 128 registers of two workgroups per CU.)
  {
    const float2* stab = reinterpret_cast<const float2*>(lds);  // [k1][thread], then 8 extra
    float2* own = reinterpret_cast<float2*>(lds + kLdsF);  // thread 0 only; the transposes never
                                                            // reach past kLdsF
    if (tid == 0) {
#pragma unroll
      for (int i = 0; i < 32; ++i) own[i] = v[i];
    }
    wave_lds_sync();  // thread 0's slot is visible to lanes 0..16
    if (tid < 17) {
      // task (0, 0): bins 1024 k1, partners k1 <-> 16 - k1, bins 0 and NC/2 alone (lanes 0..8);
      // task (0, 16): bins 512 + 1024 k1, partners k1 <-> 15 - k1 (lanes 9..16)
      int i1, i2, k, e;
      if (tid == 0) {
        i1 = i2 = 0;
        k = 0;
        e = 0;
      } else if (tid == 1) {
        i1 = i2 = 8;
        k = kNC / 2;
        e = 8 * kT;
      } else if (tid <= 8) {
        i1 = tid - 1;
        i2 = 17 - tid;
        k = 1024 * i1;
        e = i1 * kT;
      } else {
        i1 = tid + 7;
        i2 = 40 - tid;
        k = 512 + 1024 * (tid - 9);
        e = 16 * kT + tid - 9;
      }
      float2 X1 = own[i1], X2 = own[i2];
      const float2 ss = stab[e];
      spectrum_pair(X1, X2, ss.x, ss.y, twiddle(tw0, tw1, k));
      own[i1] = X1;
      if (i2 != i1) own[i2] = X2;
    }
    const int ka = a3 + 32 * a2;
#pragma unroll
    for (int k1 = 0; k1 < 16; ++k1) {
      const float2 ss = stab[k1 * kT + tid];
      spectrum_pair(v[k1], v[31 - k1], ss.x, ss.y, twiddle(tw0, tw1, ka + 1024 * k1));
    }
    wave_lds_sync();  // lanes 0..16 have written the slot back before thread 0 reloads it
    if (tid == 0) {
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = own[i];
    }
  }
  __syncthreads();  // the staged symbol is read: the transposes may reuse the buffer

  // ---- inverse: the transposed steps --------------------------------------------------------
  dft16_at<0>(v);
  dft16_at<16>(v);
#pragma unroll
  for (int n1 = 1; n1 < 16; ++n1) {
    v[n1] = cmul(v[n1], w512[n1 * kW2 + a2]);
    v[16 + n1] = cmul(v[16 + n1], w512[n1 * kW2 + b2]);
  }
  transpose_cb<0>(v, lds, tk, k3b, n1b);
  transpose_cb<1>(v, lds, tk, k3b, n1b);
  dft32(v);
  transpose_ba<0>(v, lds, tid, k3b, n1b);
  transpose_ba<1>(v, lds, tid, k3b, n1b);
  twiddle_a<IO == kIoPlain>(v, tid, tw0, tw1);
  dft32_middle(v);

  if constexpr (IO == kIoPlain) {
    float* __restrict__ out = u0 + c.out0;
    if (lam == kHalf / 2 && c.out_len == kHalf) {  // every middle point is an output pair
#pragma unroll
      for (int j = 8; j < 24; ++j)
        store2u(out + static_cast<uint32_t>(2 * (tid + kT * (j - 8))), v[j].x, -v[j].y);
    } else {
#pragma unroll
      for (int j = 8; j < 24; ++j) {
        const int i = 2 * (tid + kT * j) - lam;
        if (static_cast<unsigned>(i) < static_cast<unsigned>(c.out_len)) out[i] = v[j].x;
        if (static_cast<unsigned>(i + 1) < static_cast<unsigned>(c.out_len)) out[i + 1] = -v[j].y;
      }
    }
    return;
  }

  // ---- outputs to LDS: sample 2m is Re, 2m+1 is -Im of point m = t + 512 j ------------------
  const int out_len = c.out_len;
  if (lam == kHalf / 2 && out_len == kHalf) {  // every middle point is an output pair
#pragma unroll
    for (int j = 8; j < 24; ++j)
      *reinterpret_cast<float2*>(lds + 2 * (tid + kT * (j - 8))) = make_float2(v[j].x, -v[j].y);
  } else {
#pragma unroll
    for (int j = 8; j < 24; ++j) {
      const int i = 2 * (tid + kT * j) - lam;
      if (static_cast<unsigned>(i) < static_cast<unsigned>(out_len)) lds[i] = v[j].x;
      if (static_cast<unsigned>(i + 1) < static_cast<unsigned>(out_len)) lds[i + 1] = -v[j].y;
    }
  }
  __syncthreads();

  // ---- scatter the segment's outputs ----------------------------------------------------------
  // Each wavefront reads its own 512 staged outputs per round; once read, that slice holds the
  // wavefront's list of completed runs, flushed one FP64 value per lane.
  const AtomicFlush flush{y};
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  static_assert(run_list_bytes<3, kListed>() <= 64 * kLane * sizeof(float),
                "run list must fit the wavefront's slice of the staged outputs");
  static_assert((kHalf + kT * kLane - 1) / (kT * kLane) * (kT * kLane) <= kLdsF,
                "every round's slices lie inside the staging buffer");
  for (int base = 0; base + 64 * kLane * wave < out_len; base += kT * kLane) {
    const int i0 = base + tid * kLane;
    float u[kLane];
    LanePointing<kLane, false> lane;
    lane.load(win, lam + i0, lam, lam + out_len);
#pragma unroll
    for (int j = 0; j < kLane; ++j) u[j] = lds[i0 + j];
    lane.bridge_flags(u);
    wave_point_runs<kLane, kListed>(lane.kk, lane.qq, lane.uu, u, flush,
                                    lds + base + 64 * kLane * wave);
  }
}

// Symbol pairs of every band in the register kernel's read order: entry [k1][thread] is
// (S[k], S[NC - k]) for bin k = a3 + 32 a2 + 1024 k1 of the thread's first task; then the 8
// bins 512 + 1024 j of the first thread's second task.
__global__ __launch_bounds__(kT) void k_reg_table(const float* __restrict__ spec,
                                                  float2* __restrict__ tab) {
  const int tid = threadIdx.x;
  const float* __restrict__ S = spec + static_cast<int64_t>(blockIdx.x) * (kNC + 1);
  float2* __restrict__ T = tab + static_cast<int64_t>(blockIdx.x) * kTab;
  int a3, a2, b3, b2;
  reg_tasks(tid, a3, a2, b3, b2);
  const int ka = a3 + 32 * a2;
  for (int k1 = 0; k1 < 16; ++k1) {
    const int k = ka + 1024 * k1;
    T[k1 * kT + tid] = make_float2(S[k], S[kNC - k]);
  }
  if (tid < 8) {
    const int k = 512 + 1024 * tid;
    T[16 * kT + tid] = make_float2(S[k], S[kNC - k]);
  }
}

}  // namespace

mm_status build_reg_table(Plan* P, hipStream_t s) {
  if (P->n_bands == 0) return MM_OK;
  MM_TRY(dalloc(P, &P->spec_reg, static_cast<size_t>(P->n_bands) * kTab));
  hipLaunchKernelGGL(k_reg_table, dim3(static_cast<unsigned>(P->n_bands)), dim3(kT), 0, s,
                     P->spec, P->spec_reg);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

bool apply_reg_supported(const Plan* P) {
  return P->fft_n == kN && P->fft_n - 2 * static_cast<int64_t>(P->lambda_max) <= kHalf;
}

mm_status launch_toeplitz_reg(Plan* P, const float* t, float* u, const int32_t* done,
                              hipStream_t s) {
  if (!apply_reg_supported(P) || P->spec_reg == nullptr)
    return fail(MM_ERR_UNSUPPORTED, "register FFT kernel: segment shape");
  hipLaunchKernelGGL((k_apply_reg<kIoPlain>), dim3(static_cast<unsigned>(P->n_chunks)), dim3(kT), 0,
                     s, P->lpix, P->wq, P->wu, static_cast<const double*>(nullptr), t,
                     static_cast<double*>(nullptr), u, 1, int64_t{0}, int64_t{0}, P->chunks,
                     P->spec_reg, P->tw0, P->tw1, P->lambda_max, done);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

mm_status launch_apply_reg(Plan* P, const double* x, const float* d, int64_t ldx, double* y,
                           int64_t ldy, int32_t ncol, const int32_t* done, hipStream_t s) {
  if (!apply_reg_supported(P) || P->spec_reg == nullptr)
    return fail(MM_ERR_UNSUPPORTED, "register FFT kernel: segment shape");
  const int64_t grid = static_cast<int64_t>(P->n_chunks) * ncol;
  if (grid > INT32_MAX) return fail(MM_ERR_UNSUPPORTED, "too many segment x column workgroups");
  const dim3 g(static_cast<unsigned>(grid));
  if (d != nullptr)
    hipLaunchKernelGGL((k_apply_reg<kIoRhs>), g, dim3(kT), 0, s, P->lpix, P->wq, P->wu, x, d, y,
                       static_cast<float*>(nullptr), ncol, ldx, ldy, P->chunks, P->spec_reg,
                       P->tw0, P->tw1, P->lambda_max, done);
  else
    hipLaunchKernelGGL((k_apply_reg<kIoApply>), g, dim3(kT), 0, s, P->lpix, P->wq, P->wu, x, d, y,
                       static_cast<float*>(nullptr), ncol, ldx, ldy, P->chunks, P->spec_reg,
                       P->tw0, P->tw1, P->lambda_max, done);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

}  // namespace mm
