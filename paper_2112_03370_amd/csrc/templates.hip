// Template map-making: the system product P^T F_T P with
//
//     F_T = W^-1 (I - T (T^T W^-1 T)^+ T^T W^-1)                                (Eq. defFT)
//
// for diagonal weights W^-1 and Legendre baselines (Appendix A, Eq. polytemplate): on every
// baseline interval of L samples the templates are sqrt((2k+1)/L) P_k(x_j), k < n_poly, at the
// midpoints x_j = (2j+1)/L - 1.  The orthogonalisation kernel T^T W^-1 T is block-diagonal, one
// n_poly x n_poly block per baseline, built and pseudo-inverted on the device in FP64 at plan
// time (eigen-directions below 1e-12 of the largest dropped, the paper's SVD threshold).  A baseline lies inside one stationary interval (or outside all of them), so
// its weight w is the c_0 of that interval's band; gap samples (flagged or excised) weigh 0.
//
// The product runs as one kernel, one workgroup per baseline, every step in FP64:
//   1. t_s = (P x)_s (or the data sample), weighted v_s = w t_s; projections a_k = sum_s T_sk v_s
//      reduced over the workgroup (the time-domain projection of the templates algebra)
//   2. c = K_b^+ a
//   3. u_s = w (t_s - sum_k T_sk c_k)  (template projection subtracted); y += P^T u through the
//      wavefront run merge
// A lane holds 8 consecutive samples and a wavefront steps through the baseline kHeld steps at a
// time: the pointing of the first kHeld steps is loaded in one go and stays in registers between 1
// and 3, t waits in LDS, so baselines of up to 1,024 (64 threads), 4,096 (256) or 8,192 (512)
// samples are read once; longer ones re-gather the rest.  Samples outside every baseline get
// u = w t through the diagonal product.
//
// What bounds it: the chain table entry -> pointing -> pixels -> sums -> coefficients -> pointing
// sums, whose waits 16 wavefronts per CU have to cover, then the FP64 instructions.  128 detectors
// x 2^20 samples, baselines of 8,192, 3 templates: 896 us with 4 samples per lane, all of them in
// registers and the scaled Legendre recurrence twice per sample; 501 us here (3.2 TB/s of pointing).
// The registers spilled at 512 threads cost traffic: 5.7 GB per 2^28 samples, 4.9 GB with 4 samples
// per lane and no spills; eight wavefronts per CU and no spills 4.1 GB, but 1,197 us against 996.
// Re-reading the pointing in 3 instead of holding it: 762 us (the reads come late, not from HBM).
// t in registers instead of LDS: 889 us (spills).  One workgroup size for all baselines
// left the short ones with idle wavefronts: 64 x 2^19 samples, baselines of 500 (3 templates)
// 1,147 us with 512 threads, 167 us with 64; of 600 (1 template) 834 and 159 us; of 3,000
// 323 us and, with 256, 153 us.
#include <algorithm>
#include <cmath>

#include "fft_lds.h"
#include "mm_internal.h"
#include "segment_io.h"
#include "wave_runs.h"

namespace mm {

namespace {

constexpr int kTT = 512;     // threads per workgroup of the kernel blocks' build
constexpr int kLane = 8;     // consecutive samples per lane and step
constexpr int kHeld = 2;     // steps whose pointing stays in registers
constexpr int kListed = 64;  // runs listed per wavefront

// Scaled Legendre values T_k = scale_k P_k(x), k < NP, by the three-term recurrence
// k P_k = (2k - 1) x P_(k-1) - (k - 1) P_(k-2), with 1/k as a constant.
template <int NP>
__device__ __forceinline__ void legendre(double x, const double* scale, double (&T)[NP]) {
  double p0 = 1.0, p1 = x;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    double pk;
    if (k == 0) {
      pk = p0;
    } else if (k == 1) {
      pk = p1;
    } else {
      constexpr double kInv[kMaxTemplates] = {0.0, 1.0, 1.0 / 2, 1.0 / 3, 1.0 / 4, 1.0 / 5,
                                               1.0 / 6, 1.0 / 7};
      pk = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) * kInv[k];
      p0 = p1;
      p1 = pk;
    }
    T[k] = scale[k] * pk;
  }
}

// Legendre values P_k(x), k < NP, without the scales, which the projections and the coefficients
// take once per baseline: P_k = ((2k - 1) / k) x P_(k-1) - ((k - 1) / k) P_(k-2).
template <int NP>
__device__ __forceinline__ void legendre_plain(double x, double (&T)[NP]) {
  T[0] = 1.0;
  if constexpr (NP > 1) T[1] = x;
#pragma unroll
  for (int k = 2; k < NP; ++k)
    T[k] = fma((2.0 * k - 1.0) / k * x, T[k - 1], -((k - 1.0) / k) * T[k - 2]);
}

// t of a lane between the two halves of the kernel, in the lane's own LDS slots.
__device__ __forceinline__ void park(double2* slot, const double (&t)[kLane], int n) {
#pragma unroll
  for (int j = 0; j < kLane; j += 2) slot[j / 2 * n] = make_double2(t[j], t[j + 1]);
}
__device__ __forceinline__ void fetch(const double2* slot, double (&t)[kLane], int n) {
#pragma unroll
  for (int j = 0; j < kLane; j += 2) {
    const double2 v = slot[j / 2 * n];
    t[j] = v.x;
    t[j + 1] = v.y;
  }
}

// a_k += sum_j P_k(x_j) t_j, x_j = x0 + j dx (t is zero at flagged samples).
template <int NP>
__device__ __forceinline__ void project(const double (&t)[kLane], double x0, double dx,
                                        double (&a)[NP]) {
#pragma unroll
  for (int j = 0; j < kLane; ++j) {
    double P[NP];
    legendre_plain<NP>(fma(dx, static_cast<double>(j), x0), P);
    a[0] += t[j];
#pragma unroll
    for (int k = 1; k < NP; ++k) a[k] = fma(P[k], t[j], a[k]);
  }
}

// t_j = w t_j - sum_k P_k(x_j) c_k.
template <int NP>
__device__ __forceinline__ void subtract(double (&t)[kLane], double x0, double dx, double w,
                                         const double (&c)[NP]) {
#pragma unroll
  for (int j = 0; j < kLane; ++j) {
    double P[NP];
    legendre_plain<NP>(fma(dx, static_cast<double>(j), x0), P);
    double r = fma(w, t[j], -c[0]);
#pragma unroll
    for (int k = 1; k < NP; ++k) r = fma(-P[k], c[k], r);
    t[j] = r;
  }
}

// Wavefronts per SIMD: 512 threads need four for two workgroups per CU and spill some of their
// registers for it (25 at three templates, 52 to 65 at four to seven, 115 at eight).  With room for
// two and no spills, 128 x 2^19 samples and baselines of 8,192 take 316 us instead of 263 (3
// templates), 337 for 289 (4), 361 for 301 (5), 380 for 335 (6), 405 for 379 (7), 424 for 407 (8; of
// 16,384 samples 391 for 404), but with one template, where nothing spills, 182 for 203.
// Smaller workgroups fill a CU with three and no spills, which is faster where four would spill
// much: 64 x 2^19 samples, 3 templates, baselines of 3,000 180 -> 153 us, but 1 template, baselines
// of 600 154 -> 173 us.
template <int NP, int T>
constexpr int template_waves() {
  return T == 512 || NP < 3 ? 4 : 3;
}

template <bool kData, int NP, int T>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(template_waves<NP, T>())))
void k_template_apply(
    const int32_t* __restrict__ lpix, const float* __restrict__ wq, const float* __restrict__ wu,
    const double* __restrict__ x, const float* __restrict__ d, const TBase* __restrict__ bases,
    const double* __restrict__ kinv, double* __restrict__ y, const int32_t* __restrict__ done) {
  if (done != nullptr && *done) return;
  constexpr int kStep = T * kLane;  // samples per step
  __shared__ double red[NP][T / 64];
  __shared__ double coef[NP];
  __shared__ double lists[T / 64][run_list_bytes<3, kListed>() / sizeof(double)];
  __shared__ double kmat[NP * NP];
  __shared__ double2 parked[kHeld][kLane / 2][T];
  const int base = fft::xcd_ordered(blockIdx.x, gridDim.x);
  const TBase B = bases[base];
  const int tid = threadIdx.x;
  const SegmentStreams str = segment_streams(lpix, wq, wu, d, B.start);
  const double invL = 1.0 / static_cast<double>(B.len), dx = 2.0 * invL;
  const double w = static_cast<double>(B.w);
  const int first = kLane * tid;              // the lane's first sample in step 0
  const int wave = first - kLane * (tid & 63);  // its wavefront's: steps past the end are skipped
  auto midpoint = [&](int j) { return fma(2.0, static_cast<double>(j), 1.0) * invL - 1.0; };

  if (tid < NP * NP) kmat[tid] = kinv[static_cast<int64_t>(base) * NP * NP + tid];

  // ---- 1. gather and project ------------------------------------------------------------------
  double a[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) a[k] = 0.0;
  LanePointing<kLane, false> held[kHeld];
#pragma unroll
  for (int s = 0; s < kHeld; ++s)
    if (wave + s * kStep < B.len) held[s].load(str, first + s * kStep, 0, B.len);
#pragma unroll
  for (int s = 0; s < kHeld; ++s) {
    if (wave + s * kStep < B.len) {
      const int i = first + s * kStep;
      double t[kLane];
      if constexpr (kData)
        gather_lane<kLane, true>(str, x, i, 0, B.len, t);
      else
        held[s].resolve(x, t);
      park(&parked[s][0][tid], t, T);
      project<NP>(t, midpoint(i), dx, a);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll 1
  for (int off = kHeld * kStep; wave + off < B.len; off += kStep) {
    double t[kLane];
    gather_lane<kLane, kData>(str, x, first + off, 0, B.len, t);
    project<NP>(t, midpoint(first + off), dx, a);
  }
  // opaque from here on: the gather's FP64 copies of the weights (64 registers) are not kept for
  // the scatter
#pragma unroll
  for (int s = 0; s < kHeld; ++s)
#pragma unroll
    for (int j = 0; j < kLane; ++j) {
      asm("" : "+v"(held[s].qq[j]));
      asm("" : "+v"(held[s].uu[j]));
    }
  // workgroup sums in a fixed order
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    double v = a[k];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((tid & 63) == 0) red[k][tid >> 6] = v;
  }
  __syncthreads();

  // ---- 2. c = K^+ a, with the scales of both sides and the weight -------------------------------
  if (tid < NP) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      double ak = 0.0;
#pragma unroll
      for (int wv = 0; wv < T / 64; ++wv) ak += red[k][wv];
      acc = fma(kmat[tid * NP + k], ak * (w * sqrt((2.0 * k + 1.0) * invL)), acc);
    }
    coef[tid] = acc * (w * sqrt((2.0 * tid + 1.0) * invL));
  }
  __syncthreads();
  double c[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) c[k] = coef[k];

  // ---- 3. subtract the fit, weight, point -----------------------------------------------------
  void* list = lists[tid >> 6];
  auto drain = [&](LanePointing<kLane, false>& lane, double (&t)[kLane], int i) {
    subtract<NP>(t, midpoint(i), dx, w, c);
    lane.bridge_flags(t);
    wave_merge_runs_of<kLane, 3, kListed>(
        lane.kk,
        [&](int j, int q) {
          return q == 0 ? t[j] : static_cast<double>(q == 1 ? lane.qq[j] : lane.uu[j]) * t[j];
        },
        AtomicFlush{y}, list);
  };
#pragma unroll
  for (int s = 0; s < kHeld; ++s) {
    if (wave + s * kStep < B.len) {
      double t[kLane];
      fetch(&parked[s][0][tid], t, T);
      drain(held[s], t, first + s * kStep);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll 1
  for (int off = kHeld * kStep; wave + off < B.len; off += kStep) {
    LanePointing<kLane, false> lane;
    double t[kLane];
    lane.load(str, first + off, 0, B.len);
    gather_lane<kLane, kData>(str, x, first + off, 0, B.len, t);
    drain(lane, t, first + off);
  }
}

// Pseudo-inverse of a symmetric positive semi-definite NP x NP block by cyclic Jacobi rotations
// (eigenvalues below rtol times the largest dropped), in registers: the same algorithm as the
// host routine used for the block recurrences.
template <int NP>
__device__ __forceinline__ void small_sym_pinv(double (&a)[NP][NP], double (&v)[NP][NP],
                                               double rtol, double (&out)[NP][NP]) {
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int j = 0; j < NP; ++j) v[i][j] = i == j ? 1.0 : 0.0;
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0, tot = 0.0;
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        tot += a[i][j] * a[i][j];
        if (i != j) off += a[i][j] * a[i][j];
      }
    if (off <= 1e-30 * tot || tot == 0.0) break;
#pragma unroll
    for (int p = 0; p < NP - 1; ++p)
#pragma unroll
      for (int q = p + 1; q < NP; ++q) {
        const double apq = a[p][q];
        if (apq == 0.0) continue;
        const double theta = (a[q][q] - a[p][p]) / (2.0 * apq);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
        const double c = 1.0 / sqrt(t * t + 1.0), sn = t * c;
#pragma unroll
        for (int k = 0; k < NP; ++k) {  // columns p, q
          const double akp = a[k][p], akq = a[k][q];
          a[k][p] = c * akp - sn * akq;
          a[k][q] = sn * akp + c * akq;
        }
#pragma unroll
        for (int k = 0; k < NP; ++k) {  // rows p, q
          const double apk = a[p][k], aqk = a[q][k];
          a[p][k] = c * apk - sn * aqk;
          a[q][k] = sn * apk + c * aqk;
        }
#pragma unroll
        for (int k = 0; k < NP; ++k) {  // eigenvectors
          const double vkp = v[k][p], vkq = v[k][q];
          v[k][p] = c * vkp - sn * vkq;
          v[k][q] = sn * vkp + c * vkq;
        }
      }
  }
  double wmax = 0.0;
#pragma unroll
  for (int i = 0; i < NP; ++i) wmax = fmax(wmax, a[i][i]);
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int j = 0; j < NP; ++j) out[i][j] = 0.0;
#pragma unroll
  for (int e = 0; e < NP; ++e) {
    const double w = a[e][e];
    if (!(w > rtol * wmax) || w <= 0.0) continue;
    const double inv = 1.0 / w;
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
      for (int j = 0; j < NP; ++j) out[i][j] += v[i][e] * inv * v[j][e];
  }
}

// Kernel block of one baseline, K = sum_j w T(j) T(j)^T over its unflagged samples (Legendre
// templates T), and its pseudo-inverse (zero for a block of zeros), one workgroup per baseline:
// every pair (i <= k) is accumulated in the same pass over the samples, reduced across the
// workgroup, and the first thread inverts the block.
template <int NP>
__global__ __launch_bounds__(kTT) void k_template_kernel(const int32_t* __restrict__ lpix,
                                                         const TBase* __restrict__ bases,
                                                         double* __restrict__ Kinv) {
  constexpr int NPAIR = NP * (NP + 1) / 2;
  __shared__ double red[NPAIR][kTT / 64];
  __shared__ double scale[kMaxTemplates];
  const TBase B = bases[blockIdx.x];
  const int tid = threadIdx.x;
  const double invL = 1.0 / static_cast<double>(B.len);
  if (tid < kMaxTemplates) scale[tid] = sqrt((2.0 * tid + 1.0) * invL);
  __syncthreads();
  const double w = static_cast<double>(B.w);
  double acc[NPAIR];
#pragma unroll
  for (int q = 0; q < NPAIR; ++q) acc[q] = 0.0;
  for (int j = tid; j < B.len; j += kTT) {
    if (lpix[B.start + j] < 0) continue;
    double T[NP];
    legendre<NP>(fma(2.0, static_cast<double>(j), 1.0) * invL - 1.0, scale, T);
    int q = 0;
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
      for (int k = i; k < NP; ++k, ++q) acc[q] = fma(w * T[i], T[k], acc[q]);
  }
#pragma unroll
  for (int q = 0; q < NPAIR; ++q) {
    double v = acc[q];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((tid & 63) == 0) red[q][tid >> 6] = v;
  }
  __syncthreads();
  if (tid != 0) return;
  // the rotations work in registers for up to five templates, in LDS beyond (register room)
  constexpr bool kRegs = NP <= 5;
  __shared__ double lds_g[kRegs ? 1 : NP][NP], lds_v[kRegs ? 1 : NP][NP],
      lds_o[kRegs ? 1 : NP][NP];
  double reg_g[kRegs ? NP : 1][NP], reg_v[kRegs ? NP : 1][NP], reg_o[kRegs ? NP : 1][NP];
  auto& G = *reinterpret_cast<double(*)[NP][NP]>(kRegs ? &reg_g[0][0] : &lds_g[0][0]);
  auto& V = *reinterpret_cast<double(*)[NP][NP]>(kRegs ? &reg_v[0][0] : &lds_v[0][0]);
  auto& Gi = *reinterpret_cast<double(*)[NP][NP]>(kRegs ? &reg_o[0][0] : &lds_o[0][0]);
  bool zero = true;
  int q = 0;
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int k = i; k < NP; ++k, ++q) {
      double sum = 0.0;
#pragma unroll
      for (int wv = 0; wv < kTT / 64; ++wv) sum += red[q][wv];
      G[i][k] = G[k][i] = sum;
      zero = zero && sum == 0.0;
    }
  double* out = Kinv + static_cast<int64_t>(blockIdx.x) * NP * NP;
  if (zero) {
#pragma unroll
    for (int i = 0; i < NP * NP; ++i) out[i] = 0.0;
    return;
  }
  small_sym_pinv<NP>(G, V, 1e-12, Gi);
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int k = 0; k < NP; ++k) out[i * NP + k] = Gi[i][k];
}

}  // namespace

mm_status build_templates(Plan* P, const mm_geometry* g, const std::vector<Tile>& tiles,
                          hipStream_t s) {
  const int n_poly = g->n_poly;
  if (n_poly <= 0) return MM_OK;
  if (n_poly > kMaxTemplates)
    return fail(MM_ERR_UNSUPPORTED, "n_poly > " + std::to_string(kMaxTemplates));
  if (P->lambda_max != 0)
    return fail(MM_ERR_UNSUPPORTED, "template map-making takes diagonal weights (band_ncoef = 1)");
  if (g->n_baselines < 0) return fail(MM_ERR_INVALID, "n_baselines < 0");
  if (g->n_baselines > 0 && (!g->base_start || !g->base_len))
    return fail(MM_ERR_INVALID, "baseline table pointers are NULL");
  if (g->n_baselines > INT32_MAX) return fail(MM_ERR_INVALID, "too many baselines");
  const int64_t nb = g->n_baselines;
  std::vector<int64_t> order(static_cast<size_t>(nb));
  for (int64_t i = 0; i < nb; ++i) order[static_cast<size_t>(i)] = i;
  std::sort(order.begin(), order.end(),
            [&](int64_t a, int64_t b) { return g->base_start[a] < g->base_start[b]; });
  // weights: the c_0 of the tile holding the baseline; the baseline must stay inside one block
  // (or outside all blocks) and, with detector offsets, inside one detector
  std::vector<int64_t> bstart, bend;  // blocks, sorted by start
  {
    std::vector<int> bo(static_cast<size_t>(g->n_blocks));
    for (int i = 0; i < g->n_blocks; ++i) bo[static_cast<size_t>(i)] = i;
    std::sort(bo.begin(), bo.end(), [&](int a, int b) { return g->blk_start[a] < g->blk_start[b]; });
    for (int i : bo) {
      bstart.push_back(g->blk_start[i]);
      bend.push_back(g->blk_start[i] + g->blk_len[i]);
    }
  }
  std::vector<TBase> bases;
  bases.reserve(static_cast<size_t>(nb));
  P->base_max = 0;
  int64_t prev_end = 0;
  for (int64_t i : order) {
    const int64_t s0 = g->base_start[i], L = g->base_len[i];
    if (s0 < 0 || L < 1 || s0 + L > g->n_samples)
      return fail(MM_ERR_INVALID, "baseline " + std::to_string(i) + " outside [0, n_samples)");
    if (L > INT32_MAX) return fail(MM_ERR_INVALID, "baseline longer than 2^31 samples");
    if (s0 < prev_end) return fail(MM_ERR_INVALID, "baselines overlap");
    prev_end = s0 + L;
    // block containing s0 (last block starting at or before s0)
    const auto it = std::upper_bound(bstart.begin(), bstart.end(), s0);
    const int64_t bi = (it - bstart.begin()) - 1;
    const bool inside = bi >= 0 && s0 < bend[static_cast<size_t>(bi)];
    if (inside && s0 + L > bend[static_cast<size_t>(bi)])
      return fail(MM_ERR_INVALID, "baseline " + std::to_string(i) + " crosses a stationary interval");
    if (!inside) {
      const int64_t next = bi + 1;
      if (next < static_cast<int64_t>(bstart.size()) && bstart[static_cast<size_t>(next)] < s0 + L)
        return fail(MM_ERR_INVALID, "baseline " + std::to_string(i) + " crosses a stationary interval");
    }
    if (g->det_offset != nullptr && g->n_dets > 0) {
      const int64_t* de = g->det_offset;
      const auto dt = std::upper_bound(de, de + g->n_dets + 1, s0);
      if (dt == de + g->n_dets + 1 || s0 + L > *dt)
        return fail(MM_ERR_INVALID, "baseline " + std::to_string(i) + " crosses a detector");
    }
    // weight of the covering tile (tiles are sorted and cover [0, n_samples))
    const auto ti = std::upper_bound(tiles.begin(), tiles.end(), s0,
                                     [](int64_t v, const Tile& t) { return v < t.start; });
    const float w = (ti == tiles.begin()) ? 1.0f : (ti - 1)->c0;
    bases.push_back(TBase{s0, static_cast<int32_t>(L), w});
    P->base_max = std::max(P->base_max, static_cast<int32_t>(L));
  }
  // samples outside every baseline: the tiles with the baselines cut out
  std::vector<Tile> free_tiles;
  {
    size_t bix = 0;
    for (const Tile& t : tiles) {
      int64_t a = t.start;
      const int64_t e = t.start + t.len;
      while (a < e) {
        while (bix < bases.size() && bases[bix].start + bases[bix].len <= a) ++bix;
        int64_t stop = e;
        if (bix < bases.size() && bases[bix].start <= a) {
          a = std::min<int64_t>(e, bases[bix].start + bases[bix].len);  // skip the covered part
          continue;
        }
        if (bix < bases.size()) stop = std::min<int64_t>(e, bases[bix].start);
        free_tiles.push_back(Tile{a, static_cast<int32_t>(stop - a), t.c0});
        a = stop;
      }
    }
  }
  P->n_poly = n_poly;
  P->n_baselines = nb;
  MM_TRY(dalloc(P, &P->tbases, bases.size()));
  MM_TRY(dalloc(P, &P->tkinv, bases.size() * static_cast<size_t>(n_poly * n_poly)));
  MM_TRY(dalloc(P, &P->free_tiles, free_tiles.size()));
  P->n_free_tiles = static_cast<int32_t>(free_tiles.size());
  if (!bases.empty())
    MM_HIP_TRY(hipMemcpyAsync(P->tbases, bases.data(), bases.size() * sizeof(TBase), hipMemcpyHostToDevice, s));
  if (!free_tiles.empty())
    MM_HIP_TRY(hipMemcpyAsync(P->free_tiles, free_tiles.data(), free_tiles.size() * sizeof(Tile),
                              hipMemcpyHostToDevice, s));
  if (bases.empty()) {
    MM_HIP_TRY(hipStreamSynchronize(s));
    return MM_OK;
  }
  // kernel blocks and their pseudo-inverses on the device, one workgroup per baseline
  const dim3 grid(static_cast<unsigned>(bases.size()));
  switch (n_poly) {
    case 1: hipLaunchKernelGGL(k_template_kernel<1>, grid, dim3(kTT), 0, s, P->lpix, P->tbases, P->tkinv); break;
    case 2: hipLaunchKernelGGL(k_template_kernel<2>, grid, dim3(kTT), 0, s, P->lpix, P->tbases, P->tkinv); break;
    case 3: hipLaunchKernelGGL(k_template_kernel<3>, grid, dim3(kTT), 0, s, P->lpix, P->tbases, P->tkinv); break;
    case 4: hipLaunchKernelGGL(k_template_kernel<4>, grid, dim3(kTT), 0, s, P->lpix, P->tbases, P->tkinv); break;
    case 5: hipLaunchKernelGGL(k_template_kernel<5>, grid, dim3(kTT), 0, s, P->lpix, P->tbases, P->tkinv); break;
    case 6: hipLaunchKernelGGL(k_template_kernel<6>, grid, dim3(kTT), 0, s, P->lpix, P->tbases, P->tkinv); break;
    case 7: hipLaunchKernelGGL(k_template_kernel<7>, grid, dim3(kTT), 0, s, P->lpix, P->tbases, P->tkinv); break;
    default: hipLaunchKernelGGL(k_template_kernel<8>, grid, dim3(kTT), 0, s, P->lpix, P->tbases, P->tkinv); break;
  }
  MM_HIP_TRY(hipGetLastError());
  MM_HIP_TRY(hipStreamSynchronize(s));  // the host tables above are released on return
  return MM_OK;
}

namespace {

template <int NP, int T>
mm_status launch_npt(Plan* P, const double* x, const float* d, double* y, const int32_t* done,
                     hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(P->n_baselines));
  if (x != nullptr)
    hipLaunchKernelGGL((k_template_apply<false, NP, T>), grid, dim3(T), 0, s, P->lpix, P->wq,
                       P->wu, x, d, P->tbases, P->tkinv, y, done);
  else
    hipLaunchKernelGGL((k_template_apply<true, NP, T>), grid, dim3(T), 0, s, P->lpix, P->wq,
                       P->wu, x, d, P->tbases, P->tkinv, y, done);
  MM_HIP_TRY(hipGetLastError());
  return MM_OK;
}

// The fewest threads whose held steps take the longest baseline: every sample is then read once,
// and no wavefront idles through baselines much shorter than its workgroup's step.
template <int NP>
mm_status launch_np(Plan* P, const double* x, const float* d, double* y, const int32_t* done,
                    hipStream_t s) {
  if (P->base_max <= 64 * kLane * kHeld) return launch_npt<NP, 64>(P, x, d, y, done, s);
  if (P->base_max <= 256 * kLane * kHeld) return launch_npt<NP, 256>(P, x, d, y, done, s);
  return launch_npt<NP, 512>(P, x, d, y, done, s);
}

}  // namespace

mm_status launch_template_apply(Plan* P, const double* x, const float* d, double* y,
                                const int32_t* done, hipStream_t s) {
  TimedLaunch tl(P, K_TOEPLITZ, s);
  if (P->n_baselines > 0) {
    switch (P->n_poly) {
      case 1: MM_TRY(launch_np<1>(P, x, d, y, done, s)); break;
      case 2: MM_TRY(launch_np<2>(P, x, d, y, done, s)); break;
      case 3: MM_TRY(launch_np<3>(P, x, d, y, done, s)); break;
      case 4: MM_TRY(launch_np<4>(P, x, d, y, done, s)); break;
      case 5: MM_TRY(launch_np<5>(P, x, d, y, done, s)); break;
      case 6: MM_TRY(launch_np<6>(P, x, d, y, done, s)); break;
      case 7: MM_TRY(launch_np<7>(P, x, d, y, done, s)); break;
      default: MM_TRY(launch_np<8>(P, x, d, y, done, s)); break;
    }
  }
  if (P->n_free_tiles > 0)
    MM_TRY(launch_diag_tiles(P, P->free_tiles, P->n_free_tiles, x, d, y, done, s));
  return MM_OK;
}

}  // namespace mm
