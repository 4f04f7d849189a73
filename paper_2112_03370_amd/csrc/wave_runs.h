// Wavefront merge of equal-key runs for scatter-adds (P^T and the block-Jacobi build).
//
// Each lane holds SPL consecutive samples (lane l + 1 continues lane l) with their keys (pixel
// ids, -1 = skip) and NV FP64 values.  Time-ordered data visit a pixel for several consecutive
// samples, so keys come in runs.  The lane first sums the pieces of its own runs; runs strictly
// inside the lane are complete.  The run that ends the lane (its tail) may continue in the next
// lanes: an inclusive segmented scan over the lane tails (a new segment starts where the key
// changes or where a lane holds more than one run) gives every lane the sum of its chain so far.
// The lane that closes a chain completes it, unless the next lane's first run has the same key, in
// which case that lane adds the chain to its first run.  The result: one flush per run and
// wavefront instead of one atomic per sample.
#pragma once

#include <hip/hip_runtime.h>

namespace mm {

// Orders LDS accesses of one wavefront across its lanes: what lanes wrote before the call is
// visible to reads by other lanes of the same wavefront after it, and reads before it complete
// before later writes to the same slots.  A wavefront-scope release/acquire fence pair around a
// wave barrier; it must be reached by the whole wavefront (uniform control flow).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Lanes below this one that are set in a wavefront mask.
__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(
      static_cast<unsigned>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(m), 0u)));
}

// Exclusive prefix sum over the wavefront of a small per-lane count c < 2^BITS.
template <int BITS>
__device__ __forceinline__ int wave_exclusive_count(int c, int& total) {
  int before = 0;
  total = 0;
#pragma unroll
  for (int b = 0; b < BITS; ++b) {
    const unsigned long long m = __ballot((c >> b) & 1);
    before += lanes_below(m) << b;
    total += __popcll(m) << b;
  }
  return before;
}

// LDS of a wavefront's run list: CAP keys, then NV CAP values.
template <int NV, int CAP>
constexpr int run_list_bytes() {
  return CAP * static_cast<int>(sizeof(int) + NV * sizeof(double));
}

// The runs that the wavefront completes are first listed in LDS (CAP slots of one key and NV
// values per wavefront, at `list`, 8-byte aligned) and then flushed one value per lane (lanes
// NV r .. NV r + NV - 1 take the NV values of run r, through flush.one(key, component, value)):
// ceil(NV R / 64) instructions for R runs, and the values of one run go out in one instruction.
// Flushing each run where it ends would issue one round at every lane position where some lane
// closes a run inside it, which on scans with short runs (a circle clipping pixel corners) means
// several rounds of nearly idle atomic instructions per wavefront; and where the runs fall on
// different cache lines (pixel ids far apart along the scan), a run costs one memory-side atomic
// request instead of NV.  More than CAP runs are listed and flushed CAP at a time.
// The values come from a function v(sample, component), for callers short of registers.
template <int SPL, int NV, int CAP, class Value, class Flush>
__device__ __forceinline__ void wave_merge_runs_listed_of(const int (&key)[SPL], const Value& v,
                                                          const Flush& flush, void* list) {
  static_assert(SPL >= 2 && SPL <= 9, "inner-run counts must fit the 3-bit wavefront prefix");
  const int lane = static_cast<int>(threadIdx.x & 63u);
  int* skey = static_cast<int*>(list);
  double* sval = reinterpret_cast<double*>(skey + CAP);
  static_assert(CAP % 2 == 0, "8-byte aligned values");

  // ---- runs inside the lane: count, then list ---------------------------------------------
  // A run starting at a key change j > 0 lies inside the lane when another change follows.
  int n_in = 0, last_keyed = 0;
#pragma unroll
  for (int j = 1; j < SPL; ++j) {
    if (key[j] != key[j - 1]) {
      n_in += last_keyed;
      last_keyed = key[j] >= 0 ? 1 : 0;
    }
  }
  int r_in = 0, in_base = 0;
  if (__any(n_in > 0)) in_base = wave_exclusive_count<3>(n_in, r_in);  // wavefront-uniform
  wave_lds_sync();  // the previous call's listed runs have been read before slots are reused

  auto put = [&](int slot, int k, const double (&w)[NV]) {
    skey[slot] = k;
#pragma unroll
    for (int c = 0; c < NV; ++c) sval[slot * NV + c] = w[c];
  };
  // The lane's walk: lists its inner runs whose slots lie in [first, first + CAP) and leaves its
  // first run (when it holds more than one) in head and its last in acc.
  double acc[NV];
  double head[NV];
  int hk = -1, tk = -1;
  bool single = true;
  auto walk = [&](int first) {
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      acc[c] = v(0, c);
      head[c] = 0.0;
    }
    int cur = key[0];
    hk = -1;
    single = true;
    int slot = in_base - first;
#pragma unroll
    for (int j = 1; j < SPL; ++j) {
      if (key[j] != cur) {
        if (single) {
          hk = cur;
#pragma unroll
          for (int c = 0; c < NV; ++c) head[c] = acc[c];
          single = false;
        } else if (cur >= 0) {
          if (static_cast<unsigned>(slot) < static_cast<unsigned>(CAP)) put(slot, cur, acc);
          ++slot;
        }
        cur = key[j];
#pragma unroll
        for (int c = 0; c < NV; ++c) acc[c] = v(j, c);
      } else {
#pragma unroll
        for (int c = 0; c < NV; ++c) acc[c] += v(j, c);
      }
    }
    tk = cur;
  };
  walk(0);

  // ---- segmented inclusive scan of the lane tails ------------------------------------------
  const int prev_tk = __shfl_up(tk, 1);
  const bool start = (lane == 0) || !single || (prev_tk != tk);
  double S[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) S[c] = acc[c];
  int f = start ? 1 : 0;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    if (__ballot((!f) && lane >= d) == 0) break;  // wavefront-uniform exit
    double up[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) up[c] = __shfl_up(S[c], d);
    const int fup = __shfl_up(f, d);
    if (lane >= d && !f) {
#pragma unroll
      for (int c = 0; c < NV; ++c) S[c] += up[c];
      f = fup;
    }
  }

  // ---- the lane's head and closing tail ------------------------------------------------------
  double prevS[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) prevS[c] = __shfl_up(S[c], 1);
  const int next_start = __shfl_down(start ? 1 : 0, 1);
  const int next_single = __shfl_down(single ? 1 : 0, 1);
  const int next_hk = __shfl_down(hk, 1);

  const bool has_head = !single && hk >= 0;
  double H[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c)
    H[c] = has_head && lane > 0 && prev_tk == hk ? head[c] + prevS[c] : head[c];
  const bool ends = (lane == 63) || next_start;
  const bool has_tail =
      ends && tk >= 0 && !((lane < 63) && !next_single && next_hk == tk);
  const int head_key = hk, tail_key = tk;
  // slots in lane order, a lane's first run before its last: neighbouring pixels stay together
  const unsigned long long m_head = __ballot(has_head), m_tail = __ballot(has_tail);
  const int s_head = r_in + lanes_below(m_head) + lanes_below(m_tail);
  const int s_tail = s_head + (has_head ? 1 : 0);
  const int total = r_in + __popcll(m_head) + __popcll(m_tail);

  // ---- list heads and tails, flush one value of one listed run per lane --------------------
  for (int first = 0;;) {
    if (has_head && static_cast<unsigned>(s_head - first) < static_cast<unsigned>(CAP))
      put(s_head - first, head_key, H);
    if (has_tail && static_cast<unsigned>(s_tail - first) < static_cast<unsigned>(CAP))
      put(s_tail - first, tail_key, S);
    wave_lds_sync();  // runs listed by other lanes of the wavefront are visible
    const int n = min(total - first, CAP) * NV;
    for (int e = lane; e - lane < n; e += 64) {
      if (e < n) {
        const int r = e / NV;
        flush.one(skey[r], e - r * NV, sval[e]);
      }
    }
    first += CAP;
    if (first >= total) break;  // wavefront-uniform
    wave_lds_sync();  // the listed runs have been read before their slots are reused
    if (first < r_in) walk(first);
  }
}

template <int SPL, int NV, int CAP, class Flush>
__device__ __forceinline__ void wave_merge_runs_listed(const int (&key)[SPL],
                                                       const double (&v)[SPL][NV],
                                                       const Flush& flush, void* list) {
  wave_merge_runs_listed_of<SPL, NV, CAP>(
      key, [&](int j, int c) { return v[j][c]; }, flush, list);
}

}  // namespace mm
