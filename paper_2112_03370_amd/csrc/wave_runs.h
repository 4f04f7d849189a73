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
template <int NV, int CAP>
struct RunList {
  static_assert(CAP % 2 == 0, "8-byte aligned values");
  int* key;
  double* val;
  __device__ __forceinline__ explicit RunList(void* list)
      : key(static_cast<int*>(list)), val(reinterpret_cast<double*>(key + CAP)) {}
  // Lists a run whose number lies in [0, CAP) of the current pass.
  __device__ __forceinline__ void put(int slot, int k, const double (&w)[NV]) const {
    if (static_cast<unsigned>(slot) < static_cast<unsigned>(CAP)) {
      key[slot] = k;
#pragma unroll
      for (int c = 0; c < NV; ++c) val[slot * NV + c] = w[c];
    }
  }
};

// A lane's runs: the first (when it holds more than one; hk = -1 otherwise or when it is skipped)
// and the last; those between are listed.
template <int NV>
struct LaneRuns {
  double head[NV], acc[NV];
  int hk, tk;
  bool single;
};

// Runs that begin and end inside a lane, whose first sample is not the lane's first.
template <int SPL>
__device__ __forceinline__ int inner_runs(const int (&key)[SPL]) {
  static_assert(SPL >= 2 && SPL <= 9, "inner-run counts must fit the 3-bit wavefront prefix");
  // A run starting at a key change j > 0 lies inside the lane when another change follows.
  int n_in = 0, last_keyed = 0;
#pragma unroll
  for (int j = 1; j < SPL; ++j) {
    if (key[j] != key[j - 1]) {
      n_in += last_keyed;
      last_keyed = key[j] >= 0 ? 1 : 0;
    }
  }
  return n_in;
}

// The lane's walk over values v(sample, component): its first and last runs, and its inner runs,
// of which the wavefront's numbers start at `slot`, into the list.
template <int SPL, int NV, int CAP, class Value>
__device__ __forceinline__ void walk_runs(const int (&key)[SPL], const Value& v, int slot,
                                          const RunList<NV, CAP>& list, LaneRuns<NV>& r) {
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    r.acc[c] = v(0, c);
    r.head[c] = 0.0;
  }
  int cur = key[0];
  r.hk = -1;
  r.single = true;
#pragma unroll
  for (int j = 1; j < SPL; ++j) {
    if (key[j] != cur) {
      if (r.single) {
        r.hk = cur;
#pragma unroll
        for (int c = 0; c < NV; ++c) r.head[c] = r.acc[c];
        r.single = false;
      } else if (cur >= 0) {
        list.put(slot, cur, r.acc);
        ++slot;
      }
      cur = key[j];
#pragma unroll
      for (int c = 0; c < NV; ++c) r.acc[c] = v(j, c);
    } else {
#pragma unroll
      for (int c = 0; c < NV; ++c) r.acc[c] += v(j, c);
    }
  }
  r.tk = cur;
}

// Joins the lanes' runs and flushes every run of the wavefront; the first r_in of its list are
// inner runs, listed already as far as they fit, and again(first) lists those from `first` on.
template <int NV, int CAP, class Again, class Flush>
__device__ __forceinline__ void join_and_flush(const LaneRuns<NV>& r, int r_in,
                                               const RunList<NV, CAP>& list, const Again& again,
                                               const Flush& flush) {
  const int lane = static_cast<int>(threadIdx.x & 63u);
  const int hk = r.hk, tk = r.tk;
  const bool single = r.single;

  // ---- segmented inclusive scan of the lane tails ------------------------------------------
  const int prev_tk = __shfl_up(tk, 1);
  const bool start = (lane == 0) || !single || (prev_tk != tk);
  double S[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) S[c] = r.acc[c];
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
    H[c] = has_head && lane > 0 && prev_tk == hk ? r.head[c] + prevS[c] : r.head[c];
  const bool ends = (lane == 63) || next_start;
  const bool has_tail =
      ends && tk >= 0 && !((lane < 63) && !next_single && next_hk == tk);
  // slots in lane order, a lane's first run before its last: neighbouring pixels stay together
  const unsigned long long m_head = __ballot(has_head), m_tail = __ballot(has_tail);
  const int s_head = r_in + lanes_below(m_head) + lanes_below(m_tail);
  const int s_tail = s_head + (has_head ? 1 : 0);
  const int total = r_in + __popcll(m_head) + __popcll(m_tail);

  // ---- list heads and tails, flush one value of one listed run per lane --------------------
  for (int first = 0;;) {
    if (has_head) list.put(s_head - first, hk, H);
    if (has_tail) list.put(s_tail - first, tk, S);
    wave_lds_sync();  // runs listed by other lanes of the wavefront are visible
    const int n = min(total - first, CAP) * NV;
    for (int e = lane; e - lane < n; e += 64) {
      if (e < n) {
        const int k = e / NV;
        flush.one(list.key[k], e - k * NV, list.val[e]);
      }
    }
    first += CAP;
    if (first >= total) break;  // wavefront-uniform
    wave_lds_sync();  // the listed runs have been read before their slots are reused
    if (first < r_in) again(first);
  }
}

// Runs of NV values given by v(sample, component).
template <int SPL, int NV, int CAP, class Value, class Flush>
__device__ __forceinline__ void wave_merge_runs_of(const int (&key)[SPL], const Value& v,
                                                   const Flush& flush, void* at) {
  const RunList<NV, CAP> list(at);
  const int n_in = inner_runs(key);
  int r_in = 0, in_base = 0;
  if (__any(n_in > 0)) in_base = wave_exclusive_count<3>(n_in, r_in);  // wavefront-uniform
  wave_lds_sync();  // the previous call's listed runs have been read before slots are reused
  LaneRuns<NV> r;
  walk_runs(key, v, in_base, list, r);
  join_and_flush(
      r, r_in, list,
      [&](int first) {
        LaneRuns<NV> unused;
        walk_runs(key, v, in_base - first, list, unused);
      },
      flush);
}

template <int SPL, int NV, int CAP, class Flush>
__device__ __forceinline__ void wave_merge_runs_listed(const int (&key)[SPL],
                                                       const double (&v)[SPL][NV],
                                                       const Flush& flush, void* at) {
  wave_merge_runs_of<SPL, NV, CAP>(
      key, [&](int j, int c) { return v[j][c]; }, flush, at);
}

// The pointing sums P^T: runs of u, q u and w u.
//
// Where no lane of the wavefront sees more than two pixels (pixels visited for at least SPL
// samples), a lane's two sums are formed without branches: each sample counts in one of them and
// as a zero in the other.  The walk executes both sides of its branch at nearly every sample, since
// some lane of 64 changes pixel there, with the products formed beforehand: about twice the
// instructions, in kernels that are bound by the issue of vector instructions.  kOnePixel: one sum
// per lane where no lane sees a second pixel.
template <int SPL, int CAP, bool kOnePixel = false, class T, class Flush>
__device__ __forceinline__ void wave_point_runs(const int (&key)[SPL], const float (&q)[SPL],
                                                const float (&w)[SPL], const T (&u)[SPL],
                                                const Flush& flush, void* at) {
  const RunList<3, CAP> list(at);
  int changes = 0;
#pragma unroll
  for (int j = 1; j < SPL; ++j) changes += key[j] != key[j - 1] ? 1 : 0;
  wave_lds_sync();  // the previous call's listed runs have been read before slots are reused
  const auto value = [&](int j, int c) {
    const double t = static_cast<double>(u[j]);
    return c == 0 ? t : static_cast<double>(c == 1 ? q[j] : w[j]) * t;
  };
  int r_in = 0, in_base = 0;
  LaneRuns<3> r;
  if (kOnePixel && !__any(changes > 0)) {  // wavefront-uniform
    r.single = true;
    r.hk = -1;
    r.tk = key[0];
#pragma unroll
    for (int c = 0; c < 3; ++c) r.head[c] = r.acc[c] = 0.0;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const double t = static_cast<double>(u[j]);
      r.acc[0] += t;
      r.acc[1] = fma(static_cast<double>(q[j]), t, r.acc[1]);
      r.acc[2] = fma(static_cast<double>(w[j]), t, r.acc[2]);
    }
  } else if (!__any(changes > 1)) {  // wavefront-uniform
    r.single = changes == 0;
    r.hk = r.single ? -1 : key[0];
    r.tk = key[SPL - 1];
#pragma unroll
    for (int c = 0; c < 3; ++c) r.head[c] = r.acc[c] = 0.0;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const double qd = static_cast<double>(q[j]), wd = static_cast<double>(w[j]);
      const bool last = j == SPL - 1 || key[j] == r.tk;
      const double tail = static_cast<double>(last ? u[j] : T(0));
      r.acc[0] += tail;
      r.acc[1] = fma(qd, tail, r.acc[1]);
      r.acc[2] = fma(wd, tail, r.acc[2]);
      if (j < SPL - 1) {
        const double head = static_cast<double>(last ? T(0) : u[j]);
        r.head[0] += head;
        r.head[1] = fma(qd, head, r.head[1]);
        r.head[2] = fma(wd, head, r.head[2]);
      }
    }
  } else {
    const int n_in = inner_runs(key);
    in_base = wave_exclusive_count<3>(n_in, r_in);
    walk_runs(key, value, in_base, list, r);
  }
  join_and_flush(
      r, r_in, list,
      [&](int first) {
        LaneRuns<3> unused;
        walk_runs(key, value, in_base - first, list, unused);
      },
      flush);
}

}  // namespace mm
