// Per-segment time-domain I/O shared by the fused system-product kernels: the gather of
// t = P x (or of the data d) for a lane of consecutive samples, and the FP64 atomic flush of
// merged scatter runs into y = P^T u.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mm {

struct AtomicFlush {
  double* y;
  __device__ void one(int key, int c, double v) const {
    unsafeAtomicAdd(y + 3 * static_cast<int64_t>(key) + c, v);
  }
};

// 16-byte global accesses at 4-byte alignment: time streams are read from wherever a stationary
// interval or a window starts.  gfx950 takes dword-aligned dwordx4 accesses, so lanes need no
// aligned start; an unaligned wavefront only touches one more cache line.  (Scalar loads in their
// place, one wait per sample, made one product of 61 detectors x 200,003 samples, lambda = 2047,
// 2 % flags, take 254 us; with these loads 209 us, and with the flags and short runs handled as
// below and in wave_runs.h 94 us.)
typedef int int4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef float float4_u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void load4u(const int32_t* p, int* v) {
  const int4_u t = *reinterpret_cast<const int4_u*>(p);
  v[0] = t.x;
  v[1] = t.y;
  v[2] = t.z;
  v[3] = t.w;
}
__device__ __forceinline__ void load4u(const float* p, float* v) {
  const float4_u t = *reinterpret_cast<const float4_u*>(p);
  v[0] = t.x;
  v[1] = t.y;
  v[2] = t.z;
  v[3] = t.w;
}
typedef float float2_u __attribute__((ext_vector_type(2), aligned(4)));
__device__ __forceinline__ float2 load2u(const float* p) {
  const float2_u t = *reinterpret_cast<const float2_u*>(p);
  return make_float2(t.x, t.y);
}
__device__ __forceinline__ void store2u(float* p, float a, float b) {
  *reinterpret_cast<float2_u*>(p) = float2_u{a, b};
}
__device__ __forceinline__ void store4u(float* p, float a, float b, float c, float d) {
  *reinterpret_cast<float4_u*>(p) = float4_u{a, b, c, d};
}

// The pointing streams of one segment (and the data when gathering d), from the segment's first
// window sample on: that sample may lie before the streams' own first sample (a window that
// starts before the first interval), where nothing is read.  Uniform base plus 32-bit sample
// offset: one address register per lane instead of a 64-bit add per access.
struct SegmentStreams {
  const int32_t* lpix;
  const float* wq;
  const float* wu;
  const float* d;
};

__device__ __forceinline__ SegmentStreams segment_streams(const int32_t* lpix, const float* wq,
                                                          const float* wu, const float* d,
                                                          int64_t first) {
  return SegmentStreams{lpix + first, wq + first, wu + first, d + first};
}

// Pointing of one lane: samples [i, i + S) of a segment (the data instead of the weights when
// gathering d).  Samples outside [lo, hi) get key -1 and are not read.
template <int S, bool kFromData>
struct LanePointing {
  int kk[S];
  float qq[S], uu[S];

  // All S samples inside the streams.
  __device__ __forceinline__ void load(const SegmentStreams& p, uint32_t i) {
#pragma unroll
    for (uint32_t c = 0; c < S; c += 4) {
      load4u(p.lpix + (i + c), kk + c);
      load4u((kFromData ? p.d : p.wq) + (i + c), qq + c);
      if constexpr (!kFromData) load4u(p.wu + (i + c), uu + c);
    }
  }

  __device__ __forceinline__ void load(const SegmentStreams& p, int i, int lo, int hi) {
    if (i >= lo && i + S <= hi) {
      load(p, static_cast<uint32_t>(i));
      return;
    }
#pragma unroll
    for (int j = 0; j < S; ++j) {
      kk[j] = -1;
      qq[j] = uu[j] = 0.0f;
    }
#pragma unroll
    for (int j = 0; j < S; ++j) {  // the lanes that straddle an edge
      if (i + j >= lo && i + j < hi) {
        kk[j] = p.lpix[i + j];
        qq[j] = (kFromData ? p.d : p.wq)[i + j];
        if constexpr (!kFromData) uu[j] = p.wu[i + j];
      }
    }
  }

  __device__ __forceinline__ int least_key() const {
    int least = kk[0];
#pragma unroll
    for (int j = 1; j < S; ++j) least = min(least, kk[j]);
    return least;
  }

  // Flagged samples continue the run of pixels that surrounds them, with zero weight and zero
  // value: for the scatter, where every break in a run costs a listed run and its atomics.  Lanes
  // without any pixel keep key -1.  (Weights and values at flagged samples may hold anything.)
  template <class T>
  __device__ __forceinline__ void bridge_flags(T (&v)[S]) {
    if (!__any(least_key() < 0)) return;
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const bool skip = kk[j] < 0;
      v[j] = skip ? T(0) : v[j];
      qq[j] = skip ? 0.0f : qq[j];
      uu[j] = skip ? 0.0f : uu[j];
      if (j > 0) kk[j] = skip ? kk[j - 1] : kk[j];
    }
#pragma unroll
    for (int j = S - 2; j >= 0; --j) kk[j] = kk[j] < 0 ? kk[j + 1] : kk[j];
  }

  // Scan runs keep a pixel for several consecutive samples, so a lane usually sees one or two
  // pixels: the lane's first and last pixels are loaded together, with the first other pixel
  // between them where some lane of the wavefront has one (short runs), all behind a single wait;
  // further pixels, one at a time, only when they occur.  fetch() issues those loads and
  // finish() forms the samples, so that a caller can have several lanes' loads in flight.
  struct Pixels {
    int ka, kb, kc;  // first, last and first other pixel; -1: none
    bool flagged, more;  // wavefront-uniform: some lane has flagged samples, an other pixel
    double a[3], b[3], c[3];
  };

  __device__ __forceinline__ static void load_pixel(const double* __restrict__ x, int k,
                                                    double (&m)[3]) {
    const double* p = x + 3 * static_cast<int64_t>(k);
    m[0] = p[0];
    m[1] = p[1];
    m[2] = p[2];
  }

  __device__ __forceinline__ void fetch(const double* __restrict__ x, Pixels& f) const {
    if constexpr (!kFromData) {
      // The tests for flagged samples sit behind a wavefront-uniform branch (per sample, the
      // compiler turns them into a branch around that sample's sums).
      f.ka = kk[0];
      f.kb = kk[S - 1];
      bool other = false;
      f.flagged = __any(least_key() < 0);
      if (f.flagged) {
        f.ka = f.kb = -1;  // the first and last pixels observed
#pragma unroll
        for (int j = 0; j < S; ++j) {
          f.kb = kk[j] >= 0 ? kk[j] : f.kb;
          f.ka = kk[S - 1 - j] >= 0 ? kk[S - 1 - j] : f.ka;
        }
#pragma unroll
        for (int j = 1; j < S - 1; ++j) other |= kk[j] >= 0 && kk[j] != f.ka && kk[j] != f.kb;
      } else {
#pragma unroll
        for (int j = 1; j < S - 1; ++j) other |= kk[j] != f.ka && kk[j] != f.kb;
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) f.a[q] = f.b[q] = f.c[q] = 0.0;
      if (f.ka >= 0) load_pixel(x, f.ka, f.a);
      if (f.kb >= 0 && f.kb != f.ka) load_pixel(x, f.kb, f.b);
      f.more = __any(other);
      f.kc = -1;
      if (f.more) {
#pragma unroll
        for (int j = S - 2; j > 0; --j)
          f.kc = kk[j] >= 0 && kk[j] != f.ka && kk[j] != f.kb ? kk[j] : f.kc;
        if (f.kc >= 0) load_pixel(x, f.kc, f.c);
      }
    }
  }

  // kOnePixel: wavefronts whose lanes all see one pixel form one sum per sample instead of two.
  template <bool kOnePixel = false, class T>
  __device__ __forceinline__ void finish(const double* __restrict__ x, Pixels& f,
                                         T (&v)[S]) const {
    if constexpr (kFromData) {
#pragma unroll
      for (int j = 0; j < S; ++j) v[j] = kk[j] < 0 ? T(0) : static_cast<T>(qq[j]);
    } else {
      if (kOnePixel && !__any(f.kb != f.ka)) {
#pragma unroll
        for (int j = 0; j < S; ++j)
          v[j] = static_cast<T>(f.a[0] + static_cast<double>(qq[j]) * f.a[1] +
                                static_cast<double>(uu[j]) * f.a[2]);
      } else {
#pragma unroll
        for (int j = 0; j < S; ++j) {
          // both candidate pixels' sums, then one select (cheaper than selecting three FP64
          // pixel values)
          const double q = static_cast<double>(qq[j]), u = static_cast<double>(uu[j]);
          const double ta = f.a[0] + q * f.a[1] + u * f.a[2];
          const double tb = f.b[0] + q * f.b[1] + u * f.b[2];
          v[j] = static_cast<T>(kk[j] == f.ka ? ta : tb);
        }
      }
      if (f.flagged) {
#pragma unroll
        for (int j = 0; j < S; ++j) v[j] = kk[j] < 0 ? T(0) : v[j];
      }
      if (f.more) {
        int done = 0;  // samples before this one are resolved as far as kc goes
        while (true) {
#pragma unroll
          for (int j = 1; j < S - 1; ++j) {
            const double t = f.c[0] + static_cast<double>(qq[j]) * f.c[1] +
                             static_cast<double>(uu[j]) * f.c[2];
            if (f.kc >= 0 && kk[j] == f.kc) v[j] = static_cast<T>(t);
          }
          // the next pixel after kc's first sample that none of the loaded ones was
          int next = -1, at = S;
#pragma unroll
          for (int j = S - 2; j > 0; --j)
            if (j > done && kk[j] >= 0 && kk[j] != f.ka && kk[j] != f.kb && kk[j] != f.kc) {
              next = kk[j];
              at = j;
            }
          if (!__any(next >= 0)) break;
          done = at;
          f.kc = next;
          if (f.kc >= 0) load_pixel(x, f.kc, f.c);
        }
      }
    }
  }

  template <class T>
  __device__ __forceinline__ void resolve(const double* __restrict__ x, T (&v)[S]) const {
    Pixels f;
    fetch(x, f);
    finish(x, f, v);
  }
};

// t of one lane of window samples [i, i + S): P x, or the data, zero outside [lo, hi).  Lanes that
// lie outside altogether (the window's overhang at a block's ends: whole wavefronts) skip the sums.
template <int S, bool kFromData, class T>
__device__ __forceinline__ void gather_lane(const SegmentStreams& win,
                                            const double* __restrict__ x, int i, int lo, int hi,
                                            T (&v)[S]) {
  if (i + S <= lo || i >= hi) {
#pragma unroll
    for (int j = 0; j < S; ++j) v[j] = T(0);
    return;
  }
  LanePointing<S, kFromData> lane;
  lane.load(win, i, lo, hi);
  lane.resolve(x, v);
}

}  // namespace mm
