// kernels.hip -- the smaller HIP kernels for gfx950, and their launchers.
//
//  k_aux      rebuild the per-block offsets for streams written elsewhere
//  k_range    min / max / non-finite count (tau_0 = range, Sec. 5.1)
//  k_sum_sq   sums for the accuracy gain (Sec. 5.1.1)
//  k_cast_*   the float32-cast compressor (Sec. 3)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "block_device.hpp"

namespace pmc {

// ---------------------------------------------------------------------------
// Per-block bit offsets of streams written elsewhere: each chunk's 16 blocks are
// parsed one after the other by one lane, a serial chain, so latency and the
// chains in flight are what counts.  A wave stages the words of L chunks in LDS
// and L of its lanes parse them; all components go in one launch.  Few chunks
// per wave keep the lanes' loops short (the wave takes as many windows as its
// slowest lane) and the waves many: L = 4 while that leaves at most 4 waves
// per SIMD (64^3 float64, 4 components: 68 us, 90 with L = 16), 16 beyond
// (256^3 float32, 8 components: 218 us, 304 with L = 8; the upload of such a
// store takes 3 ms).  One launch per component with 64 chunks per wave read
// from global memory had 51 waves in flight for 3 M values and took 145 us per
// component; all 6 take 79 us now.  L = 64: unstaged, for an index whose chunks
// are longer than any encoder writes (which a loader may still be given).
template <class T, int kCodec, class R>
__device__ __forceinline__ void aux_chunk(const AuxArgs& a, int comp, uint64_t chunk, R& r, uint32_t from, bool ok,
                                          const uint8_t* sq) {
  const uint64_t b0 = chunk * kChunkBlocks, b1 = min<uint64_t>(a.g.nblocks, b0 + kChunkBlocks);
  const int minexp = a.minexp[comp];
  uint32_t* const aux = a.aux[comp];
  uint32_t any = 0;
#pragma unroll 1
  for (uint64_t blk = b0; blk < b1; ++blk) {
    aux[blk] = ok ? (uint32_t)r.consumed(from) : 0u;
    uint32_t flags = 0;
    if (ok) ok = (kCodec == 0 ? block_skip<T>(r, minexp, sq, flags) : pq_block_skip<T>(r)) && !r.bad();
    any |= flags;
  }
  if (!ok) atomicOr(a.status, 1u);
  // flags, read first: most waves of such a component would raise them
  if (any & ~(uint32_t)*(volatile unsigned long long*)(a.full + comp)) atomicOr(a.full + comp, (unsigned long long)any);
}
template <class T, int kCodec, int L>
__global__ __launch_bounds__(64) void k_aux(AuxArgs a) {
  extern __shared__ uint32_t s_words[];  // a.cap words in rows of 64, and three more
  __shared__ uint8_t s_squeeze[256];
  const int comp = (int)blockIdx.y;
  const uint32_t lane = threadIdx.x;
  const uint32_t* index = reinterpret_cast<const uint32_t*>(a.s[comp] + kHeaderBytes);
  const uint32_t* payload = index + a.g.nchunks;
  const uint64_t words = a.words[comp];
  const uint64_t c0 = (uint64_t)blockIdx.x * L, c1 = min<uint64_t>(c0 + L, a.g.nchunks);
  uint64_t w0 = 0, w1 = words;
  bool ok = true;
  if constexpr (L < 64) {
    w0 = index[c0];
    w1 = c1 < a.g.nchunks ? (uint64_t)index[c1] : words;
    ok = w0 <= w1 && w1 <= words && w1 - w0 <= a.cap;  // (so checked on the host)
    const uint32_t span = ok ? (uint32_t)(w1 - w0) : 0u;
    for (uint32_t k = 0; k < span; k += 64) {
      const uint32_t j = k + lane < span ? k + lane : span - 1;
      __builtin_amdgcn_global_load_lds((gmem_void_t*)(payload + w0 + j), (lds_void_t*)(s_words + k), 4, 0, 0);
    }
  }
  squeeze_table(s_squeeze);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  const uint64_t chunk = c0 + lane;
  if (lane >= (uint32_t)L || chunk >= c1) return;
  const uint64_t start = index[chunk];
  const uint64_t stop = chunk + 1 < a.g.nchunks ? (uint64_t)index[chunk + 1] : words;
  // a chunk holds at least one block, hence at least one bit
  ok = ok && w0 <= start && start < stop && stop <= w1 && stop <= 0xFFFFFFFFull;
  if constexpr (L < 64) {
    LBits r;
    const uint32_t from = ok ? (uint32_t)(start - w0) : 0u;
    r.init(s_words, from, ok ? (uint32_t)(stop - w0) : 0u, a.cap);
    aux_chunk<T, kCodec>(a, comp, chunk, r, from, ok, s_squeeze);
  } else {
    GBits r;
    r.init(payload, (uint32_t)start, (uint32_t)(ok ? stop : start));
    aux_chunk<T, kCodec>(a, comp, chunk, r, (uint32_t)start, ok, s_squeeze);
  }
}

// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long ordered(double v) {
  unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// min / max over the finite samples and the count of the others.  Keys are
// the samples' bits mapped to unsigned integers of the same order (sign and
// zero sign included), so the reduction is exact integer min / max in the
// field's own width; a workgroup's result is widened to the double key of the
// same value, for the host to combine.  16-byte loads when aligned.
template <class T> struct RangeKey;
template <> struct RangeKey<float> {
  typedef uint32_t K;
  static __device__ __forceinline__ K key(float v) {
    const uint32_t b = __float_as_uint(v);
    return (b >> 31) ? ~b : (b | 0x80000000u);
  }
  static __device__ __forceinline__ bool finite(float v) { return (__float_as_uint(v) & 0x7F800000u) != 0x7F800000u; }
  static __device__ __forceinline__ double value(K k) {
    return (double)__uint_as_float((k >> 31) ? (k & 0x7FFFFFFFu) : ~k);
  }
};
template <> struct RangeKey<double> {
  typedef unsigned long long K;
  static __device__ __forceinline__ K key(double v) { return ordered(v); }
  static __device__ __forceinline__ bool finite(double v) {
    return ((unsigned long long)__double_as_longlong(v) & 0x7FF0000000000000ull) != 0x7FF0000000000000ull;
  }
  static __device__ __forceinline__ double value(K k) {
    return __longlong_as_double((long long)((k >> 63) ? (k & 0x7FFFFFFFFFFFFFFFull) : ~k));
  }
};

// One workgroup's share as a partial (kRangeWords words: least key, largest
// key, non-finite count, the keys as doubles' keys), which the host combines
// from pinned memory the device writes.  A pass over memory; what else it cost
// was the reduction across the device: the first workgroups all raised the
// same two words with atomics, which one cache line serialises (about 10 ns
// each).  One plain store per workgroup, no more workgroups than CUs and 16
// waves in each to keep the loads in flight take the whole call down by 15 us
// for 64^3 float64, 50 us for 9.2 M float32 values and 10 us for 512^3 (118 to
// 108 us, 5.0 TB/s, the rate a large copy reaches; two workgroups per CU 111,
// 512^3 float64 196 and 203).
constexpr uint32_t kRangeThreads = 1024;
template <class T>
__global__ __launch_bounds__(kRangeThreads) void k_range(const T* __restrict__ x, uint64_t n,
                                                         unsigned long long* __restrict__ out) {
  typedef RangeKey<T> RK;
  typedef typename RK::K K;
  K lo = ~(K)0, hi = 0;
  uint32_t bad = 0;
  auto take = [&](T v) {
    const K k = RK::key(v);
    const bool fin = RK::finite(v);
    lo = fin && k < lo ? k : lo;
    hi = fin && k > hi ? k : hi;
    bad += fin ? 0u : 1u;
  };
  const uint64_t tid = (uint64_t)blockIdx.x * kRangeThreads + threadIdx.x, stride = (uint64_t)gridDim.x * kRangeThreads;
  constexpr uint64_t V = 16 / sizeof(T);  // samples per 16-byte load
  uint64_t done = 0;
  if (((uintptr_t)x & 15) == 0) {
    typedef typename std::conditional<sizeof(T) == 4, float4, double2>::type V16;
    const V16* xv = reinterpret_cast<const V16*>(x);
    auto take16 = [&](const V16& v) {
      if constexpr (sizeof(T) == 4) {
        take(v.x);
        take(v.y);
        take(v.z);
        take(v.w);
      } else {
        take(v.x);
        take(v.y);
      }
    };
    const uint64_t nv = n / V;
    uint64_t i = tid;
    for (; i + 3 * stride < nv; i += 4 * stride) {  // four 16-byte loads in flight
      const V16 a0 = xv[i], a1 = xv[i + stride], a2 = xv[i + 2 * stride], a3 = xv[i + 3 * stride];
      take16(a0);
      take16(a1);
      take16(a2);
      take16(a3);
    }
    for (; i < nv; i += stride) take16(xv[i]);
    done = nv * V;
  }
  for (uint64_t i = done + tid; i < n; i += stride) take(x[i]);
  auto reduce = [&]() {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      const K a = __shfl_xor(lo, d, 64), b = __shfl_xor(hi, d, 64);
      lo = a < lo ? a : lo;
      hi = b > hi ? b : hi;
      bad += __shfl_xor(bad, d, 64);
    }
  };
  reduce();
  constexpr uint32_t W = kRangeThreads / 64;
  __shared__ K s_lo[W], s_hi[W];
  __shared__ uint32_t s_bad[W];
  const uint32_t wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    s_lo[wv] = lo;
    s_hi[wv] = hi;
    s_bad[wv] = bad;
  }
  __syncthreads();
  if (wv == 0) {
    lo = lane < W ? s_lo[lane] : ~(K)0;
    hi = lane < W ? s_hi[lane] : 0;
    bad = lane < W ? s_bad[lane] : 0u;
    reduce();
    if (lane == 0) {
      unsigned long long* o = out + (uint64_t)kRangeWords * blockIdx.x;
      const bool any = lo != ~(K)0;  // this workgroup saw a finite sample
      o[0] = any ? ordered(RK::value(lo)) : ~0ull;
      o[1] = any ? ordered(RK::value(hi)) : 0ull;
      o[2] = bad;
    }
  }
}

// p[0, n) = v
__global__ void k_fill64(unsigned long long* p, uint64_t n, unsigned long long v) {
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// sums of d = a - b - shift and of d^2 in float64 over a field (b NULL: 0),
// for the accuracy gain of Sec. 5.1.1 (standard deviation of the data,
// root-mean-square error of a reconstruction).  Deterministic: each
// workgroup reduces a fixed grid-stride share in a fixed order into its own
// partial pair, and one workgroup then adds the partials in index order.
constexpr int kSumGroups = 1024;  // workgroups of the first stage (the partials)

__device__ __forceinline__ void block_sum2(double& s, double& q, double* sh) {
  const uint32_t t = threadIdx.x;
  sh[t] = s;
  sh[256 + t] = q;
  __syncthreads();
  for (uint32_t h = 128; h > 0; h >>= 1) {
    if (t < h) {
      sh[t] = sh[t] + sh[t + h];
      sh[256 + t] = sh[256 + t] + sh[256 + t + h];
    }
    __syncthreads();
  }
  s = sh[0];
  q = sh[256];
}

template <class T>
__global__ __launch_bounds__(256) void k_sum_sq(const T* __restrict__ a, const T* __restrict__ b, double shift,
                                                uint64_t n, double* partials) {
  __shared__ double sh[512];
  double s = 0.0, q = 0.0;
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    const double d = ((double)a[i] - (b ? (double)b[i] : 0.0)) - shift;
    s = s + d;
    q = q + d * d;
  }
  block_sum2(s, q, sh);
  if (threadIdx.x == 0) {
    partials[2 * blockIdx.x] = s;
    partials[2 * blockIdx.x + 1] = q;
  }
}

__global__ __launch_bounds__(256) void k_sum_sq_final(const double* partials, uint32_t groups, double* out) {
  __shared__ double sh[512];
  double s = 0.0, q = 0.0;
  for (uint32_t g = threadIdx.x; g < groups; g += 256) {
    s = s + partials[2 * g];
    q = q + partials[2 * g + 1];
  }
  block_sum2(s, q, sh);
  if (threadIdx.x == 0) {
    out[0] = s;
    out[1] = q;
  }
}

template <class T>
hipError_t launch_sum_sq(const T* a, const T* b, double shift, uint64_t n, double* ws, double* out, hipStream_t s) {
  uint64_t groups = (n + 255) / 256;
  if (groups > kSumGroups) groups = kSumGroups;
  if (groups == 0) groups = 1;
  hipLaunchKernelGGL(k_sum_sq<T>, dim3((uint32_t)groups), dim3(256), 0, s, a, b, shift, n, ws);
  hipLaunchKernelGGL(k_sum_sq_final, dim3(1), dim3(256), 0, s, ws, (uint32_t)groups, out);
  return hipGetLastError();
}
uint64_t sum_sq_ws_bytes() { return (uint64_t)kSumGroups * 16 + 256; }

// ---------------------------------------------------------------------------
// Sec. 3's scalar special case as a second compressor behind the same
// driver: C(e) = fl32(e) (round to nearest even float32), D(y) = y in the
// field's type.  One thread per value runs all n components of Alg. 1 in
// registers: e = x - x~ in the field's type, y = fl32(e), x~ = x~ + y; the
// measured errors max |x - x~_i| (float64) are raised per wave with atomics on
// their bit patterns (non-negative doubles order like their bits).
// (NC: a compile-time bound on n, so that the per-component maxima have fixed
// registers; launched with the smallest of 4, 8, 32 that holds n)
template <class T, int NC>
__global__ __launch_bounds__(256) void k_cast_encode(const T* __restrict__ x, uint64_t N, int n,
                                                     float* __restrict__ comps, unsigned long long* linf_bits) {
  double mx[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) mx[i] = 0.0;
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  for (uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x; j < N; j += stride) {
    const T xj = x[j];
    T xt = (T)0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      if (i < n) {
        const float y = (float)(xj - xt);  // the residual in the field's type, then rounded once
        comps[(uint64_t)i * N + j] = y;
        xt = xt + (T)y;
        const double err = __builtin_fabs((double)xj - (double)xt);
        mx[i] = err > mx[i] ? err : mx[i];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    if (i < n) {
      const double wm = wave_max(mx[i]);
      const unsigned long long wb = (unsigned long long)__double_as_longlong(wm);
      if ((threadIdx.x & 63) == 0 && wb > *(volatile unsigned long long*)&linf_bits[i]) atomicMax(&linf_bits[i], wb);
    }
  }
}
// x~_k = (...((+0 + y_1) + y_2) ...) + y_k in the field's type
template <class T>
__global__ __launch_bounds__(256) void k_cast_decode(const float* __restrict__ comps, uint64_t N, int k,
                                                     T* __restrict__ out) {
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  for (uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x; j < N; j += stride) {
    T acc = (T)0;
    for (int i = 0; i < k; ++i) acc = acc + (T)comps[(uint64_t)i * N + j];
    out[j] = acc;
  }
}
template <class T>
hipError_t launch_cast_encode(const T* x, uint64_t N, int n, float* comps, unsigned long long* linf, hipStream_t s) {
  uint64_t wgs = (N + 255) / 256;
  if (wgs > 4096) wgs = 4096;
  if (wgs == 0) wgs = 1;
  if (n <= 4) hipLaunchKernelGGL((k_cast_encode<T, 4>), dim3((uint32_t)wgs), dim3(256), 0, s, x, N, n, comps, linf);
  else if (n <= 8) hipLaunchKernelGGL((k_cast_encode<T, 8>), dim3((uint32_t)wgs), dim3(256), 0, s, x, N, n, comps, linf);
  else hipLaunchKernelGGL((k_cast_encode<T, kMaxComps>), dim3((uint32_t)wgs), dim3(256), 0, s, x, N, n, comps, linf);
  return hipGetLastError();
}
template <class T> hipError_t launch_cast_decode(const float* comps, uint64_t N, int k, T* out, hipStream_t s) {
  uint64_t wgs = (N + 255) / 256;
  if (wgs > 4096) wgs = 4096;
  if (wgs == 0) wgs = 1;
  hipLaunchKernelGGL(k_cast_decode<T>, dim3((uint32_t)wgs), dim3(256), 0, s, comps, N, k, out);
  return hipGetLastError();
}
template hipError_t launch_cast_encode<float>(const float*, uint64_t, int, float*, unsigned long long*, hipStream_t);
template hipError_t launch_cast_encode<double>(const double*, uint64_t, int, float*, unsigned long long*, hipStream_t);
template hipError_t launch_cast_decode<float>(const float*, uint64_t, int, float*, hipStream_t);
template hipError_t launch_cast_decode<double>(const float*, uint64_t, int, double*, hipStream_t);

template <class T, int kCodec> void launch_aux_codec(AuxArgs a, int ncomp, uint64_t max_span, hipStream_t s) {
  constexpr uint64_t kWaves = 4 * 1024;  // 4 per SIMD
  constexpr uint64_t kLds = 48 * 1024;   // (four chunks of raw float64 blocks: 33 KiB)
  auto bytes = [](uint64_t words) { return ((words + 63) / 64 * 64 + 3) * 4; };
  auto grid = [&](uint64_t l) { return dim3((uint32_t)((a.g.nchunks + l - 1) / l), (uint32_t)ncomp); };
  if ((a.g.nchunks + 3) / 4 * (uint64_t)ncomp > kWaves && bytes(4 * max_span) <= kLds) {
    a.cap = (uint32_t)(4 * max_span);
    hipLaunchKernelGGL((k_aux<T, kCodec, 16>), grid(16), dim3(64), (uint32_t)bytes(a.cap), s, a);
  } else if (bytes(max_span) <= kLds) {
    a.cap = (uint32_t)max_span;
    hipLaunchKernelGGL((k_aux<T, kCodec, 4>), grid(4), dim3(64), (uint32_t)bytes(a.cap), s, a);
  } else {
    a.cap = 0;
    hipLaunchKernelGGL((k_aux<T, kCodec, 64>), grid(64), dim3(64), (uint32_t)bytes(0), s, a);
  }
}
template <class T> hipError_t launch_aux(AuxArgs a, int ncomp, uint64_t max_span, int codec, hipStream_t s) {
  if (codec == 0) launch_aux_codec<T, 0>(a, ncomp, max_span, s);
  else launch_aux_codec<T, 1>(a, ncomp, max_span, s);
  return hipGetLastError();
}
uint32_t range_groups(uint64_t n, uint64_t max_groups) {
  uint64_t wgs = (n + 4 * kRangeThreads - 1) / (4 * kRangeThreads);
  if (wgs > kRangeGroups) wgs = kRangeGroups;
  if (wgs > max_groups) wgs = max_groups;
  return wgs ? (uint32_t)wgs : 1u;
}
template <class T> hipError_t launch_range(const T* x, uint64_t n, unsigned long long* out, uint32_t groups, hipStream_t s) {
  hipLaunchKernelGGL(k_range<T>, dim3(groups), dim3(kRangeThreads), 0, s, x, n, out);
  return hipGetLastError();
}
hipError_t launch_fill64(unsigned long long* p, uint64_t n, unsigned long long v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill64, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

template hipError_t launch_aux<float>(AuxArgs, int, uint64_t, int, hipStream_t);
template hipError_t launch_aux<double>(AuxArgs, int, uint64_t, int, hipStream_t);
template hipError_t launch_range<float>(const float*, uint64_t, unsigned long long*, uint32_t, hipStream_t);
template hipError_t launch_range<double>(const double*, uint64_t, unsigned long long*, uint32_t, hipStream_t);
template hipError_t launch_sum_sq<float>(const float*, const float*, double, uint64_t, double*, double*, hipStream_t);
template hipError_t launch_sum_sq<double>(const double*, const double*, double, uint64_t, double*, double*,
                                          hipStream_t);

}  // namespace pmc
