// block_device.hpp -- device helpers around one 4x4x4 block per lane: its place
// in the field, gather and scatter with edge replication, error maxima.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "codec_device.hpp"
#include "launch.hpp"

namespace pmc {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void gmem_void_t;

// ---------------------------------------------------------------------------
// block gather / scatter with edge replication for partial blocks
struct BlockPos {
  uint64_t x0, y0, z0;
  uint32_t vx, vy, vz;  // valid extents (1..4)
};

__device__ __forceinline__ BlockPos block_pos(const Geo& g, uint64_t blk) {
  BlockPos b;
  uint64_t bx = blk % g.nbx;
  uint64_t t = blk / g.nbx;
  uint64_t by = t % g.nby;
  uint64_t bz = t / g.nby;
  b.x0 = 4 * bx;
  b.y0 = 4 * by;
  b.z0 = 4 * bz;
  b.vx = (uint32_t)min<uint64_t>(4, g.nx - b.x0);
  b.vy = (uint32_t)min<uint64_t>(4, g.ny - b.y0);
  b.vz = (uint32_t)min<uint64_t>(4, g.nz - b.z0);
  return b;
}

// bit l set when sample l of the block lies inside the field
__device__ __forceinline__ uint64_t valid_mask(const BlockPos& b) {
  const uint64_t xm = (1ull << b.vx) - 1ull;                                               // a row
  const uint64_t ym = (xm | xm << 4 | xm << 8 | xm << 12) & ((1ull << (4 * b.vy)) - 1ull);  // a z slice
  const uint64_t zm = ym | ym << 16 | ym << 32 | ym << 48;
  return b.vz == 4 ? zm : zm & ((1ull << (16 * b.vz)) - 1ull);
}
// |v| for sample l, or +0 where the sample lies outside the field: the mask
// bit becomes an all-ones / all-zeros word applied to the double's bits, so
// no per-sample condition (a lane mask) has to stay live
__device__ __forceinline__ double masked_abs(uint64_t m, int l, double v) {
  const uint64_t keep = 0ull - ((m >> l) & 1ull);
  return __longlong_as_double((long long)((uint64_t)__double_as_longlong(v) & keep & 0x7FFFFFFFFFFFFFFFull));
}

// one block row (ly, lz): 4 consecutive x values; rows of partial blocks
// repeat their last valid sample (edge replication on load)
template <class T>
__device__ __forceinline__ const T* row_ptr(const T* f, const Geo& g, const BlockPos& b, int r) {
  const uint32_t ly = min<uint32_t>(r & 3, b.vy - 1), lz = min<uint32_t>(r >> 2, b.vz - 1);
  return f + b.x0 + g.nx * ((b.y0 + ly) + g.ny * (b.z0 + lz));
}

// A full block's rows start at block_base + row_step(r): the step depends only
// on the field's shape, so it is the same for every lane (scalar registers)
// and a lane keeps one address instead of one per row.
template <class T> __device__ __forceinline__ T* block_base(T* f, const Geo& g, const BlockPos& b) {
  return f + (b.x0 + g.nx * (b.y0 + g.ny * b.z0));
}
__device__ __forceinline__ uint64_t row_step(const Geo& g, int r) {
  return g.nx * (uint64_t)(r & 3) + g.nx * g.ny * (uint64_t)(r >> 2);
}

// Row pieces are 16-byte accesses at any sample: rows whose length is no
// multiple of 16 bytes take them too.  Four 4-byte accesses with a 16-byte
// stride between lanes had cost four times the requests: 251x203x181 float32
// refined component by component, six calls, 173 us, now 126.  (The encoder,
// which puts such rows into LDS once for all components, gained nothing.)
typedef float any_f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef double any_d2 __attribute__((ext_vector_type(2), aligned(8)));
template <class T> __device__ __forceinline__ void load_row16(const T* row, T v[4]) {
  if constexpr (sizeof(T) == 4) {
    const any_f4 q = *reinterpret_cast<const any_f4*>(row);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  } else {
    const any_d2 q0 = *reinterpret_cast<const any_d2*>(row);
    const any_d2 q1 = *reinterpret_cast<const any_d2*>(row + 2);
    v[0] = q0.x; v[1] = q0.y; v[2] = q1.x; v[3] = q1.y;
  }
}

template <class T>
__device__ __forceinline__ void load_block(const T* __restrict__ f, const Geo& g, const BlockPos& b, T v[64]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const T* row = row_ptr(f, g, b, r);
    if (b.vx == 4) {
      load_row16(row, v + 4 * r);
    } else {
      const uint32_t m = b.vx - 1;
      v[4 * r] = row[0];
      v[4 * r + 1] = row[min<uint32_t>(1, m)];
      v[4 * r + 2] = row[min<uint32_t>(2, m)];
      v[4 * r + 3] = row[min<uint32_t>(3, m)];
    }
  }
}

// one 16-byte row piece written with the streaming (nt) cache policy: the
// partial sums a launch writes are read back only by a later launch, after far
// more than the L2 holds has passed through it, so keeping them in L2 would
// only push out lines this launch still reads
typedef float nt_f4 __attribute__((ext_vector_type(4)));
typedef double nt_d2 __attribute__((ext_vector_type(2)));
typedef uint32_t nt_u4 __attribute__((ext_vector_type(4)));
template <class T>
__device__ __forceinline__ void store_row16_nt(T* row, T a, T b, T c, T d) {
  if constexpr (sizeof(T) == 4) {
    __builtin_nontemporal_store(any_f4{a, b, c, d}, reinterpret_cast<any_f4*>(row));
  } else {
    __builtin_nontemporal_store(any_d2{a, b}, reinterpret_cast<any_d2*>(row));
    __builtin_nontemporal_store(any_d2{c, d}, reinterpret_cast<any_d2*>(row + 2));
  }
}

template <class T>
__device__ __forceinline__ void store_block(T* __restrict__ f, const Geo& g, const BlockPos& b, const T v[64]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if ((uint32_t)(r & 3) >= b.vy || (uint32_t)(r >> 2) >= b.vz) continue;
    T* row = const_cast<T*>(row_ptr((const T*)f, g, b, r));
    if (b.vx == 4) {
      store_row16_nt(row, v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]);
    } else {
      row[0] = v[4 * r];
      if (b.vx > 1) row[1] = v[4 * r + 1];
      if (b.vx > 2) row[2] = v[4 * r + 2];
    }
  }
}

// store row r of a block (valid samples only); wfull: every lane of the wave
// has a full block of aligned rows (a wave-uniform flag), so the store needs
// no per-lane path
template <class T>
__device__ __forceinline__ void store_row(T* __restrict__ f, const Geo& g, const BlockPos& b, int r, const T v[4],
                                          bool wfull = false) {
  if (!wfull && ((uint32_t)(r & 3) >= b.vy || (uint32_t)(r >> 2) >= b.vz)) return;
  T* row = wfull ? block_base(f, g, b) + row_step(g, r) : const_cast<T*>(row_ptr((const T*)f, g, b, r));
  if (wfull || b.vx == 4) {
    store_row16_nt(row, v[0], v[1], v[2], v[3]);
  } else {
    row[0] = v[0];
    if (b.vx > 1) row[1] = v[1];
    if (b.vx > 2) row[2] = v[2];
  }
}

// the samples of a block that lie in a box, read from / written to the box's
// own dense array (x fastest); samples outside the field are outside every
// box, and samples of the block outside the box are not touched (read as +0)
template <class T>
__device__ __forceinline__ void load_box(const T* __restrict__ f, const BoxArgs& bx, const BlockPos& b, T v[64]) {
  const uint64_t nx = bx.hi[0] - bx.lo[0], ny = bx.hi[1] - bx.lo[1];
#pragma unroll
  for (int l = 0; l < 64; ++l) {
    const uint64_t x = b.x0 + (l & 3), y = b.y0 + ((l >> 2) & 3), z = b.z0 + (l >> 4);
    v[l] = (x >= bx.lo[0] && x < bx.hi[0] && y >= bx.lo[1] && y < bx.hi[1] && z >= bx.lo[2] && z < bx.hi[2])
               ? f[(x - bx.lo[0]) + nx * ((y - bx.lo[1]) + ny * (z - bx.lo[2]))]
               : (T)0;
  }
}
template <class T>
__device__ __forceinline__ void store_box_row(T* __restrict__ f, const BoxArgs& bx, const BlockPos& b, int r,
                                              const T v[4]) {
  const uint64_t nx = bx.hi[0] - bx.lo[0], ny = bx.hi[1] - bx.lo[1];
  const uint64_t y = b.y0 + (r & 3), z = b.z0 + (r >> 2);
  if (y < bx.lo[1] || y >= bx.hi[1] || z < bx.lo[2] || z >= bx.hi[2]) return;
  T* row = f + nx * ((y - bx.lo[1]) + ny * (z - bx.lo[2]));
  if (b.x0 >= bx.lo[0] && b.x0 + 4 <= bx.hi[0]) {
    store_row16_nt(row + (b.x0 - bx.lo[0]), v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t x = b.x0 + k;
      if (x >= bx.lo[0] && x < bx.hi[0]) row[x - bx.lo[0]] = v[k];
    }
  }
}
template <class T>
__device__ __forceinline__ void store_box(T* __restrict__ f, const BoxArgs& bx, const BlockPos& b, const T v[64]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) store_box_row(f, bx, b, r, v + 4 * r);
}

// load row r of a block (edge replication as in load_block); a null field
// reads as +0
template <class T>
__device__ __forceinline__ void load_row(const T* f, const Geo& g, const BlockPos& b, int r, T v[4]) {
  if (!f) {
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = (T)0;
    return;
  }
  const T* row = row_ptr(f, g, b, r);
  if (b.vx == 4) {
    load_row16(row, v);
  } else {
    const uint32_t m = b.vx - 1;
    v[0] = row[0];
    v[1] = row[min<uint32_t>(1, m)];
    v[2] = row[min<uint32_t>(2, m)];
    v[3] = row[min<uint32_t>(3, m)];
  }
}

// rows [r0, r0 + R) of a block into v[4R].  When every lane of the wave has a
// full block of aligned rows (wfull, a wave-uniform flag) the R loads are
// plain 16-byte loads at the block base plus a uniform step, with no per-lane
// branch, so they are all in flight together; otherwise each row takes
// load_row's per-lane path.  A null field reads as +0.
template <class T, int R>
__device__ __forceinline__ void load_rows(const T* f, const Geo& g, const BlockPos& b, int r0, bool wfull,
                                          T v[4 * R]) {
  if (!f) {
#pragma unroll
    for (int k = 0; k < 4 * R; ++k) v[k] = (T)0;
    return;
  }
  if (wfull) {
    const T* const base = block_base(f, g, b);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const T* row = base + row_step(g, r0 + k);
      load_row16(row, v + 4 * k);
    }
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) load_row(f, g, b, r0 + k, v + 4 * k);
  }
}

// Where x~ goes from one launch of the encoder to the next it is kept in one
// tile per wave, the wave's 64 blocks as [row r][lane][16-byte piece]
// (float32: 4 values; float64: [row r][half][lane][2 values]): coalesced
// whatever the field's shape, and the layout the encoder has x in in LDS.
constexpr uint64_t kTileValues = 64 * 64;  // values of one wave's tile
template <class T> __device__ __forceinline__ uint32_t tile_index(uint32_t lane, int r, int t) {
  if constexpr (sizeof(T) == 4) return ((uint32_t)r * 64 + lane) * 4 + (uint32_t)t;
  else return (((uint32_t)r * 2 + (uint32_t)(t >> 1)) * 64 + lane) * 2 + (uint32_t)(t & 1);
}
// (job pointers come out of constant memory as generic ones: the accesses name
// the global address space, or they would be flat instructions)
template <class T> using gptr = __attribute__((address_space(1))) T*;
template <class T> __device__ __forceinline__ gptr<T> to_global(T* p) { return (gptr<T>)p; }
// row r of this lane's block from a wave's tile
template <class T> __device__ __forceinline__ void tile_load_row(gptr<const T> tile, uint32_t lane, int r, T v[4]) {
  if constexpr (sizeof(T) == 4) {
    const nt_f4 q = *(gptr<const nt_f4>)(tile + tile_index<T>(lane, r, 0));
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  } else {
    const nt_d2 q0 = *(gptr<const nt_d2>)(tile + tile_index<T>(lane, r, 0));
    const nt_d2 q1 = *(gptr<const nt_d2>)(tile + tile_index<T>(lane, r, 2));
    v[0] = q0.x; v[1] = q0.y; v[2] = q1.x; v[3] = q1.y;
  }
}
// row r of this lane's block into a wave's tile
template <class T> __device__ __forceinline__ void tile_store_row(gptr<T> tile, uint32_t lane, int r, const T v[4]) {
  if constexpr (sizeof(T) == 4) {
    *(gptr<nt_f4>)(tile + tile_index<T>(lane, r, 0)) = nt_f4{v[0], v[1], v[2], v[3]};
  } else {
    *(gptr<nt_d2>)(tile + tile_index<T>(lane, r, 0)) = nt_d2{v[0], v[1]};
    *(gptr<nt_d2>)(tile + tile_index<T>(lane, r, 2)) = nt_d2{v[2], v[3]};
  }
}
// the whole block of lane `lane` of wave w
template <class T> __device__ __forceinline__ void tile_load(const T* tiles, uint64_t w, uint32_t lane, T v[64]) {
  const gptr<const T> tile = to_global(tiles) + w * kTileValues;
#pragma unroll
  for (int r = 0; r < 16; ++r) tile_load_row<T>(tile, lane, r, v + 4 * r);
}
template <class T> __device__ __forceinline__ void tile_store(T* tiles, uint64_t w, uint32_t lane, const T v[64]) {
  const gptr<T> tile = to_global(tiles) + w * kTileValues;
#pragma unroll
  for (int r = 0; r < 16; ++r) tile_store_row<T>(tile, lane, r, v + 4 * r);
}

__device__ __forceinline__ BlockPos opaque_pos(BlockPos b) {
  b.x0 = opaque(b.x0);
  b.y0 = opaque(b.y0);
  b.z0 = opaque(b.z0);
  return b;
}

// a + v * scale where v * scale is exact: one fused multiply-add equals the
// plain sum of the (exact) product
__device__ __forceinline__ float fma_exact(float v, float scale, float a) { return __builtin_fmaf(v, scale, a); }
__device__ __forceinline__ double fma_exact(double v, double scale, double a) { return a + v * scale; }

// NaN-propagating max, matching "take a if not a <= m"
__device__ __forceinline__ double nmax(double m, double a) { return a <= m ? m : a; }
// the same maximum where no operand is NaN: one v_max_f64 instead of a
// compare and two selects.  The candidate checks take it: |x - x~_i| with
// x finite (an input with NaN or Inf fails the call whatever its streams)
// and x~_i finite or, on overflow, infinite (x~_{i-1} stays within tau of x)
__device__ __forceinline__ double nmax_num(double m, double a) { return __builtin_fmax(m, a); }

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = nmax(v, __shfl_xor(v, d, 64));
  return v;
}

}  // namespace pmc
