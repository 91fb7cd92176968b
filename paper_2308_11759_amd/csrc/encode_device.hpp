// encode_device.hpp -- Alg. 1 (Sec. 4.1) for one field: every component of a
// block in one pass of one lane, instantiated per element type by
// encode_f32.hip and encode_f64.hip.
//
// One wave takes 64 consecutive blocks (4 chunks) through all components: the
// residual, block coding, decode-for-verify, the x~ update and the measured
// error (Sec. 4.3), and the chunk bitstreams assembled in LDS.  x stays in LDS
// and x~ in registers for the whole pass, so a component touches memory only
// for its payload and block offsets.  What does not fit beside x~ is formed
// again instead of held: the residual (x - x~) for every candidate and, in
// the rare cases that need it there, for the emission.
//
// What bounds it: the vector ALUs (3.8 K instructions per wave and component at
// 512^3 float32, 1.5 of 2.0 ms), then what two waves per SIMD (float64: one,
// x alone is 32 KiB of LDS) leave of the LDS latency.  One launch per component
// with x~ in memory moved 1.73 GB per 512^3 component and ran 8 of them in 3.1
// ms (float64 256^3: 1.1 ms, now 0.6; codec 1 at 256^3 float32: 0.50, now 0.38).
#pragma once
#include "block_device.hpp"

namespace pmc {

enum { MODE_EMPTY = 0, MODE_CODED = 1, MODE_RAW = 2 };

// LDS words of a wave's emission window: with x (16 or 32 KiB) and the
// unsqueeze table it fills an eighth (float32: 8 one-wave workgroups per CU)
// or a quarter (float64: 4) of the CU's 160 KiB.  A span of up to 6.9 bits per
// value (13.8 in float64) is emitted in one pass.
template <class T> constexpr uint32_t emit_words() { return sizeof(T) == 4 ? 880u : 1792u; }
constexpr uint32_t kEmitPad = 4;  // a put touches up to two words past its last bit

// the block's x values in LDS, [row r][lane][4 values] (f32) or
// [row r][half h][lane][2 values] (f64): each 16-byte piece of a row is one
// direct global->LDS load (global_load_lds_dwordx4), so x never occupies
// VGPRs; partial or unaligned rows are written by plain loads
template <class T> struct XLds {
  T* base;  // s_x
  uint32_t lane;
  __device__ __forceinline__ T* slot(int r, int t) const {
    if constexpr (sizeof(T) == 4) return base + ((uint32_t)r * 64 + lane) * 4 + t;
    else return base + (((uint32_t)r * 2 + (t >> 1)) * 64 + lane) * 2 + (t & 1);
  }
  __device__ __forceinline__ T at(int l) const { return *slot(l >> 2, l & 3); }
};

// edge replication of a partial block's residual, in registers: each padded
// sample takes the value of the last valid sample on each axis (x, then y,
// then z), as the block gather of a partial block does
template <class T>
__device__ __forceinline__ void replicate_edges(T e[64], uint32_t vx, uint32_t vy, uint32_t vz) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int t = 1; t < 4; ++t) e[4 * r + t] = (uint32_t)t < vx ? e[4 * r + t] : e[4 * r + t - 1];
#pragma unroll
  for (int lz = 0; lz < 4; ++lz)
#pragma unroll
    for (int ly = 1; ly < 4; ++ly)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int l = 4 * ly + 16 * lz + t;
        e[l] = (uint32_t)ly < vy ? e[l] : e[l - 4];
      }
#pragma unroll
  for (int lz = 1; lz < 4; ++lz)
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      const int l = 16 * lz + m;
      e[l] = (uint32_t)lz < vz ? e[l] : e[l - 16];
    }
}

// (the direct loads are only issued here: the caller waits, s_waitcnt 0,
// before reading s_x.  x is read from memory once, so its loads take the
// streaming (nt) policy, cache-policy bit 1)
constexpr int kNt = 2;
template <class T>
__device__ __forceinline__ void load_block_lds(gptr<const T> f, const Geo& g, const BlockPos& b, T* s_x, uint32_t lane,
                                               bool wfull) {
  const bool vec = wfull || (b.vx == 4 && g.rows_aligned);
  XLds<T> X{s_x, lane};
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t ly = min<uint32_t>(r & 3, b.vy - 1), lz = min<uint32_t>(r >> 2, b.vz - 1);
    const gptr<const T> row = f + (b.x0 + g.nx * ((b.y0 + ly) + g.ny * (b.z0 + lz)));
    if (vec) {
      if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_global_load_lds((gmem_void_t*)row, (lds_void_t*)(s_x + r * 256), 16, 0, kNt);
      } else {
        __builtin_amdgcn_global_load_lds((gmem_void_t*)row, (lds_void_t*)(s_x + (r * 2) * 128), 16, 0, kNt);
        __builtin_amdgcn_global_load_lds((gmem_void_t*)(row + 2), (lds_void_t*)(s_x + (r * 2 + 1) * 128), 16, 0,
                                         kNt);
      }
    } else {
      const uint32_t m = b.vx - 1;
#pragma unroll
      for (int t = 0; t < 4; ++t) *X.slot(r, t) = row[min<uint32_t>(t, m)];
    }
  }
}

// ---------------------------------------------------------------------------
// bits of one lane into the wave's window of zeroed LDS words, OR-ed where
// words are shared with neighbouring lanes.  pos counts from the window's
// first bit.  kWindows: the wave's span takes several windows, so words outside
// this one go to the spare word behind it (a negative position wraps to a
// large word index).
template <bool kWindows> struct BitOr {
  uint32_t* buf;
  uint32_t nw;  // words of the window; word nw is spare
  int32_t pos;
  __device__ __forceinline__ void word(uint32_t k, uint32_t v) const {
    if constexpr (kWindows) k = k < nw ? k : nw;
    atomicOr(&buf[k], v);
  }
  // count <= 64, value holds only its low `count` bits
  __device__ __forceinline__ void put(uint64_t value, uint32_t count) {
    const uint32_t o = (uint32_t)pos & 31u, k = (uint32_t)(pos >> 5);
    const uint64_t a = value << o;
    const uint32_t hi = (uint32_t)(value >> 32);
    word(k, (uint32_t)a);
    word(k + 1, (uint32_t)(a >> 32));
    word(k + 2, (hi >> 1) >> (~o & 31u));  // hi >> (32 - o), 0 for o = 0
    pos += (int32_t)count;
  }
  // count <= 32
  __device__ __forceinline__ void put32(uint32_t value, uint32_t count) {
    const uint32_t o = (uint32_t)pos & 31u, k = (uint32_t)(pos >> 5);
    word(k, value << o);
    word(k + 1, (value >> 1) >> (~o & 31u));
    pos += (int32_t)count;
  }
};

// unsqueeze of m's low 32 bits only (the result stays below bit 64)
__device__ __forceinline__ uint64_t unsqueeze32(uint32_t m, const uint16_t* tab) {
  const uint32_t b0 = m & 0xFFu, b1 = (m >> 8) & 0xFFu, b2 = (m >> 16) & 0xFFu, b3 = m >> 24;
  const uint32_t c1 = (uint32_t)__builtin_popcount(b0);
  const uint32_t c2 = c1 + (uint32_t)__builtin_popcount(b1);
  const uint32_t c3 = c2 + (uint32_t)__builtin_popcount(b2);
  return (uint64_t)tab[b0] | ((uint64_t)tab[b1] << (8 + c1)) | ((uint64_t)tab[b2] << (16 + c2)) |
         ((uint64_t)tab[b3] << (24 + c3));
}

// emit one plane with the group-testing coder, n = significant prefix: the
// n verbatim bits, then the whole group-test section at once.  In the section
// the i-th newly significant coefficient, at k past the prefix, puts its
// terminator at bit k + i (unsqueeze); every terminator but the last is
// followed by a positive test, bit 0 is the first test, and a negative test
// ends the section.  When the last significant coefficient is coefficient 63
// its terminator is implied and the section ends just before it.
template <bool kWindows>
__device__ __forceinline__ void plane_emit(BitOr<kWindows>& w, uint64_t wd, uint32_t& n, const uint16_t* tab) {
  if (n > 0) w.put((wd << (64u - n)) >> (64u - n), n);
  if (n >= 64) return;
  const uint64_t rest = wd >> n;
  if (rest == 0) {  // a single negative test
    w.pos += 1;
    return;
  }
  const uint32_t top = 63u - (uint32_t)__builtin_clzll(rest);  // last new coefficient, past the prefix
  const uint32_t lastt = top + (uint32_t)__builtin_popcountll(rest);  // its terminator's bit
  const bool implied = n + top == 63u;
  const uint32_t len = implied ? lastt : lastt + 2u;
  if (__all(top < 32u && lastt < 63u)) {  // (a wave-uniform choice: the section fits 64 bits)
    const uint64_t t = unsqueeze32((uint32_t)rest, tab);
    // positive tests: bit 0 and the bit after every terminator but the last;
    // an implied terminator is dropped as well
    const uint64_t drop = (implied ? 3ull : 2ull) << lastt;
    w.put((t | (t << 1) | 1ull) & ~drop, len);
  } else {
    uint64_t tlo, thi;
    unsqueeze64(rest, tab, tlo, thi);
    uint64_t slo = tlo | (tlo << 1) | 1ull, shi = thi | (thi << 1) | (tlo >> 63);
    const uint32_t a = lastt + 1u;
    if (a < 64u) slo &= ~(1ull << a);
    else if (a < 128u) shi &= ~(1ull << (a - 64u));  // (128: all 64 coefficients new, the last one implied)
    if (implied) {
      if (lastt < 64u) slo &= ~(1ull << lastt);
      else shi &= ~(1ull << (lastt - 64u));
    }
    w.put(slo, len < 64u ? len : 64u);
    if (len > 64u) w.put(shi, len - 64u);
  }
  n += top + 1u;
}

// Plane words of W planes (W = 4 or 8) from the biased coefficients v = q +
// M (M the negabinary mask; the negabinary word is v ^ M): A[W-1-t] holds
// plane base + t of coefficients 0..31, A[2W-1-t] of 32..63, for the lane's
// own base <= P - W.  The W bits of every coefficient are gathered into words
// of 32 / W slices and go through the W x W bit transposes of
// transpose_groups (its own inverse).  About 160 (W = 4) or 250 (W = 8)
// vector operations instead of 450 for 16 planes at once: residual components
// code 3 to 5 planes.
template <int W, class U>
__device__ __forceinline__ void plane_slots(const U v[64], int base, uint32_t A[2 * W]) {
  constexpr int P = 8 * (int)sizeof(U);
  const int sh = P - W - base;
  auto gather = [&](auto slice) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < W; ++i) {
        if constexpr (W == 8) {
          const uint32_t a0 = slice(v[32 * h + i]), a1 = slice(v[32 * h + 8 + i]);
          const uint32_t a2 = slice(v[32 * h + 16 + i]), a3 = slice(v[32 * h + 24 + i]);
          const uint32_t lo = __builtin_amdgcn_perm(a1, a0, 0x0C0C0400u), hi = __builtin_amdgcn_perm(a3, a2, 0x04000C0Cu);
          A[W * h + i] = lo | hi;
        } else {
          uint32_t w = 0;
#pragma unroll
          for (int g = 0; g < 32 / W; ++g)
            w |= __builtin_amdgcn_ubfe(slice(v[32 * h + W * g + i]), 0u, (uint32_t)W) << (W * g);
          A[W * h + i] = w;
        }
      }
  };
  if constexpr (sizeof(U) == 4) {
    gather([&](U x) { return (uint32_t)x >> sh; });
  } else {
    // (a wave-uniform choice: every plane in the high words)
    if (__all(sh >= 32)) gather([&](U x) { return (uint32_t)(x >> 32) >> (sh & 31); });
    else gather([&](U x) { return (uint32_t)(x >> sh); });
  }
  const uint32_t MM = (sh & 1) ? 0x55555555u : 0xAAAAAAAAu;
#pragma unroll
  for (int i = 0; i < 2 * W; ++i) A[i] ^= MM;
  transpose_groups<W>(A);
}

// bits of planes [zl, p) of the group-testing coder, W planes at a time from
// the first non-empty one; the zl empty planes above cost one bit each.  A is
// left with the last group's words: all there are where no lane has more than
// W planes.  No per-lane branches (nor anywhere
// between the candidate's wave-uniform choices of a route): around one, the
// compiler keeps each side's results live through the other side.
template <int W, class U>
__device__ __forceinline__ uint32_t planes_cost(const U v[64], int zl, int p, uint32_t A[2 * W]) {
  constexpr int P = 8 * (int)sizeof(U);
  uint32_t n = 0, bits = (uint32_t)zl;
  auto group = [&](int b, uint32_t* G) {
    const int base = b < P - W ? b : P - W;
    plane_slots<W>(v, base, G);
#pragma unroll
    for (int t = 0; t < W; ++t) {
      const bool on = base + t >= b && base + t < p;
      const uint64_t wd = (uint64_t)G[W - 1 - t] | ((uint64_t)G[2 * W - 1 - t] << 32);
      // n verbatim bits, one test per new coefficient, the distance to the
      // last one, and the closing test (or the implied last one)
      const bool more = n < 64 && (wd >> (n & 63u)) != 0;
      const uint32_t h1 = 64u - (uint32_t)__builtin_clzll(wd | 1ull);  // past the last one
      const uint32_t m = (uint32_t)__builtin_popcountll(wd >> (n & 63u));
      const uint32_t cm = m + h1 + (h1 < 64u ? 1u : 0u) - (h1 < 64u ? 0u : 1u);
      const uint32_t c = more ? cm : n + (n < 64u ? 1u : 0u);
      bits += on ? c : 0u;
      n = on && more ? h1 : n;
    }
  };
  group(zl, A);
#pragma unroll 1
  for (int k = W; __any(zl + k < p); k += W) group(zl + k, A);
  return bits;
}

// emit planes [b, min(p, base + W)) of a group whose plane words are in G
template <int W, bool kWindows>
__device__ __forceinline__ void group_emit(BitOr<kWindows>& w, uint32_t G[2 * W], int base, int b, int p, uint32_t& n,
                                           const uint16_t* tab) {
#pragma unroll 1
  for (int t = base; t < base + W && t < p; ++t) {
    if (t >= b) plane_emit(w, (uint64_t)G[W - 1] | ((uint64_t)G[2 * W - 1] << 32), n, tab);
#pragma unroll
    for (int k = W - 1; k > 0; --k) {  // the next plane to the top
      G[k] = G[k - 1];
      G[W + k] = G[W + k - 1];
    }
  }
}
// emit planes [zl, p) from the coefficients
template <bool kWindows, class U>
__device__ __forceinline__ void planes_emit(BitOr<kWindows>& w, const U v[64], int zl, int p, const uint16_t* tab) {
  constexpr int P = 8 * (int)sizeof(U), W = 8;
  uint32_t n = 0;
  w.pos += zl;
#pragma unroll 1
  for (int b = zl; b < p; b += W) {
    const int base = b < P - W ? b : P - W;
    uint32_t G[2 * W];
    plane_slots<W>(v, base, G);
    group_emit<W>(w, G, base, b, p, n, tab);
  }
}

// ---------------------------------------------------------------------------
// small wave reductions without LDS: a row is 16 lanes, one chunk
template <int N> __device__ __forceinline__ uint32_t row_shr(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + N, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t row_incl_scan(uint32_t v) {
  v += row_shr<1>(v);
  v += row_shr<2>(v);
  v += row_shr<4>(v);
  v += row_shr<8>(v);
  return v;
}
template <int N> __device__ __forceinline__ double row_shr(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  return __longlong_as_double((long long)((uint64_t)row_shr<N>((uint32_t)b) |
                                          ((uint64_t)row_shr<N>((uint32_t)(b >> 32)) << 32)));
}
__device__ __forceinline__ double read_lane(double v, int l) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  return __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l) |
                                          ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l) << 32)));
}
// largest of the lanes' non-negative values (every lane active)
__device__ __forceinline__ double wave_max_pos(double v) {
  v = __builtin_fmax(v, row_shr<1>(v));
  v = __builtin_fmax(v, row_shr<2>(v));
  v = __builtin_fmax(v, row_shr<4>(v));
  v = __builtin_fmax(v, row_shr<8>(v));
  return __builtin_fmax(__builtin_fmax(read_lane(v, 15), read_lane(v, 31)),
                        __builtin_fmax(read_lane(v, 47), read_lane(v, 63)));
}

// the candidate check: row holds the dequantised values over scale (the
// products are exact) and becomes x~_i = x~_{i-1} + x_i in the field precision;
// the largest |x - x~_i| in double over the block's valid samples.  One check
// after the routes that fill row: with one in each, the compiler merged their
// common parts around 64 more live values.
template <class T, bool kFull>
__device__ __forceinline__ double check_rows(const XLds<T>& X, const T xt[64], uint64_t vmask, T scale, T row[64]) {
  double ea = 0.0;
#pragma unroll
  for (int l = 0; l < 64; ++l) {
    row[l] = fma_exact(row[l], scale, xt[l]);
    const double df = (double)X.at(l) - (double)row[l];
    ea = nmax_num(ea, kFull ? __builtin_fabs(df) : masked_abs(vmask, l, df));
  }
  return ea;
}

// the block grid of a job in constant memory, member by member
template <class F> __device__ __forceinline__ Geo load_geo(const F& f) {
  Geo g;
  g.nx = f.g.nx;
  g.ny = f.g.ny;
  g.nz = f.g.nz;
  g.nbx = f.g.nbx;
  g.nby = f.g.nby;
  g.nbz = f.g.nbz;
  g.nblocks = f.g.nblocks;
  g.nchunks = f.g.nchunks;
  g.rows_aligned = f.g.rows_aligned;
  g.pad = 0;
  return g;
}

// One wave = 64 consecutive blocks = 4 chunks; `wave` numbers these groups
// within the field f (components [f.comp0, f.comp1) of f.ncomp).  s_x: 64 * 64
// values of LDS, s_emit: emit_words<T>() + kEmitPad words, both owned by this
// wave.  kFull: every block is full and rows are aligned (all three dimensions
// multiples of 4), so the per-lane edge paths compile away.  kCodec: 0 the
// block-transform codec, 1 prediction and quantisation.
template <class T, bool kFull, int kCodec, class F>
__device__ __forceinline__ void encode_wave(const F& f, uint32_t wave, T* s_x, uint32_t* s_emit, const uint16_t* unsq) {
  typedef typename FT<T>::U U;
  typedef typename FT<T>::S S;
  constexpr int P = FT<T>::P;
  constexpr int EB = FT<T>::EBITS;
  constexpr uint32_t NW = emit_words<T>();

  if (f.comp0 >= f.comp1) return;  // a field of a batch with fewer components
  const uint32_t lane = threadIdx.x;
  const uint64_t blk = (uint64_t)wave * 64 + lane;
  const Geo g = load_geo(f);
  const bool active = blk < g.nblocks;
  BlockPos bp = block_pos(g, active ? blk : 0);
  if constexpr (kFull) {
    bp.vx = 4;
    bp.vy = 4;
    bp.vz = 4;
  }
  // every lane has a full block of aligned rows: row accesses without per-lane paths
  const bool wfull = kFull || __all(bp.vx == 4 && bp.vy == 4 && bp.vz == 4 && g.rows_aligned);
  load_block_lds<T>(to_global((const T*)f.x), g, bp, s_x, lane, wfull);
  const uint64_t vmask = kFull ? ~0ull : valid_mask(bp);
  const uint32_t vx = bp.vx, vy = bp.vy, vz = bp.vz;
  const int ncomp = f.ncomp, comp1 = f.comp1;
  const gptr<T> tile = to_global((T*)f.tiles) + (uint64_t)wave * kTileValues;  // only between launches
  const gptr<uint32_t> slot = to_global(f.staging) + (uint64_t)wave * f.slot_words;
  const uint32_t limit = wave + 1 == job_waves(f) ? f.slot_last : f.slot_words;
  uint32_t cur = 0;  // words of the slot in use
  __builtin_amdgcn_s_waitcnt(0);  // direct loads and LDS writes complete

  // x~_{i-1}, and the error before the component, max |x - x~_{i-1}| in
  // double over the block's samples
  T xt[64];
  double eb = 0.0;
  int i = f.comp0;
  if (i > 0) {  // a later launch: from the tile
    const XLds<T> X{s_x, lane};
#pragma unroll
    for (int k = 0; k < 16; ++k) tile_load_row<T>(tile, lane, k, xt + 4 * k);
#pragma unroll
    for (int l = 0; l < 64; ++l) eb = nmax_num(eb, masked_abs(vmask, l, (double)X.at(l) - (double)xt[l]));
  } else {
#pragma unroll
    for (int l = 0; l < 64; ++l) xt[l] = (T)0;
  }
  // the residual x - x~_{i-1}, edge-replicated in a partial block.  Formed
  // from opaque copies, so that it is formed where it is asked for and not
  // held in between.
  auto residual = [&](T r[64]) {
    const XLds<T> X{s_x, opaque(lane)};
#pragma unroll
    for (int l = 0; l < 64; ++l) r[l] = X.at(l) - xt[l];
    if constexpr (!kFull) {
      if (!wfull) replicate_edges(r, vx, vy, vz);
    }
  };
#pragma unroll 1
  for (; i < comp1; ++i) {
    i = __builtin_amdgcn_readfirstlane(opaque(i));
    const bool first = i == 0;
    const double tau = f.tau[i];
    const int minexp = f.minexp[i];
    bool nonfinite = false, miss = false;
    int mode = MODE_EMPTY, delta = 0, zl = 0, p = 0, emax = 0;
    uint32_t nbits = 1;
    double err = eb;
    T row[64];       // x~_i of a block that changes it
    uint32_t A[16];  // plane words of the candidates, 4 or 8 planes
    int aw = 0;      // which, if they are all the planes of every lane, else 0 (wave-uniform)

    // acceptance: smallest plane count p >= p0 whose block meets tau without
    // raising the error; else empty (already within tau) or raw.  The loop is
    // the wave's: a lane that has its candidate takes it again, to the same
    // result, while others go on, so that nothing is held across iterations
    // for it (a per-lane exit kept row and A live through the whole body:
    // hundreds of spills).  Lanes without a block follow along.
    bool pending = active;
#pragma unroll 1
    do {
      T r[64];
      residual(r);
      // largest |residual| (the block exponent, the all-zero test).  The
      // first component's is the largest |x|, as an integer maximum that a
      // NaN or an infinity wins (non-finite input); later residuals are
      // finite: a component is only accepted with max |x - x~_i| <= min(tau,
      // the error before it), so |x - x~| never exceeds the block's |x|.
      U maxabs = 0;
      if (first) {
#pragma unroll
        for (int l = 0; l < 64; ++l) {
          const U ab = abs_bits(r[l]);
          maxabs = ab > maxabs ? ab : maxabs;
        }
        nonfinite = maxabs >= abs_bits((T)__builtin_inf());
        // (edge samples repeat valid ones; a NaN fails the call, whatever is coded)
        eb = (double)from_raw(maxabs, (T)0);
      } else {
        T m = (T)0;
#pragma unroll
        for (int l = 0; l < 64; ++l) m = fmax_t(m, fabs_t(r[l]));
        maxabs = abs_bits(m);
      }
      emax = block_emax<T>(maxabs);
      p = emax - minexp + kGuard;
      p = (p < 0 ? 0 : (p > P ? P : p)) + delta;

      const XLds<T> X{s_x, opaque(lane)};
      bool feasible = false;
      uint32_t cb = 0;
      T scale = (T)1;
      if constexpr (kCodec == 0) {
        U v[64];  // the coefficients in coded order plus the negabinary mask
        forward_coeffs_biased<T>(r, emax, v);
        U any = 0;
#pragma unroll
        for (int l = 0; l < 64; ++l) any |= v[l] ^ FT<T>::NB;
        zl = any ? (sizeof(U) == 4 ? __builtin_clz((uint32_t)any) : __builtin_clzll((uint64_t)any)) : P;
        const bool ok = active && maxabs != 0 && p >= 1 && p <= P;
        p = ok ? p : 1;  // (of no consequence: a cheap candidate)
        zl = zl < p ? zl : p;
        const int np = p - zl;
        cb = 2u + (uint32_t)(delta + 1) + (uint32_t)EB;
        if (__all(np <= 4)) {
          cb += planes_cost<4>(v, zl, p, A);
          aw = 4;
        } else {
          cb += planes_cost<8>(v, zl, p, A);
          aw = __all(np <= 8) ? 8 : 0;
        }
        feasible = ok && cb <= (uint32_t)FT<T>::RAW_BITS;
        if (__all(!feasible || (p <= 10 && hi16_exact(emax, (T)0)))) {
          // planes in the top ten bit positions, every result normal: the
          // packed 16-bit lifting (see lift_dequant_add_hi16)
          const uint32_t m16 = 0xFFFFu & ~(0xFFFFu >> (p & 15)), m2 = m16 | (m16 << 16);
          const v2s off = __builtin_bit_cast(v2s, m2 & 0xAAAAAAAAu);
          v2s R[32];
#pragma unroll
          for (int m = 0; m < 32; ++m)
            R[m] = wsub(__builtin_bit_cast(v2s, __builtin_amdgcn_perm(high_word(v[kInvOrder.at[2 * m + 1]]),
                                                                      high_word(v[kInvOrder.at[2 * m]]), 0x07060302u) & m2),
                        off);
          lift_zy_hi16(R);
#pragma unroll
          for (int k = 0; k < 8; ++k) lift_x_hi16<T>(R, k, row + 8 * k);
          scale = hi16_scale<T>(emax);
        } else if (sizeof(T) == 8 && __all(!feasible || (p <= 26 && emax >= -992))) {
          // float64 with the top p <= 26 planes: the inverse transform on
          // the coefficients' high 32-bit words (see decode_hi32)
          const uint32_t m = plane_mask<uint32_t>(32, p), off = m & 0xAAAAAAAAu;
          int32_t h[64];
#pragma unroll
          for (int k = 0; k < 64; ++k) h[kOrder.at[k]] = (int32_t)((high_word(v[k]) & m) - off);
          inverse_words(h);
#pragma unroll
          for (int l = 0; l < 64; ++l) row[l] = (T)__builtin_ldexp((double)h[l], emax - 30);
        } else {
          const U m = plane_mask<U>(P, p), off = m & FT<T>::NB;
          S q[64];
#pragma unroll
          for (int k = 0; k < 64; ++k) q[kOrder.at[k]] = (S)((v[k] & m) - off);
          inverse_words(q);
          // (float32 through double, the general way: a faster one where the
          // exponent allows it would cost registers here, not time)
#pragma unroll
          for (int l = 0; l < 64; ++l) row[l] = dequantize(q[l], emax);
        }
      } else {
        // bin 2 tau 2^-delta; the block's integers, its code width, its size
        const double inv0 = 1.0 / (2.0 * tau);
        {
          S q[64];
          if (pq_quantize<T>(r, inv0, delta, q) && delta <= kPqMaxDelta && active && maxabs != 0) {
            bool pred;
            cb = pq_bits<T>(delta, pq_width(q, pred));
            feasible = cb <= (uint32_t)FT<T>::RAW_BITS;
          }
        }
        // each integer is formed again and turned into its value, so that no
        // array of integers is held beside the residual
        const double inv = __builtin_ldexp(inv0, delta), h = __builtin_ldexp(2.0 * tau, -delta);
#pragma unroll
        for (int l = 0; l < 64; ++l) {
          const S qq = (S)__builtin_rint((double)opaque(r[l]) * inv);
          row[l] = (T)((double)qq * h);
        }
      }
      const double ea = check_rows<T, kFull>(X, xt, vmask, scale, row);
      const bool accept = feasible && ea <= tau && ea <= eb;
      if (accept) {
        mode = MODE_CODED;
        nbits = cb;
        err = ea;
      } else if (pending && maxabs != 0 && !(eb <= tau)) {
        if (feasible) ++delta;
        else mode = MODE_RAW;
      }
      pending = pending && !accept && feasible && maxabs != 0 && !(eb <= tau);
    } while (__any(pending));
    if (active) {
      if (mode == MODE_EMPTY) err = eb;
      if (mode == MODE_RAW) nbits = (uint32_t)FT<T>::RAW_BITS;
      if (mode == MODE_RAW) {  // x~_i reproduces x up to the rounding of the residual
        const XLds<T> X{s_x, opaque(lane)};
        double ea = 0.0;
#pragma unroll
        for (int l = 0; l < 64; ++l) {
          const T xl = X.at(l);
          row[l] = xt[l] + (xl - xt[l]);
          ea = nmax(ea, masked_abs(vmask, l, (double)xl - (double)row[l]));
        }
        err = ea;
        miss = !(ea <= tau && ea <= eb);
      } else if (mode == MODE_EMPTY) {
        miss = !(eb <= tau);
      }
    } else {
      err = 0.0;
      nbits = 0;
    }
    eb = err;  // the next component's error before coding: same samples, same order

    // the wave's statistics of this component, one record (no atomics)
    bool over = false;
    uint32_t start, tot;
    uint32_t cw0, cw1, cw2, cw3;
    const uint32_t incl = row_incl_scan(nbits);  // offsets of the blocks inside their chunk
    const uint32_t off = incl - nbits;
    {
      cw0 = ((uint32_t)__builtin_amdgcn_readlane((int)incl, 15) + 31u) / 32u;
      cw1 = ((uint32_t)__builtin_amdgcn_readlane((int)incl, 31) + 31u) / 32u;
      cw2 = ((uint32_t)__builtin_amdgcn_readlane((int)incl, 47) + 31u) / 32u;
      cw3 = ((uint32_t)__builtin_amdgcn_readlane((int)incl, 63) + 31u) / 32u;
      tot = cw0 + cw1 + cw2 + cw3;
      // the span goes behind the earlier ones in the slot; where it does not
      // fit, a later launch goes on from here
      const uint32_t need = (tot + 3u) & ~3u;
      start = cur;
      over = cur + need > limit;
      cur += need;
      const uint32_t ne = (uint32_t)__popcll(__ballot(active && mode == MODE_EMPTY));
      const uint32_t nr = (uint32_t)__popcll(__ballot(mode == MODE_RAW));
      const uint32_t ns = (uint32_t)__popcll(__ballot(mode == MODE_CODED && delta > 0));
      const uint32_t nm = (uint32_t)__popcll(__ballot(miss));
      const uint32_t rf = kCodec == 0 && mode == MODE_CODED ? route_flags<T>(p, emax) : 0u;
      const bool not16 = __any(rf & kNotHi16), not32 = sizeof(T) == 8 && __any(rf & kNotHi32);
      const bool bad = __any(active && nonfinite);
      const double wm = wave_max_pos(err);
      if (lane == 0) {
        const uint64_t at = (uint64_t)i * job_waves(f) + wave;
        to_global(f.wave_linf)[at] = wm;
        to_global(f.wave_stat)[at] = ne | (nr << 7) | (ns << 14) | (nm << 21) | (not16 ? kStatNotHi16 : 0u) |
                          (not32 ? kStatNotHi32 : 0u) |
                          (bad ? kStatNonfinite : 0u) | (over ? kStatOver : 0u);
        if (ncomp > 1) to_global(f.wave_start)[at] = start;
      }
      const uint64_t chunk = (uint64_t)wave * 4 + lane;
      if (lane < 4 && chunk < g.nchunks)
        to_global(f.chunk_words)[(uint64_t)i * g.nchunks + chunk] =
            over ? 0u : lane == 0 ? cw0 : lane == 1 ? cw1 : lane == 2 ? cw2 : cw3;
    }
    if (over) {  // uniform: no data for this component and the later ones
      for (int j = i + 1; j < comp1; ++j) {
        const uint64_t at = (uint64_t)j * job_waves(f) + wave, chunk = (uint64_t)wave * 4 + lane;
        if (lane == 0) {
          to_global(f.wave_linf)[at] = 0.0;
          to_global(f.wave_stat)[at] = kStatOver;
          to_global(f.wave_start)[at] = 0;
        }
        if (lane < 4 && chunk < g.nchunks) to_global(f.chunk_words)[(uint64_t)j * g.nchunks + chunk] = 0;
      }
      return;
    }
    if (active) to_global((uint32_t*)f.region)[(uint64_t)i * f.aux_stride + blk] = off;

    // emit the four chunk bitstreams, adjacent in the wave's span, through
    // the LDS window.  The plane words held from the cost serve a span of one
    // window; otherwise the residual and its coefficients are formed again
    // while x~_{i-1} is in its registers.
    const gptr<uint32_t> dst = slot + start;
    const uint32_t c = lane >> 4;
    const uint32_t base = c == 0 ? 0u : c == 1 ? cw0 : c == 2 ? cw0 + cw1 : cw0 + cw1 + cw2;
    const int32_t bit0 = (int32_t)(32u * base + off);
    auto clear = [&](uint32_t pieces) {
      __syncthreads();
      for (uint32_t k = lane; k < pieces + 1u; k += 64)
        reinterpret_cast<uint4*>(s_emit)[k] = make_uint4(0u, 0u, 0u, 0u);
      __syncthreads();
    };
    auto copy_out = [&](uint32_t w0, uint32_t pieces) {  // 16-byte pieces
      __syncthreads();
      for (uint32_t k = lane; k < pieces; k += 64) {
        const uint4 q = reinterpret_cast<const uint4*>(s_emit)[k];
        __builtin_nontemporal_store(nt_u4{q.x, q.y, q.z, q.w}, (gptr<nt_u4>)(dst + w0) + k);
      }
    };
    // a coded block's header of codec 0: nonempty, coded; the escalation count in unary; the exponent
    auto emit_head = [&](auto& w) {
      if (__all(delta == 0)) {
        w.put32(1u | ((uint32_t)(emax + FT<T>::BIAS) << 3), 3u + (uint32_t)EB);
      } else {
        w.put32(1u, 2);
        w.put(delta >= 64 ? ~0ull : (1ull << delta) - 1ull, (uint32_t)delta);
        w.put32((uint32_t)(emax + FT<T>::BIAS) << 1, 1u + (uint32_t)EB);
      }
    };
    // x~_i: before the emission in float32's codec 0, which then need not hold
    // row across it (2.6 -> 2.0 ms per 512^3 and 8 components); the others have
    // the registers, and moving early costs them (256^3 float64 0.57 -> 0.65 ms)
    constexpr bool kEarly = sizeof(T) == 4 && kCodec == 0;
    auto commit = [&]() {
      if constexpr (kEarly) {
#pragma unroll
        for (int l = 0; l < 64; ++l) xt[l] = mode != MODE_EMPTY ? row[l] : xt[l];
      }
    };
    // (an empty block is one 0 bit)
    if (kCodec == 0 && tot <= NW && !__any(mode == MODE_RAW) &&
        aw != 0) {
      commit();
      clear((tot + 3u) / 4u);
      if (mode == MODE_CODED) {
        BitOr<false> w{s_emit, NW, bit0};
        emit_head(w);
        uint32_t n = 0;
        w.pos += zl;
        if (aw == 4) group_emit<4>(w, A, zl < P - 4 ? zl : P - 4, zl, p, n, unsq);
        else group_emit<8>(w, A, zl < P - 8 ? zl : P - 8, zl, p, n, unsq);
      }
      copy_out(0, (tot + 3u) / 4u);
    } else {
      T r[64];
      U v[kCodec == 0 ? 64 : 1];
      residual(r);
      if constexpr (kCodec == 0) {
        if (mode == MODE_CODED) {
          forward_coeffs_biased<T>(r, emax, v);
        } else {
#pragma unroll
          for (int l = 0; l < 64; ++l) v[l] = raw_bits_lo(r[l]);
        }
      }
      commit();
#pragma unroll 1
      for (uint32_t w0 = 0; w0 < tot; w0 += NW) {
        const uint32_t pieces = ((tot - w0 < NW ? tot - w0 : NW) + 3u) / 4u;
        clear(pieces);
        BitOr<true> w{s_emit, NW, bit0 - (int32_t)(32u * w0)};
        if (w.pos < (int32_t)(32u * NW) && w.pos + (int32_t)nbits > 0) {
          if (mode == MODE_CODED) {
            if constexpr (kCodec == 0) {
              emit_head(w);
              planes_emit(w, v, zl, p, unsq);
            } else {
              // the accepted candidate's integers again (the same arithmetic)
              S q[64];
              (void)pq_quantize<T>(r, 1.0 / (2.0 * tau), delta, q);
              bool pred;
              const uint32_t width = pq_width(q, pred);
              w.put32(1u, 2);
              w.put(delta >= 64 ? ~0ull : (1ull << delta) - 1ull, (uint32_t)delta);
              w.put32((pred ? 2u : 0u) | (width << 2), 8);
              if (pred) lorenzo_fwd(q);
#pragma unroll
              for (int l = 0; l < 64; ++l) {
                if constexpr (sizeof(U) == 4) w.put32(zigzag(q[l]), width);
                else w.put(zigzag(q[l]), width);
              }
            }
          } else if (mode == MODE_RAW) {
            // the residual's bits, four samples at a time and rotated once
            // round in all, so that the loop indexes registers by constants
            w.put32(3u, 2);
#pragma unroll 1
            for (int k = 0; k < 16; ++k) {
              U h[4];
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                if constexpr (kCodec == 0) h[t] = v[t];
                else h[t] = raw_bits_lo(r[t]);
                if constexpr (sizeof(U) == 4) w.put32(h[t], 32);
                else w.put(h[t], 64);
              }
#pragma unroll
              for (int l = 0; l < 64; ++l) {
                if constexpr (kCodec == 0) v[l] = l < 60 ? v[l + 4] : h[l - 60];
                else r[l] = l < 60 ? r[l + 4] : from_raw(h[l - 60], (T)0);
              }
            }
          }
        }
        copy_out(w0, pieces);
      }
    }
    if constexpr (!kEarly) {
      if (mode != MODE_EMPTY) {
#pragma unroll
        for (int l = 0; l < 64; ++l) xt[l] = row[l];
      }
    }
  }
  if (comp1 < ncomp && active) {  // for the next component's launch
#pragma unroll
    for (int k = 0; k < 16; ++k) tile_store_row(tile, lane, k, xt + 4 * k);
  }
}

typedef __attribute__((address_space(4))) const FieldJob CFieldJob;

// The job of a single field comes as the kernel's argument, read (as a batch's
// table is) through the constant address space, so that its values are loaded
// where they are needed instead of being held across the wave's work.
// (codec 1's residual, integers and x~ take 380 registers in float32: two waves
// per SIMD spill 130 of them and are no faster, 0.38 ms per 256^3 and 8
// components either way.  In float64 they spill 235 of 512, 900 bytes of scratch
// per lane; a compression of 256^3 takes 1.03 ms all the same, 1.69 with a
// launch per component, which spilled none.  Codec 0 spills 64 registers, with
// edge paths 96, in float64 146 and 232, in batches 72 and 245.)
template <class T, bool kFull, int kCodec>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && kCodec == 0 ? 2 : 1))) void k_encode(
    FieldJob) {
  __shared__ __align__(16) T s_x[64 * 64];
  __shared__ __align__(16) uint32_t s_emit[emit_words<T>() + kEmitPad];
  __shared__ uint16_t s_unsq[256];
  unsqueeze_table(s_unsq);
  const CFieldJob& f = *(const CFieldJob*)__builtin_amdgcn_kernarg_segment_ptr();
  encode_wave<T, kFull, kCodec>(f, blockIdx.x, s_x, s_emit, s_unsq);
}

// Batches: the waves of many fields, listed as items; each workgroup walks the
// list with a static stride, so a field's bytes depend only on its own blocks,
// never on the schedule.
template <class T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 2 : 1))) void k_encode_batch(BatchArgs b) {
  __shared__ __align__(16) T s_x[64 * 64];
  __shared__ __align__(16) uint32_t s_emit[emit_words<T>() + kEmitPad];
  __shared__ uint16_t s_unsq[256];
  unsqueeze_table(s_unsq);
  const CFieldJob* const fields = (const CFieldJob*)b.fields;
  for (uint32_t it = blockIdx.x; it < b.nitems; it += gridDim.x) {
    const Item w = b.items[it];
    const CFieldJob& f = fields[w.field];
    encode_wave<T, false, 0>(f, w.index, s_x, s_emit, s_unsq);
    __syncthreads();  // the next item reuses the LDS
  }
}

template <class T> hipError_t launch_encode(const FieldJob& f, hipStream_t s) {
  // every block full and every row aligned: the kernel without edge paths
  const bool full = f.g.nx % 4 == 0 && f.g.ny % 4 == 0 && f.g.nz % 4 == 0 && f.g.rows_aligned;
  const dim3 grid(job_waves(f)), wg(64);
  if (f.codec == 0) {
    if (full) hipLaunchKernelGGL((k_encode<T, true, 0>), grid, wg, 0, s, f);
    else hipLaunchKernelGGL((k_encode<T, false, 0>), grid, wg, 0, s, f);
  } else {
    if (full) hipLaunchKernelGGL((k_encode<T, true, 1>), grid, wg, 0, s, f);
    else hipLaunchKernelGGL((k_encode<T, false, 1>), grid, wg, 0, s, f);
  }
  return hipGetLastError();
}
template <class T> hipError_t launch_encode_batch(const BatchArgs& a, uint32_t grid, hipStream_t s) {
  if (a.nitems == 0) return hipSuccess;
  hipLaunchKernelGGL(k_encode_batch<T>, dim3(grid), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace pmc
