// decode_device.hpp -- the retrieval kernels (Alg. 2) and their launchers,
// instantiated per element type by decode_f32.hip and decode_f64.hip.
//
//  k_decode          components [k0, k1) of a field added left to right into
//                    x~; one lane per block, located by the chunk index plus a
//                    per-block bit offset written by the encoder
//  k_decode_box      the blocks meeting a box, written as the box alone
//  k_decode_split    either, with one wave per component (fields and boxes of
//                    few waves)
//  k_decode_queries  many retrievals in one launch
//  k_decode_tiles    x~ for the encoder to go on from
#pragma once
#include "block_device.hpp"

namespace pmc {

// ---------------------------------------------------------------------------
// Alg. 2 over one block per lane: x~ = (((x~_in or +0) + x_1) + x_2) ... in
// the field precision; the block's bits start at its chunk's word offset plus
// the block's bit offset from the per-block index
//
// routes of the inverse transform: kRouteAuto picks per wave (float64: the
// high-word route where it applies); kRouteFull the plain route; kRouteHi16
// the float32 high-half route, for components whose every block has p <= 10
// and hi16_exact(emax) (the caller guarantees it)
// float64 fields whose blocks qualify decode in 256 registers, two waves per
// SIMD: kRouteHi16 for the residual components (p <= 10 and hi16_exact(emax)),
// kRouteFirst for a store's first one (no raw blocks, p <= 26 and emax >= -992).
// x~ takes 128 of the registers, so with every route in one loop only one wave
// fits and its LDS latency stands open: 256^3, k = 8, 201 us, now 131.
constexpr int kRouteAuto = 0, kRouteFull = 1, kRouteHi16 = 2, kRouteFirst = 3;

// a coded block's header after its first two bits, and its leading empty
// planes; false on a malformed one
template <class T, class R>
__device__ __forceinline__ bool coded_head(R& r, uint32_t h, int minexp, int& emax, int& p, int& zlead) {
  constexpr int P = FT<T>::P;
  constexpr int EB = FT<T>::EBITS;
  // unary escalation count, then the biased block exponent
  int delta = (int)__builtin_ctz(~(h >> 2) | 0x40000000u);
  if (3 + delta + EB <= 32) {
    emax = (int)((h >> (3 + delta)) & ((1u << EB) - 1u)) - FT<T>::BIAS;
    r.skip((uint32_t)(3 + delta + EB));
  } else {
    r.skip(2);
    delta = 0;
#pragma unroll 1
    while (r.get(1)) {  // (rare: a long escalation; kept as a loop)
      if (++delta > P) return false;
    }
    emax = (int)r.get((uint32_t)EB) - FT<T>::BIAS;
  }
  p = emax - minexp + kGuard;
  p = (p < 0 ? 0 : (p > P ? P : p)) + delta;
  if (emax < 2 - FT<T>::BIAS || p < 1 || p > P) return false;
  // Leading empty planes: until a coefficient is significant, a plane
  // without a new one is a single 0 (its negative group test), so the first
  // zeros of the block's plane data are that many empty planes, skipped at once.
  const int z0 = (int)__builtin_ctz(r.peek32() | 0x80000000u);
  zlead = z0 < p ? z0 : p;
  r.skip((uint32_t)zlead);
  return true;
}

template <class T, int kRoute = kRouteAuto, class R>
__device__ __forceinline__ bool decode_block_add(R& r, int minexp, T acc[64], const uint8_t* sq, bool rel) {
  typedef typename FT<T>::U U;
  constexpr int P = FT<T>::P;
  const uint32_t h = r.peek32();
  if (!(h & 1u)) {  // empty: x_i = 0 leaves x~ unchanged
    r.skip(1);
    return true;
  }
  if (h & 2u) {  // raw block
    r.skip(2);
#pragma unroll
    for (int l = 0; l < 64; ++l) {
      T v = from_raw((U)r.get64((uint32_t)P), (T)0);
      acc[l] = acc[l] + v;
    }
    return true;
  }
  int emax, p, zlead;
  if (!coded_head<T>(r, h, minexp, emax, p, zlead)) return false;
  if constexpr (sizeof(T) == 8 && kRoute == kRouteAuto) {
    // residual components whose coded planes all lie in the top ten bit
    // positions and keep every result normal and finite: the lifting on the words' top
    // 16 bits, two per register, from 4 or 8 slots (wave-uniform choices)
    if (rel && __all(p <= 10 && hi16_exact(emax, (T)0))) {
      const int np = p - zlead;
      v2s R2[32];
      if (__all(np <= 4)) {
        slots_hi16<4>(r, p, zlead, sq, R2);
        lift_dequant_add_hi16(R2, emax, acc);
        return true;
      }
      if (__all(np <= 8)) {
        slots_hi16<8>(r, p, zlead, sq, R2);
        lift_dequant_add_hi16(R2, emax, acc);
        return true;
      }
    }
    // every coded plane in the top 26 bit positions and every result
    // normal: the lifting on the coefficients' high words (a wave-uniform
    // choice; both routes give the same sums)
    if (__all(p <= 26 && emax >= -992)) {
      const int np = p - zlead;
      if (__all(np <= 4)) decode_hi32<4>(r, p, zlead, emax, acc, sq, rel);
      else if (__all(np <= 8)) decode_hi32<8>(r, p, zlead, emax, acc, sq, rel);
      else decode_hi32<16>(r, p, zlead, emax, acc, sq, rel);
      return true;
    }
  }
  if constexpr (kRoute == kRouteHi16) {
    // residual components (rel): the packed pairs straight from 4 or 8
    // slots, else from the 32-bit (high) words of 16
    v2s R2[32];
    const int np = p - zlead;
    if (__all(np <= 4)) {
      slots_hi16<4>(r, p, zlead, sq, R2);
    } else if (__all(np <= 8)) {
      slots_hi16<8>(r, p, zlead, sq, R2);
    } else {
      int32_t c[64];
      if constexpr (sizeof(T) == 4) planes_slots<T, 16>(r, c, p, zlead, sq, rel);
      else coeffs_hi32<16>(r, p, zlead, c, sq, rel);
      pack_hi16(c, R2);
    }
    lift_dequant_add_hi16(R2, emax, acc);
    return true;
  }
  if constexpr (kRoute != kRouteHi16) {
    typename FT<T>::S c[64], q[64];
    planes_read<T>(r, c, p, zlead, sq, rel);
    inverse_zy_ints<T>(c, q);
    inverse_x<T>(q);
    dequant_add(q, emax, acc);
  }
  return true;
}

// a float64 store's first component on kRouteFirst: the block's words h and
// exponent (zeros for an empty block), for the caller to turn into x~_1
// outside the divergent part: x~ is not live while this decodes
template <class R>
__device__ __forceinline__ bool decode_first(R& r, int minexp, int32_t h[64], int& emax, const uint8_t* sq) {
  const uint32_t hd = r.peek32();
  if (!(hd & 1u)) {
    r.skip(1);
    return true;
  }
  int p, zlead;
  if ((hd & 2u) || !coded_head<double>(r, hd, minexp, emax, p, zlead)) return false;
  const int np = p - zlead;
  if (__all(np <= 8)) words_hi32<8>(r, p, zlead, h, sq, false);
  else words_hi32<16>(r, p, zlead, h, sq, false);
  return true;
}

// words of one wave's four chunks staged in LDS per component (13.3 KB, so
// that 12 one-wave workgroups fit a CU's LDS); spans larger than this use
// the global-memory reader (the host picks the variant from the largest span
// of the streams it decodes)
constexpr uint32_t kStageWords = 3326;
// The staging buffer is double-buffered while spans are small: two halves of
// kHalfWords data words (64-word multiples, since a copy writes whole 64-word
// rows) plus 3 spare words each for the reader's look-ahead.  The next
// component's words load into one half while the wave decodes from the other.
// A component whose span exceeds a half uses the whole buffer and is staged
// without overlap.
constexpr uint32_t kHalfWords = 1600;
constexpr uint32_t kHalf1 = kHalfWords + 3;  // word offset of the second half
static_assert(kHalf1 + kHalfWords + 3 <= kStageWords + 3, "halves fit the buffer");

// the wave's span of payload words of one component: its chunks [4w, 4w + 4)
// are consecutive in the payload
struct Span {
  uint64_t s0, s1;
  bool ok;
};
__device__ __forceinline__ Span wave_span(const uint32_t* index, uint64_t nchunks, uint64_t words, uint64_t w,
                                          uint32_t cap = kStageWords) {
  const uint64_t c0 = w * 4, c1 = min<uint64_t>(c0 + 4, nchunks);
  Span sp;
  sp.s0 = index[c0];
  sp.s1 = c1 < nchunks ? (uint64_t)index[c1] : words;
  sp.ok = sp.s0 <= sp.s1 && sp.s1 <= words && sp.s1 - sp.s0 <= cap;
  return sp;
}
// issue (not wait for) the copy of a span into the staging words at `base`
__device__ __forceinline__ void stage_span(const uint32_t* payload, const Span& sp, uint32_t* stage, uint32_t base) {
  const uint32_t lane = threadIdx.x;
  const uint32_t span = (uint32_t)(sp.s1 - sp.s0);
  for (uint32_t k = 0; k < span; k += 64) {
    const uint32_t j = k + lane < span ? k + lane : span - 1;
    __builtin_amdgcn_global_load_lds((gmem_void_t*)(payload + sp.s0 + j), (lds_void_t*)(stage + base + k), 4, 0, 0);
  }
}

// one block of one component, codec 0 (minexp) or codec 1 (step = 2 tau)
template <class T, int kCodec, int kRoute = kRouteAuto, class R>
__device__ __forceinline__ bool decode_block_codec(R& r, int minexp, double step, T acc[64], const uint8_t* sq,
                                                   bool rel) {
  if constexpr (kCodec == 0) return decode_block_add<T, kRoute>(r, minexp, acc, sq, rel);
  else return pq_decode_add<T>(r, step, acc);
}

// decode the wave's 64 blocks [64 w, 64 w + 64) of a field: x~ = in (or +0)
// plus components [0, ncomp) of the given streams, left to right.  Every lane
// runs the component loop (the staging copies are shared); false on a
// malformed stream.  kFull: every block of the field is full and rows are
// aligned (all dimensions multiples of 4): no per-lane edge paths.  kTile: in
// and out are the encoder's tiles.
template <class T, bool kStaged, bool kBox = false, bool kFull = false, int kCodec = 0, bool kHiRes = false, bool kTile = false>
__device__ __forceinline__ bool decode_wave(const Geo& g, const uint8_t* const* s, const uint32_t* const* aux,
                                            const uint64_t* words, const int* minexp, const double* step, int ncomp,
                                            uint32_t relmask, const T* in, T* out, uint64_t w, const uint8_t* sq,
                                            uint32_t* stage, const BoxArgs* box = nullptr, T* out2 = nullptr) {
  const uint32_t lane = threadIdx.x;
  const uint64_t blk = w * 64 + lane;
  bool active = blk < g.nblocks;
  BlockPos bp = block_pos(g, active ? blk : 0);
  if constexpr (kFull) {
    bp.vx = 4;
    bp.vy = 4;
    bp.vz = 4;
  }
  if constexpr (kBox) {  // only this row's blocks in the box are decoded (each by
                         // one workgroup); the wave still stages its chunks,
                         // whose bit offsets locate every block
    active = active && blk >= box->row_first && blk <= box->row_last;
  }
  const uint64_t chunk = blk / kChunkBlocks;
  T acc[64];
  constexpr bool kHi64 = kHiRes && sizeof(T) == 8;  // (then in is null where component 0 is decoded)
  int32_t h0[kHi64 ? 64 : 1];
  int emax0 = 0;
  if constexpr (kHi64) {
#pragma unroll
    for (int l = 0; l < 64; ++l) h0[l] = 0;
  }
  if (in && active) {
    if constexpr (kBox) load_box(in, *box, bp, acc);
    else if constexpr (kTile) tile_load<T>(in, w, lane, acc);
    else if constexpr (kFull) load_rows<T, 16>(in, g, opaque_pos(bp), 0, true, acc);
    else load_block(in, g, opaque_pos(bp), acc);
  } else {
#pragma unroll
    for (int l = 0; l < 64; ++l) acc[l] = (T)0;
  }
  bool ok = true;
  if constexpr (kStaged) {
    // component i: its span, where it sits in LDS, and this lane's chunk range
    // and bit offset (loaded together with the span's words)
    Span cur{0, 0, false};
    uint32_t cur_base = 0, cur_cap = kStageWords;
    uint32_t start = 0, stop = 0, off = 0;  // word offsets (a payload has < 2^32 words) and bit offset
    if (ncomp > 0) {
      const uint32_t* index = reinterpret_cast<const uint32_t*>(s[0] + kHeaderBytes);
      cur = wave_span(index, g.nchunks, words[0], w);
      cur_cap = cur.s1 - cur.s0 <= kHalfWords ? kHalfWords : kStageWords;
      if (cur.ok) stage_span(index + g.nchunks, cur, stage, 0);
      if (active) {
        start = index[chunk];
        stop = chunk + 1 < g.nchunks ? index[chunk + 1] : (uint32_t)min<uint64_t>(words[0], 0xFFFFFFFFull);
        off = aux[0][blk];
      }
    }
    auto component = [&](int i, auto route) {
        __builtin_amdgcn_s_waitcnt(0);  // component i's words and lane values
        __syncthreads();
        // the next component: into the other half while this one decodes, when
        // both fit a half
        Span nxt{0, 0, false};
        uint32_t nxt_base = 0, nxt_cap = kStageWords;
        uint32_t nstart = 0, nstop = 0, noff = 0;
        bool pre = false;
        const uint32_t* nindex = nullptr;
        if (i + 1 < ncomp) {
          nindex = reinterpret_cast<const uint32_t*>(s[i + 1] + kHeaderBytes);
          nxt = wave_span(nindex, g.nchunks, words[i + 1], w);
          pre = nxt.ok && cur.ok && cur.s1 - cur.s0 <= kHalfWords && nxt.s1 - nxt.s0 <= kHalfWords;
          if (pre) {
            nxt_base = cur_base == 0 ? kHalf1 : 0;
            nxt_cap = kHalfWords;
            stage_span(nindex + g.nchunks, nxt, stage, nxt_base);
            if (active) {
              nstart = nindex[chunk];
              nstop = chunk + 1 < g.nchunks ? nindex[chunk + 1] : (uint32_t)min<uint64_t>(words[i + 1], 0xFFFFFFFFull);
              noff = aux[i + 1][blk];
            }
          }
        }
        if (active && ok) {
          if (!cur.ok || words[i] > 0xFFFFFFFFull || start > stop || stop > words[i] ||
              off >= (uint64_t)(stop - start) * 32 || start < cur.s0 || stop > cur.s1) {
            ok = false;
          } else {
            const uint32_t s0 = (uint32_t)cur.s0;
            LBits r;
            r.init(stage + cur_base, start - s0 + (off >> 5), stop - s0, cur_cap);
            r.skip((uint32_t)(off & 31));
            if constexpr (kHi64 && decltype(route)::value == kRouteFirst)
              ok = decode_first(r, minexp[i], h0, emax0, sq) && !r.bad();
            else
              ok = decode_block_codec<T, kCodec, decltype(route)::value>(r, minexp[i], step[i], acc, sq,
                                                                          (relmask >> i) & 1u) && !r.bad();
          }
        }
        if (i + 1 < ncomp && !pre) {  // staged after this component, into the whole buffer's first half or all of it
          __syncthreads();  // every lane is done with this component's words
          nxt_base = 0;
          nxt_cap = nxt.s1 - nxt.s0 <= kHalfWords ? kHalfWords : kStageWords;
          if (nxt.ok) stage_span(nindex + g.nchunks, nxt, stage, 0);
          if (active) {
            nstart = nindex[chunk];
            nstop = chunk + 1 < g.nchunks ? nindex[chunk + 1] : (uint32_t)min<uint64_t>(words[i + 1], 0xFFFFFFFFull);
            noff = aux[i + 1][blk];
          }
        }
        cur = nxt;
        cur_base = nxt_base;
        cur_cap = nxt_cap;
        start = nstart;
        stop = nstop;
        off = noff;
    };
    if constexpr (kHiRes) {
      // the store's first component (if decoded here) on the full route,
      // the residual ones on the high-half route only
      int i = 0;
      if (ncomp > 0 && !(relmask & 1u)) {
        if constexpr (kHi64) {
          component(0, std::integral_constant<int, kRouteFirst>{});
#pragma unroll
          for (int l = 0; l < 64; ++l) acc[l] = __builtin_ldexp((double)h0[l], emax0 - 30);  // (+0) + x_1
        } else {
          component(0, std::integral_constant<int, kRouteFull>{});
        }
        i = 1;
      }
      for (; i < ncomp; ++i) component(i, std::integral_constant<int, kRouteHi16>{});
    } else {
      for (int i = 0; i < ncomp; ++i) component(i, std::integral_constant<int, kRouteAuto>{});
    }
  } else {
    for (int i = 0; i < ncomp; ++i) {
      if (!active || !ok) continue;
      const uint32_t* index = reinterpret_cast<const uint32_t*>(s[i] + kHeaderBytes);
      const uint32_t* payload = index + g.nchunks;
      const uint64_t start = index[chunk];
      const uint64_t stop = chunk + 1 < g.nchunks ? (uint64_t)index[chunk + 1] : words[i];
      const uint64_t off = aux[i][blk];
      if (start > stop || stop > words[i] || stop > 0xFFFFFFFFull || off >= (stop - start) * 32) {
        ok = false;
        continue;
      }
      GBits r;
      r.init(payload, (uint32_t)(start + (off >> 5)), (uint32_t)stop);
      r.skip((uint32_t)(off & 31));
      ok = decode_block_codec<T, kCodec>(r, minexp[i], step[i], acc, sq, (relmask >> i) & 1u) && !r.bad();
    }
  }
  // a block whose stream did not parse is written as quiet NaNs, so the
  // output never keeps stale memory (the status word reports it as well)
  if (active && !ok) {
#pragma unroll
    for (int l = 0; l < 64; ++l) acc[l] = (T)__builtin_nan("");
  }
  // the block position is recomputed here rather than kept in registers
  if (active) {
    if constexpr (kBox) {
      store_box(out, *box, block_pos(g, opaque(w) * 64 + lane), acc);
    } else if constexpr (kTile) {
      tile_store<T>(out, w, lane, acc);
    } else if constexpr (kFull) {
      const BlockPos bo = block_pos(g, opaque(w) * 64 + lane);
#pragma unroll
      for (int r = 0; r < 16; ++r) store_row(out, g, bo, r, acc + 4 * r, true);
    } else {
      const BlockPos bo = block_pos(g, opaque(w) * 64 + lane);
      store_block(out, g, bo, acc);
      if (out2) store_block(out2, g, bo, acc);
    }
  }
  return ok || !active;
}

// kHiRes: the launch's residual components decode on the high-half route alone
// and, in float64, its first component on kRouteFirst (every block of them
// qualifies: the encoder and the index rebuild leave flags)
template <class T, bool kStaged, bool kFull, int kCodec, bool kHiRes = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : kHiRes ? 2 : 1))) void k_decode(
    DecArgs<T> a) {
  __shared__ uint8_t s_squeeze[256];
  __shared__ uint32_t s_stage[kStaged ? kStageWords + 3 : 1];
  squeeze_table(s_squeeze);
  if (!decode_wave<T, kStaged, false, kFull, kCodec, kHiRes>(a.g, a.s, a.aux, a.words, a.minexp, a.step, a.ncomp, a.relmask,
                                                     a.in, a.out, blockIdx.x, s_squeeze, s_stage))
    atomicOr(a.status, 1u);
}

// x~ as the encoder takes it up (a.in and a.out hold one tile per wave), from
// components in place; once per launch of the encoder after the first, so the
// plain reader and routes do
template <class T, int kCodec>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : 1))) void k_decode_tiles(DecArgs<T> a) {
  __shared__ uint8_t s_squeeze[256];
  squeeze_table(s_squeeze);
  if (!decode_wave<T, false, false, false, kCodec, false, true>(a.g, a.s, a.aux, a.words, a.minexp, a.step, a.ncomp,
                                                                a.relmask, a.in, a.out, blockIdx.x, s_squeeze, nullptr))
    atomicOr(a.status, 1u);
}

// region retrieval: workgroup (row, i) decodes the i-th wave of the box's
// block row `row` (rows in y-then-z order); waves past the row's last block
// exit.  a.in / a.out are box arrays (a.in: the box after earlier components).
// A wave whose blocks span several box rows (narrow fields) is staged once
// per row, and each row's workgroup decodes only that row's blocks.
template <class T, bool kStaged, int kCodec, bool kHiRes = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : kHiRes ? 2 : 1))) void k_decode_box(
    DecArgs<T> a, BoxArgs b) {
  __shared__ uint8_t s_squeeze[256];
  __shared__ uint32_t s_stage[kStaged ? kStageWords + 3 : 1];
  const uint32_t row = blockIdx.x / b.waves_per_row, i = blockIdx.x % b.waves_per_row;
  const uint64_t nry = b.bhi[1] - b.blo[1];
  const uint64_t by = b.blo[1] + row % nry, bz = b.blo[2] + row / nry;
  b.row_first = (bz * a.g.nby + by) * a.g.nbx + b.blo[0];
  b.row_last = (bz * a.g.nby + by) * a.g.nbx + b.bhi[0] - 1;
  const uint64_t w = b.row_first / 64 + i;
  if (w > b.row_last / 64) return;  // uniform over the workgroup
  squeeze_table(s_squeeze);
  if (!decode_wave<T, kStaged, true, false, kCodec, kHiRes>(a.g, a.s, a.aux, a.words, a.minexp, a.step, a.ncomp, a.relmask,
                                                    a.in, a.out, w, s_squeeze, s_stage, &b))
    atomicOr(a.status, 1u);
}

// The same sums with one wave per component (2 to 8 of them in a workgroup).
// A wave decodes one block per lane and its time is the latency of that serial
// chain, times the number of components when one wave decodes them all; where
// the blocks alone leave the SIMDs idle, the components, which are independent
// until they are added, fill them.  Each wave decodes its component onto -0
// (the neutral element of the sum: also an empty block's), the first one onto
// x~_in or +0, and the workgroup adds the partial results left to right
// through LDS, a few of a block's 16 rows at a time, in the memory the words
// were staged in.  64^3 float32, 8 components (64 waves): 44.9 us, now 17.4; a
// 64^3 box of a 512^3 field 66, now 31.
// (float32 asks for three waves per SIMD, 168 registers, as split_plan counts:
// the box on the high-half routes had come out at 169 and two)
template <class T, bool kHiRes> constexpr int split_most() { return sizeof(T) == 4 || kHiRes ? kMaxSplit : kMaxSplit64; }
template <class T, bool kBox, int kCodec, bool kHiRes>
__global__ __launch_bounds__((64 * split_most<T, kHiRes>()))
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : split_most<T, kHiRes>() / 4))) void k_decode_split(
    DecArgs<T> a, SplitArgs sp, BoxArgs b) {
  extern __shared__ __attribute__((aligned(16))) uint32_t s_dyn[];  // sp.lds_bytes
  __shared__ uint8_t s_squeeze[256];
  __shared__ uint64_t s_ok[kMaxSplit];
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t i = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Geo& g = a.g;
  uint64_t w = blockIdx.x;
  if constexpr (kBox) {
    const uint32_t row = blockIdx.x / b.waves_per_row, k = blockIdx.x % b.waves_per_row;
    const uint64_t nry = b.bhi[1] - b.blo[1];
    const uint64_t by = b.blo[1] + row % nry, bz = b.blo[2] + row / nry;
    b.row_first = (bz * g.nby + by) * g.nbx + b.blo[0];
    b.row_last = (bz * g.nby + by) * g.nbx + b.bhi[0] - 1;
    w = b.row_first / 64 + k;
    if (w > b.row_last / 64) return;  // uniform over the workgroup
  }
  const uint64_t blk = w * 64 + lane;
  bool active = blk < g.nblocks;
  if constexpr (kBox) active = active && blk >= b.row_first && blk <= b.row_last;
  const uint64_t chunk = blk / kChunkBlocks;
  const uint32_t* index = reinterpret_cast<const uint32_t*>(a.s[i] + kHeaderBytes);
  const uint64_t words = a.words[i];
  const Span cur = wave_span(index, g.nchunks, words, w, sp.cap[i]);
  uint32_t* stage = s_dyn + sp.base[i];
  if (cur.ok) {
    const uint32_t span = (uint32_t)(cur.s1 - cur.s0);
    const uint32_t* payload = index + g.nchunks + cur.s0;
    for (uint32_t k = 0; k < span; k += 64) {
      const uint32_t j = k + lane < span ? k + lane : span - 1;
      __builtin_amdgcn_global_load_lds((gmem_void_t*)(payload + j), (lds_void_t*)(stage + k), 4, 0, 0);
    }
  }
  uint32_t start = 0, stop = 0, off = 0;
  if (active) {
    start = index[chunk];
    stop = chunk + 1 < g.nchunks ? index[chunk + 1] : (uint32_t)min<uint64_t>(words, 0xFFFFFFFFull);
    off = a.aux[i][blk];
  }
  T acc[64];
  if (i == 0 && a.in && active) {
    const BlockPos bp = block_pos(g, blk);
    if constexpr (kBox) load_box(a.in, b, bp, acc);
    else load_block(a.in, g, bp, acc);
  } else {
    const T zero = i == 0 ? (T)0 : -(T)0;
#pragma unroll
    for (int l = 0; l < 64; ++l) acc[l] = zero;
  }
  __builtin_amdgcn_s_waitcnt(0);  // the wave's words, and its lanes' values
  squeeze_table(s_squeeze);
  bool ok = true;
  if (active) {
    if (!cur.ok || words > 0xFFFFFFFFull || start > stop || stop > words ||
        off >= (uint64_t)(stop - start) * 32 || start < cur.s0 || stop > cur.s1)
      ok = false;
  }
  const bool rel = (a.relmask >> i) & 1u;
  LBits r;
  if (active && ok) {
    const uint32_t s0 = (uint32_t)cur.s0;
    r.init(stage, start - s0 + (off >> 5), stop - s0, sp.cap[i]);
    r.skip((uint32_t)(off & 31));
  }
  if constexpr (kHiRes) {
    if (!rel) {  // (the launch's first component, if it is the store's)
      if constexpr (sizeof(T) == 8) {
        int32_t h0[64];
        int emax0 = 0;
#pragma unroll
        for (int l = 0; l < 64; ++l) h0[l] = 0;
        if (active && ok) ok = decode_first(r, a.minexp[i], h0, emax0, s_squeeze) && !r.bad();
#pragma unroll
        for (int l = 0; l < 64; ++l) acc[l] = __builtin_ldexp((double)h0[l], emax0 - 30);
      } else {
        if (active && ok)
          ok = decode_block_codec<T, kCodec, kRouteFull>(r, a.minexp[i], a.step[i], acc, s_squeeze, rel) && !r.bad();
      }
    } else if (active && ok) {
      ok = decode_block_codec<T, kCodec, kRouteHi16>(r, a.minexp[i], a.step[i], acc, s_squeeze, rel) && !r.bad();
    }
  } else if (active && ok) {
    ok = decode_block_codec<T, kCodec>(r, a.minexp[i], a.step[i], acc, s_squeeze, rel) && !r.bad();
  }
  const uint64_t mask = __ballot(ok);
  if (lane == 0) {
    s_ok[i] = mask;
    if (~mask) atomicOr(a.status, 1u);
  }
  // the ordered sum, 4 KB of rows per component at a time: 16-byte units, lanes adjacent
  constexpr uint32_t kUnits = sizeof(T) / 4;   // of a row
  constexpr uint32_t kPer = 16 / sizeof(T);    // values in a unit
  constexpr uint32_t kRows = 16 / sizeof(T);   // rows at a time
  typedef T unit_t __attribute__((ext_vector_type(16 / sizeof(T))));
  unit_t* ex = reinterpret_cast<unit_t*>(s_dyn);
  const uint32_t nc = (uint32_t)a.ncomp;
#pragma unroll
  for (uint32_t s = 0; s < 16; s += kRows) {
    __syncthreads();  // the words, or the rows before these, have been read
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      unit_t u;
#pragma unroll
      for (uint32_t e = 0; e < kPer; ++e) u[e] = acc[4 * s + kPer * k + e];
      ex[(i * 4 + k) * 64 + lane] = u;
    }
    __syncthreads();
    for (uint32_t rr = i; rr < kRows; rr += nc) {
      uint64_t good = ~0ull;
      T v[4];
      for (uint32_t j = 0; j < nc; ++j) {
        good &= s_ok[j];
#pragma unroll
        for (uint32_t q = 0; q < kUnits; ++q) {
          const unit_t u = ex[(j * 4 + rr * kUnits + q) * 64 + lane];
#pragma unroll
          for (uint32_t e = 0; e < kPer; ++e) v[q * kPer + e] = j == 0 ? u[e] : v[q * kPer + e] + u[e];
        }
      }
      // (a block whose stream did not parse: quiet NaNs, as in decode_wave)
      if (!((good >> lane) & 1u)) v[0] = v[1] = v[2] = v[3] = (T)__builtin_nan("");
      if (active) {
        const BlockPos bp = block_pos(g, opaque(w) * 64 + lane);
        if constexpr (kBox) store_box_row(a.out, b, bp, (int)(s + rr), v);
        else store_row(a.out, g, bp, (int)(s + rr), v);
      }
    }
  }
}

// many retrieval queries in one launch: wave w belongs to the query q with
// wave_prefix[q] <= w < wave_prefix[q + 1]
template <class T, bool kStaged, int kCodec, bool kHiRes = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : kHiRes ? 2 : 1))) void k_decode_queries(
    ServeArgs a) {
  __shared__ uint8_t s_squeeze[256];
  __shared__ uint32_t s_stage[kStaged ? kStageWords + 3 : 1];
  squeeze_table(s_squeeze);
  const uint32_t w = blockIdx.x;
  uint32_t lo = 0, hi = a.nq;  // largest q with wave_prefix[q] <= w
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (a.wave_prefix[mid] <= w) lo = mid;
    else hi = mid;
  }
  // the query table is read-only for the launch: read through the constant
  // address space, so its values can be loaded again where needed instead of
  // being held across the wave's work
  typedef __attribute__((address_space(4))) const QueryDev CQueryDev;
  const CQueryDev& q = ((const CQueryDev*)a.q)[lo];
  Geo g;
  g.nx = q.g.nx;
  g.ny = q.g.ny;
  g.nz = q.g.nz;
  g.nbx = q.g.nbx;
  g.nby = q.g.nby;
  g.nbz = q.g.nbz;
  g.nblocks = q.g.nblocks;
  g.nchunks = q.g.nchunks;
  g.rows_aligned = q.g.rows_aligned;
  g.pad = 0;
  if (!decode_wave<T, kStaged, false, false, kCodec, kHiRes>(
          g, (const uint8_t* const*)q.s, (const uint32_t* const*)q.aux, (const uint64_t*)q.words,
          (const int*)q.minexp, (const double*)q.step, q.ncomp, q.relmask, reinterpret_cast<const T*>(q.in),
          reinterpret_cast<T*>(q.out), w - a.wave_prefix[lo], s_squeeze, s_stage, nullptr,
          reinterpret_cast<T*>(q.out2)))
    atomicOr(a.status, 1u);
}

// ---------------------------------------------------------------------------
// launchers
template <class T, int kCodec>
void launch_decode_codec(const DecArgs<T>& a, uint64_t max_span, bool hires, hipStream_t s) {
  const uint64_t wgs = (a.g.nblocks + 63) / 64;
  const dim3 grid((uint32_t)wgs), wg(64);
  // every block full and every row aligned: the kernel without edge paths
  const bool full = a.g.nx % 4 == 0 && a.g.ny % 4 == 0 && a.g.nz % 4 == 0 && a.g.rows_aligned;
  if constexpr (kCodec == 0) {
    if (hires && max_span <= kStageWords) {
      if (full) hipLaunchKernelGGL((k_decode<T, true, true, kCodec, true>), grid, wg, 0, s, a);
      else hipLaunchKernelGGL((k_decode<T, true, false, kCodec, true>), grid, wg, 0, s, a);
      return;
    }
  }
  if (max_span <= kStageWords) {
    if (full) hipLaunchKernelGGL((k_decode<T, true, true, kCodec>), grid, wg, 0, s, a);
    else hipLaunchKernelGGL((k_decode<T, true, false, kCodec>), grid, wg, 0, s, a);
  } else {
    if (full) hipLaunchKernelGGL((k_decode<T, false, true, kCodec>), grid, wg, 0, s, a);
    else hipLaunchKernelGGL((k_decode<T, false, false, kCodec>), grid, wg, 0, s, a);
  }
}
template <class T, bool kBox>
hipError_t launch_split(const DecArgs<T>& a, const SplitArgs& sp, const BoxArgs& b, uint64_t wgs, int codec, bool hires,
                        hipStream_t s) {
  const dim3 grid((uint32_t)wgs), wg(64u * (uint32_t)a.ncomp);
  if (a.ncomp > (hires ? split_most<T, true>() : split_most<T, false>())) return hipErrorInvalidValue;  // (split_plan's)
  if (codec != 0) hipLaunchKernelGGL((k_decode_split<T, kBox, 1, false>), grid, wg, sp.lds_bytes, s, a, sp, b);
  else if (hires) hipLaunchKernelGGL((k_decode_split<T, kBox, 0, true>), grid, wg, sp.lds_bytes, s, a, sp, b);
  else hipLaunchKernelGGL((k_decode_split<T, kBox, 0, false>), grid, wg, sp.lds_bytes, s, a, sp, b);
  return hipGetLastError();
}
template <class T>
hipError_t launch_decode(const DecArgs<T>& a, uint64_t max_span, int codec, bool hires, const SplitArgs* split,
                         hipStream_t s) {
  if (split) return launch_split<T, false>(a, *split, BoxArgs{}, (a.g.nblocks + 63) / 64, codec, hires, s);
  if (codec == 0) launch_decode_codec<T, 0>(a, max_span, hires, s);
  else launch_decode_codec<T, 1>(a, max_span, false, s);
  return hipGetLastError();
}
template <class T>
hipError_t launch_decode_box(const DecArgs<T>& a, const BoxArgs& b, uint64_t max_span, int codec, bool hires,
                             const SplitArgs* split, hipStream_t s) {
  const uint64_t rows = (b.bhi[1] - b.blo[1]) * (b.bhi[2] - b.blo[2]);
  const uint64_t wgs = rows * b.waves_per_row;
  if (wgs == 0) return hipSuccess;
  if (split) return launch_split<T, true>(a, *split, b, wgs, codec, hires, s);
  const dim3 grid((uint32_t)wgs), wg(64);
  const bool staged = max_span <= kStageWords;
  if (codec == 0) {
    if (staged && hires) hipLaunchKernelGGL((k_decode_box<T, true, 0, true>), grid, wg, 0, s, a, b);
    else if (staged) hipLaunchKernelGGL((k_decode_box<T, true, 0>), grid, wg, 0, s, a, b);
    else hipLaunchKernelGGL((k_decode_box<T, false, 0>), grid, wg, 0, s, a, b);
  } else {
    if (staged) hipLaunchKernelGGL((k_decode_box<T, true, 1>), grid, wg, 0, s, a, b);
    else hipLaunchKernelGGL((k_decode_box<T, false, 1>), grid, wg, 0, s, a, b);
  }
  return hipGetLastError();
}
template <class T> hipError_t launch_decode_tiles(const DecArgs<T>& a, int codec, hipStream_t s) {
  const dim3 grid((uint32_t)((a.g.nblocks + 63) / 64)), wg(64);
  if (codec == 0) hipLaunchKernelGGL((k_decode_tiles<T, 0>), grid, wg, 0, s, a);
  else hipLaunchKernelGGL((k_decode_tiles<T, 1>), grid, wg, 0, s, a);
  return hipGetLastError();
}
template <class T>
hipError_t launch_decode_queries(const ServeArgs& a, uint64_t max_span, int codec, bool hires, hipStream_t s) {
  if (a.nwaves == 0) return hipSuccess;
  const dim3 grid(a.nwaves), wg(64);
  const bool staged = max_span <= kStageWords;
  if (codec == 0 && hires && staged) {
    hipLaunchKernelGGL((k_decode_queries<T, true, 0, true>), grid, wg, 0, s, a);
    return hipGetLastError();
  }
  if (codec == 0) {
    if (staged) hipLaunchKernelGGL((k_decode_queries<T, true, 0>), grid, wg, 0, s, a);
    else hipLaunchKernelGGL((k_decode_queries<T, false, 0>), grid, wg, 0, s, a);
  } else {
    if (staged) hipLaunchKernelGGL((k_decode_queries<T, true, 1>), grid, wg, 0, s, a);
    else hipLaunchKernelGGL((k_decode_queries<T, false, 1>), grid, wg, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace pmc
