// pack.hip -- from the encoder's staged spans to streams: chunk offsets (an
// exclusive scan of chunk word counts), the per-component bookkeeping
// (CompMeta), and the copy of header, index and payload (format version 1).
//
//  k_pack_sums   one tile's sums of one component
//  k_pack_heads  one component: the words before each tile, its place in the
//                stream buffer, its CompMeta
//  k_pack        one tile of one component: index and payload; for small
//                fields it also does the work of the other two
//
// All components of a field go through each launch together.  What bounds them
// is launch latency for small fields and memory for large ones.  Nothing is
// reduced with atomics: with one launch per component, each of whose 4096 to
// 8192 waves raised the largest span in one word, a pack took 34 to 45 us
// whatever its size (10 ns per atomic on one line).
#include "block_device.hpp"

namespace pmc {

typedef __attribute__((address_space(4))) const FieldJob CFieldJob;
typedef uint32_t u4_any __attribute__((ext_vector_type(4), aligned(4)));  // a 16-byte access at any word

// (k_pack: 16 waves, so that the few tiles of a small field move four spans per
// wave; a span takes about 2 us of latency, and 16 of them one after the other
// held a 64^3 float64 field up for 26 us)
constexpr int kPackThreads = 1024, kSumThreads = 256;
static_assert(kSumThreads == kPackTile, "one chunk per thread");
constexpr int kTileWaves = kPackTile / 4;  // encoder waves of a tile
// Fields of up to this many chunks (a million values) take the pack alone: each
// of its workgroups adds up the chunk words of the components before its own,
// at most 16 loads per lane and component, where two more launches cost about
// 10 us.
constexpr uint64_t kDirectChunks = kPackThreads;
// ... and several workgroups to a tile, each moving a part of its spans: one
// per wave, where 16 waves took four each (64^3 float64, 4 components: 18 us).
constexpr uint32_t kDirectParts = kTileWaves / (kPackThreads / 64);

struct Sums {
  unsigned long long words;
  unsigned long long linf;  // bits of a non-negative double: they order like it
  unsigned long long counts;  // empty, raw, escalated, missed blocks, 16 bits each (at most 16384 blocks a time)
  uint32_t stat, span;
};
__device__ __forceinline__ unsigned long long max_of(unsigned long long a, unsigned long long b) { return a > b ? a : b; }
__device__ __forceinline__ void add_to(Sums& s, const Sums& o) {
  s.words += o.words;
  s.linf = max_of(s.linf, o.linf);
  s.counts += o.counts;
  s.stat |= o.stat;
  s.span = o.span > s.span ? o.span : s.span;
}
// the sums of a workgroup of W waves, in every thread
template <int W> __device__ __forceinline__ void block_add(Sums& s, Sums* sh) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    Sums o;
    o.words = __shfl_xor(s.words, d, 64);
    o.linf = __shfl_xor(s.linf, d, 64);
    o.counts = __shfl_xor(s.counts, d, 64);
    o.stat = __shfl_xor(s.stat, d, 64);
    o.span = __shfl_xor(s.span, d, 64);
    add_to(s, o);
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  s = sh[0];
  for (int w = 1; w < W; ++w) add_to(s, sh[w]);
}
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}
// this thread's chunk of one component, and its wave record
__device__ __forceinline__ void take(const CFieldJob& f, int comp, uint64_t chunk, bool has_wave, uint64_t wave, Sums& s) {
  const uint32_t w = chunk < f.g.nchunks ? to_global(f.chunk_words)[(uint64_t)comp * f.g.nchunks + chunk] : 0u;
  s.words = w;
  uint32_t q = w + __shfl_xor(w, 1, 64);  // four consecutive chunks
  q += __shfl_xor(q, 2, 64);
  s.span = q;
  s.linf = s.counts = 0;
  s.stat = 0;
  if (has_wave && wave < job_waves(f)) {
    const uint64_t at = (uint64_t)comp * job_waves(f) + wave;
    s.linf = to_global((const unsigned long long*)f.wave_linf)[at];
    const uint32_t st = to_global(f.wave_stat)[at];
    s.counts = (unsigned long long)(st & 127u) | ((unsigned long long)((st >> 7) & 127u) << 16) |
               ((unsigned long long)((st >> 14) & 127u) << 32) | ((unsigned long long)((st >> 21) & 127u) << 48);
    s.stat = st & (kStatNotHi16 | kStatNotHi32 | kStatNonfinite | kStatOver);
  }
}
// a component's totals over its tiles
struct Totals {
  unsigned long long words, linf, ne, nr, ns, nm;
  uint32_t stat, span;
};
__device__ __forceinline__ void add_counts(Totals& t, const Sums& s) {
  t.linf = max_of(t.linf, s.linf);
  t.ne += s.counts & 0xFFFFull;
  t.nr += (s.counts >> 16) & 0xFFFFull;
  t.ns += (s.counts >> 32) & 0xFFFFull;
  t.nm += s.counts >> 48;
  t.stat |= s.stat;
  t.span = s.span > t.span ? s.span : t.span;
}
__device__ __forceinline__ void write_meta(const CFieldJob& f, int comp, const Totals& s, unsigned long long offset) {
  CompMeta m = {};
  m.linf_bits = s.linf;
  m.nempty = s.ne;
  m.nraw = s.nr;
  m.nesc = s.ns;
  m.nmiss = s.nm;
  m.payload_words = s.words;
  m.stream_offset = offset;
  m.stream_bytes = (unsigned long long)kHeaderBytes + 4ull * f.g.nchunks + 4ull * s.words;
  m.flags = (s.stat & kStatNonfinite ? FLAG_NONFINITE : 0u) | (s.stat & kStatOver ? FLAG_STAGING : 0u) |
            (offset + m.stream_bytes > f.region_cap ? FLAG_OVERFLOW : 0u) | (s.words > 0xFFFFFFFFull ? FLAG_INDEX : 0u);
  m.max_span = s.span;
  m.full = (s.stat & kStatNotHi16 ? kNotHi16 : 0u) | (s.stat & kStatNotHi32 ? kNotHi32 : 0u) |
           (f.dtype == 2 && f.codec == 0 && s.nr ? kHasRaw : 0u);
  *(CompMeta*)(f.meta + comp) = m;
  if (f.host_meta) f.host_meta[comp] = m;
}
// where component comp's stream starts, from the words of the components of
// this launch before it (words[0..]) and, for a later launch, the record of
// the one before
__device__ __forceinline__ unsigned long long stream_offset(const CFieldJob& f, int comp,
                                                            const unsigned long long* words) {
  unsigned long long off = 4ull * f.ncomp * f.aux_stride;
  if (f.comp0 > 0) {
    const gptr<CompMeta> m = to_global(f.meta) + (f.comp0 - 1);
    off = (m->stream_offset + m->stream_bytes + 255ull) & ~255ull;
  }
  for (int j = f.comp0; j < comp; ++j)
    off = (off + kHeaderBytes + 4ull * f.g.nchunks + 4ull * words[j - f.comp0] + 255ull) & ~255ull;
  return off;
}

__device__ __forceinline__ void pack_sums(const CFieldJob& f, int comp, uint64_t tile) {
  __shared__ Sums sh[kSumThreads / 64];
  const uint32_t t = threadIdx.x;
  Sums s;
  take(f, comp, tile * kPackTile + t, t < (uint32_t)kTileWaves, tile * kTileWaves + t, s);
  block_add<kSumThreads / 64>(s, sh);
  if (t == 0) {
    const gptr<TileRec> r = to_global(f.tile_recs) + ((uint64_t)comp * job_tiles(f) + tile);
    r->words = s.words;
    r->linf = s.linf;
    r->counts = s.counts;
    r->stat = s.stat;
    r->span = s.span;
  }
}

__device__ __forceinline__ void pack_heads(const CFieldJob& f, int comp) {
  constexpr uint32_t W = kPackThreads / 64;
  __shared__ unsigned long long s_words[kMaxComps], s_wave[W];
  __shared__ Totals s_tot;
  const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6, ntiles = job_tiles(f);
  if (t == 0) s_tot = Totals{};
  // the components before this one: one wave each adds up their tiles
  for (int j = f.comp0 + (int)wv; j < comp; j += (int)W) {
    unsigned long long v = 0;
    for (uint64_t k = lane; k < ntiles; k += 64) v += (to_global(f.tile_recs) + ((uint64_t)j * ntiles + k))->words;
    v = wave_sum(v);
    if (lane == 0) s_words[j - f.comp0] = v;
  }
  // this one: the words before each tile, and the component's totals
  Totals all = {};
  unsigned long long carry = 0;
  for (uint64_t k0 = 0; k0 < ntiles; k0 += kPackThreads) {
    const uint64_t k = k0 + t;
    const gptr<TileRec> r = to_global(f.tile_recs) + ((uint64_t)comp * ntiles + k);
    unsigned long long w = 0;
    if (k < ntiles) {
      Sums s;
      w = r->words;
      s.linf = r->linf;
      s.counts = r->counts;
      s.stat = r->stat;
      s.span = r->span;
      add_counts(all, s);
    }
    unsigned long long inc = w;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned long long y = __shfl_up(inc, d, 64);
      if (lane >= (uint32_t)d) inc += y;
    }
    __syncthreads();
    if (lane == 63) s_wave[wv] = inc;
    __syncthreads();
    unsigned long long below = carry, total = 0;
    for (uint32_t q = 0; q < W; ++q) {
      below += q < wv ? s_wave[q] : 0ull;
      total += s_wave[q];
    }
    if (k < ntiles) r->before = below + inc - w;
    carry += total;
  }
  // (few threads have anything to add for most of these)
  if (all.linf) atomicMax(&s_tot.linf, all.linf);
  if (all.ne) atomicAdd(&s_tot.ne, all.ne);
  if (all.nr) atomicAdd(&s_tot.nr, all.nr);
  if (all.ns) atomicAdd(&s_tot.ns, all.ns);
  if (all.nm) atomicAdd(&s_tot.nm, all.nm);
  if (all.stat) atomicOr(&s_tot.stat, all.stat);
  if (all.span) atomicMax(&s_tot.span, all.span);
  __syncthreads();
  if (t == 0) {
    Totals m = s_tot;
    m.words = carry;
    write_meta(f, comp, m, stream_offset(f, comp, s_words));
  }
}

// part of parts: the workgroup's share of the tile's spans
template <bool kDirect>
__device__ __forceinline__ void pack_tile(const CFieldJob& f, int comp, uint64_t tile, uint32_t part = 0,
                                          uint32_t parts = 1) {
  __shared__ Sums sh[kPackThreads / 64];
  __shared__ unsigned long long s_words[kMaxComps];
  __shared__ uint32_t s_pre[kPackTile + 1];  // words before each chunk of the tile
  __shared__ uint32_t s_start[kTileWaves], s_wave[kPackTile / 64];
  const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint64_t nchunks = f.g.nchunks, chunk = tile * kPackTile + t;
  const gptr<uint32_t> cw = to_global(f.chunk_words);
  unsigned long long offset, before, words;
  uint32_t flags;
  if constexpr (kDirect) {
    for (int j = f.comp0 + (int)wv; j < comp; j += kPackThreads / 64) {
      unsigned long long v = 0;
      for (uint64_t k = lane; k < nchunks; k += 64) v += cw[(uint64_t)j * nchunks + k];
      v = wave_sum(v);
      if (lane == 0) s_words[j - f.comp0] = v;
    }
    // every chunk of this one has its thread; the words before the tile ride
    // in the high half (such a field's component has fewer than 2^32 words)
    Sums s;
    take(f, comp, t, t < job_waves(f), t, s);
    if (t < tile * kPackTile) s.words |= s.words << 32;
    block_add<kPackThreads / 64>(s, sh);
    words = s.words & 0xFFFFFFFFull;
    before = s.words >> 32;
    offset = stream_offset(f, comp, s_words);
    const unsigned long long end = offset + kHeaderBytes + 4ull * nchunks + 4ull * words;
    flags = (s.stat & kStatOver) || end > f.region_cap || words > 0xFFFFFFFFull;
    if (tile == 0 && part == 0 && t == 0) {
      Totals m = {};
      m.words = words;
      add_counts(m, s);
      write_meta(f, comp, m, offset);
    }
  } else {
    const gptr<CompMeta> m = to_global(f.meta) + comp;
    offset = m->stream_offset;
    words = m->payload_words;
    flags = m->flags & (FLAG_OVERFLOW | FLAG_INDEX | FLAG_STAGING);
    before = (to_global(f.tile_recs) + ((uint64_t)comp * job_tiles(f) + tile))->before;
  }
  if (flags) return;  // uniform: nothing is written past the stream buffer
  const gptr<uint32_t> head = (gptr<uint32_t>)(to_global(f.region) + offset);
  const gptr<uint32_t> index = head + kHeaderBytes / 4;
  const gptr<uint32_t> payload = index + nchunks + before;  // the tile's words

  // offsets of the tile's chunks, and where its waves' spans start
  const uint64_t wave0 = tile * kTileWaves;
  uint32_t w = 0, inc = 0;
  if (t < (uint32_t)kPackTile) {
    w = chunk < nchunks ? cw[(uint64_t)comp * nchunks + chunk] : 0u;
    inc = w;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d, 64);
      if (lane >= (uint32_t)d) inc += y;
    }
    if (lane == 63) s_wave[wv] = inc;
    if (t < (uint32_t)kTileWaves)
      s_start[t] =
          wave0 + t < job_waves(f) && f.ncomp > 1 ? to_global(f.wave_start)[(uint64_t)comp * job_waves(f) + wave0 + t] : 0u;
  }
  __syncthreads();
  if (t < (uint32_t)kPackTile) {
    for (uint32_t q = 0; q < wv; ++q) inc += s_wave[q];
    s_pre[t + 1] = inc;
    if (t == 0) s_pre[0] = 0;
    if (part == 0 && chunk < nchunks) index[chunk] = (uint32_t)before + inc - w;
  }
  __syncthreads();

  // the spans: one wave moves one encoder wave's words at a time
  for (uint32_t q = wv + part * (kPackThreads / 64); q < (uint32_t)kTileWaves && wave0 + q < job_waves(f);
       q += parts * (kPackThreads / 64)) {
    const uint32_t o = s_pre[4 * q], span = s_pre[4 * q + 4] - o, start = s_start[q];
    const uint64_t wave = wave0 + q;
    const gptr<const uint32_t> src = to_global((const uint32_t*)f.staging) + (wave * f.slot_words + start);
    const gptr<uint32_t> dst = payload + o;
    const uint32_t n16 = span / 4;
    for (uint32_t k0 = 0; k0 < n16; k0 += 256) {
      nt_u4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {  // four 16-byte loads in flight
        const uint32_t at = k0 + 64 * k + lane;
        if (at < n16) v[k] = __builtin_nontemporal_load((gptr<const nt_u4>)src + at);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t at = k0 + 64 * k + lane;
        if (at < n16) *((gptr<u4_any>)dst + at) = (u4_any)v[k];
      }
    }
    if (lane < span - 4 * n16) dst[4 * n16 + lane] = src[4 * n16 + lane];
  }

  if (tile == 0 && part == 0 && t < 16) {
    const uint64_t taub = (uint64_t)__double_as_longlong(f.tau[comp]);
    uint32_t v = 0;
    switch (t) {
      case 0: v = kMagic; break;
      case 1: v = (uint32_t)kVersion | ((uint32_t)f.codec << 8) | ((uint32_t)f.dtype << 16) | (3u << 24); break;
      case 2: v = (uint32_t)f.g.nx; break;
      case 3: v = (uint32_t)(f.g.nx >> 32); break;
      case 4: v = (uint32_t)f.g.ny; break;
      case 5: v = (uint32_t)(f.g.ny >> 32); break;
      case 6: v = (uint32_t)f.g.nz; break;
      case 7: v = (uint32_t)(f.g.nz >> 32); break;
      case 8: v = (uint32_t)taub; break;
      case 9: v = (uint32_t)(taub >> 32); break;
      case 10: v = (uint32_t)f.minexp[comp]; break;
      case 11: v = (uint32_t)kChunkBlocks; break;
      case 12: v = (uint32_t)nchunks; break;
      case 13: v = (uint32_t)(nchunks >> 32); break;
      case 14: v = (uint32_t)words; break;
      case 15: v = (uint32_t)(words >> 32); break;
    }
    head[t] = v;
  }
}

// a single field's job is the kernel's argument, a batch's come from its table
__device__ __forceinline__ const CFieldJob& arg_job() {
  return *(const CFieldJob*)__builtin_amdgcn_kernarg_segment_ptr();
}
__global__ __launch_bounds__(kSumThreads) void k_pack_sums(FieldJob) {
  const CFieldJob& f = arg_job();
  pack_sums(f, f.comp0 + (int)blockIdx.y, blockIdx.x);
}
__global__ __launch_bounds__(kPackThreads) void k_pack_heads(FieldJob) {
  const CFieldJob& f = arg_job();
  pack_heads(f, f.comp0 + (int)blockIdx.x);
}
template <bool kDirect> __global__ __launch_bounds__(kPackThreads) void k_pack(FieldJob) {
  const CFieldJob& f = arg_job();
  pack_tile<kDirect>(f, f.comp0 + (int)blockIdx.y, blockIdx.x, blockIdx.z, kDirect ? kDirectParts : 1u);
}
__global__ __launch_bounds__(kSumThreads) void k_bpack_sums(BatchArgs b) {
  const Item it = b.items[blockIdx.x];
  const CFieldJob& f = ((const CFieldJob*)b.fields)[it.field];
  const int comp = f.comp0 + (int)blockIdx.y;
  if (comp < f.comp1) pack_sums(f, comp, it.index);
}
__global__ __launch_bounds__(kPackThreads) void k_bpack_heads(BatchArgs b) {
  const CFieldJob& f = ((const CFieldJob*)b.fields)[blockIdx.x];
  const int comp = f.comp0 + (int)blockIdx.y;
  if (comp < f.comp1) pack_heads(f, comp);
}
__global__ __launch_bounds__(kPackThreads) void k_bpack(BatchArgs b) {
  const Item it = b.items[blockIdx.x];
  const CFieldJob& f = ((const CFieldJob*)b.fields)[it.field];
  const int comp = f.comp0 + (int)blockIdx.y;
  if (comp < f.comp1) pack_tile<false>(f, comp, it.index);
}

hipError_t launch_pack(const FieldJob& f, hipStream_t s) {
  const uint32_t comps = (uint32_t)(f.comp1 - f.comp0);
  const dim3 tiles(job_tiles(f), comps), wg(kPackThreads);
  if (f.g.nchunks <= kDirectChunks) {
    hipLaunchKernelGGL(k_pack<true>, dim3(tiles.x, tiles.y, kDirectParts), wg, 0, s, f);
  } else {
    hipLaunchKernelGGL(k_pack_sums, tiles, dim3(kSumThreads), 0, s, f);
    hipLaunchKernelGGL(k_pack_heads, dim3(comps), wg, 0, s, f);
    hipLaunchKernelGGL(k_pack<false>, tiles, wg, 0, s, f);
  }
  return hipGetLastError();
}
hipError_t launch_batch_pack(const BatchArgs& b, uint32_t comps, hipStream_t s) {
  const dim3 tiles(b.nitems, comps), wg(kPackThreads);
  hipLaunchKernelGGL(k_bpack_sums, tiles, dim3(kSumThreads), 0, s, b);
  hipLaunchKernelGGL(k_bpack_heads, dim3(b.nfields, comps), wg, 0, s, b);
  hipLaunchKernelGGL(k_bpack, tiles, wg, 0, s, b);
  return hipGetLastError();
}

}  // namespace pmc
