// launch.hpp -- kernel argument blocks and host launchers shared by the HIP
// kernels (kernels.hip) and the C-ABI (capi.cpp).  Internal to the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "format.hpp"  // the block grid and the stream constants

namespace pmc {

constexpr int kMaxDecode = 16;  // components decoded by one k_decode launch

enum : unsigned int {
  FLAG_NONFINITE = 1u,  // NaN / Inf in the input field
  FLAG_OVERFLOW = 2u,   // stream capacity exceeded
  FLAG_INDEX = 4u,      // payload too large for 32-bit word offsets
  FLAG_STAGING = 8u     // a wave's staging slot was too small for every component
};

// what a component's blocks ask of the decode routes (CompMeta.full): a coded
// block outside the high-half route; in float64 also one outside the high-word
// route, and a raw block
constexpr uint32_t kNotHi16 = 1u, kNotHi32 = 2u, kHasRaw = 4u;

// per-component results kept on the device during compression
struct CompMeta {
  unsigned long long linf_bits;  // max measured error, float64 bits (>= 0)
  unsigned long long nempty, ncoded, nraw, nesc, nmiss;  // ncoded: not counted on the device
  unsigned long long payload_words;
  unsigned long long stream_offset;  // byte offset of the stream in the output
  unsigned long long stream_bytes;
  unsigned int flags;
  unsigned int pad;
  unsigned long long max_span;  // largest payload words of four consecutive chunks (one decode wave)
  unsigned long long full;      // decode route flags (kNotHi16, ...) of the component's blocks
  unsigned long long reserved[4];
};
static_assert(sizeof(CompMeta) == 128, "CompMeta layout");

// chunk offsets are an exclusive scan of chunk word counts, in tiles of
// kPackTile chunks (64 encoder waves), one pack workgroup each
constexpr int kPackTile = 256;
// one tile's sums of one component
struct TileRec {
  unsigned long long words;   // payload words of the tile's chunks
  unsigned long long before;  // ... of the tiles before it
  unsigned long long linf;    // bits of the largest measured error
  unsigned long long counts;  // empty, raw, escalated, missed blocks, 16 bits each
  uint32_t stat;              // kStat* flags of any wave
  uint32_t span;              // largest payload words of four consecutive chunks
  unsigned long long pad[2];
};
static_assert(sizeof(TileRec) == 56, "TileRec layout");

// one wave's record of one component (wave_stat): the counts of empty, raw,
// escalated and missed blocks (7 bits each), then flags
constexpr uint32_t kStatNotHi16 = 1u << 28;    // kNotHi16 of a block
constexpr uint32_t kStatNonfinite = 1u << 29;  // NaN / Inf in the input
constexpr uint32_t kStatOver = 1u << 30;       // the wave's slot was too small for this component
constexpr uint32_t kStatNotHi32 = 1u << 31;    // kNotHi32 of a block

// One field being compressed: components [comp0, comp1) in one launch.  The
// encoder's waves (64 blocks, 4 chunks each) take their blocks through all of
// them and leave each component's span of payload words in the wave's staging
// slot, one behind the other; the pack moves the spans into the streams.
struct FieldJob {
  const void* x;
  Geo g;
  void* tiles;        // x~ of every wave between launches (64 * 64 values each), where components take several
  uint32_t* staging;  // wave w's slot at w * slot_words
  uint32_t slot_words, slot_last;  // words of a slot, of the last wave's
  uint32_t* chunk_words;  // [component][chunk]
  double* wave_linf;      // [component][wave] largest measured error
  uint32_t* wave_stat;    // [component][wave]
  uint32_t* wave_start;   // [component][wave] first word of the span in its slot; none for one component (0)
  TileRec* tile_recs;     // [component][tile]
  CompMeta* meta;         // [component], written by the pack's bookkeeping
  CompMeta* host_meta;    // the same in pinned host memory (may be null)
  uint8_t* region;        // the stream region: block indexes, then streams
  unsigned long long region_cap;
  uint64_t aux_stride;    // block index of component i at region + 4 * i * aux_stride
  uint8_t ncomp, comp0, comp1;
  uint8_t dtype, codec;   // dtype 1 = f32, 2 = f64
  uint8_t pad[3];
  double tau[kMaxComps];
  int32_t minexp[kMaxComps];
};
static_assert(sizeof(FieldJob) == 576, "a batch's table has its place in the workspace");
template <class F> __host__ __device__ inline uint32_t job_waves(const F& f) { return (uint32_t)((f.g.nblocks + 63) / 64); }
template <class F> __host__ __device__ inline uint32_t job_tiles(const F& f) {
  return (uint32_t)((f.g.nchunks + kPackTile - 1) / kPackTile);
}

template <class T> struct DecArgs {
  const uint8_t* s[kMaxDecode];    // stream starts
  const uint32_t* aux[kMaxDecode];  // per-block bit offsets inside the chunk
  uint64_t words[kMaxDecode];      // payload words of each stream
  int minexp[kMaxDecode];
  double step[kMaxDecode];  // codec 1: the bin 2 tau of each component
  int ncomp;
  uint32_t relmask;  // bit i: component i is a residual (not a store's first), planes counted from its first non-empty one
  const T* in;  // x~ to continue from; NULL = +0
  T* out;
  Geo g;
  unsigned int* status;  // bit 0: malformed stream
};

// a launch with one wave per component: where each component's words are
// staged in the workgroup's LDS (word offset, and words it holds)
constexpr int kMaxSplit = 8, kMaxSplit64 = 4;  // (4: float64 that is not hires)
struct SplitArgs {  // (launch_decode, launch_decode_box: null for one wave over all components)
  uint32_t base[kMaxSplit], cap[kMaxSplit];
  uint32_t lds_bytes;
};
// a box [lo, hi) of the field (value coordinates x, y, z) for region
// retrieval: blo/bhi are its block ranges; the output is the box alone, dense,
// x fastest.  Work: one workgroup per (block row of the box, wave of that row)
struct BoxArgs {
  uint64_t lo[3], hi[3];
  uint64_t blo[3], bhi[3];
  uint32_t waves_per_row;
  uint32_t pad;
  uint64_t row_first, row_last;  // set per workgroup: the blocks of its row inside the box
};

// one retrieval query of a server step: out = in (or +0) + components
// [0, ncomp) of the listed streams
struct QueryDev {
  const uint8_t* s[kMaxComps];
  const uint32_t* aux[kMaxComps];
  uint64_t words[kMaxComps];
  int minexp[kMaxComps];
  double step[kMaxComps];  // codec 1: the bin 2 tau of each component
  int ncomp;
  uint32_t relmask;  // as DecArgs::relmask
  int dtype;
  const void* in;
  void* out;
  void* out2;  // NULL, or a second place for the result
  Geo g;
};

struct ServeArgs {
  const QueryDev* q;
  const uint32_t* wave_prefix;  // nq + 1 entries
  uint32_t nq;
  uint32_t nwaves;
  unsigned int* status;
};

// rebuild the per-block bit offsets of a store's streams
struct AuxArgs {
  const uint8_t* s[kMaxComps];
  uint32_t* aux[kMaxComps];
  uint64_t words[kMaxComps];
  int minexp[kMaxComps];
  Geo g;
  uint32_t cap;  // words a wave's chunks can have
  unsigned int* status;  // set when a chunk fails to parse
  unsigned long long* full;  // [component] decode route flags, raised
};

struct Item {  // (field, group): a wave of 64 blocks or a pack tile
  uint32_t field, index;
};

struct BatchArgs {
  const FieldJob* fields;
  uint32_t nfields;
  const Item* items;  // encode waves of one dtype, or pack tiles
  uint32_t nitems;
};

// every component of a field (job.codec 0 or 1), then the scan and pack of its streams
template <class T> hipError_t launch_encode(const FieldJob& f, hipStream_t s);
hipError_t launch_pack(const FieldJob& f, hipStream_t s);
// the same for a batch (comps: the most components [comp0, comp1) of any field)
template <class T> hipError_t launch_encode_batch(const BatchArgs& a, uint32_t grid, hipStream_t s);
hipError_t launch_batch_pack(const BatchArgs& tiles, uint32_t comps, hipStream_t s);

// ncomp streams at once; max_span: the most payload words of four consecutive
// chunks (aligned to four) of any of them
template <class T> hipError_t launch_aux(AuxArgs a, int ncomp, uint64_t max_span, int codec, hipStream_t s);
// max_span: the largest word span of a wave's four chunks over the decoded
// streams; spans up to the LDS staging capacity use the staged kernel
// hires: as launch_decode's, for every query of the launch
template <class T>
hipError_t launch_decode_queries(const ServeArgs& a, uint64_t max_span, int codec, bool hires, hipStream_t s);
// hires: no residual component of the launch (store index > 0) has kNotHi16 and,
// in float64, a first one neither kNotHi32 nor kHasRaw (and a.in is null then):
// the decoder runs on those routes alone
template <class T>
hipError_t launch_decode(const DecArgs<T>& a, uint64_t max_span, int codec, bool hires, const SplitArgs* split,
                         hipStream_t s);
// components [0, a.ncomp) of the blocks meeting the box, written to a.out as the box alone
template <class T>
hipError_t launch_decode_box(const DecArgs<T>& a, const BoxArgs& b, uint64_t max_span, int codec, bool hires,
                             const SplitArgs* split, hipStream_t s);
// components [0, a.ncomp) added to the encoder's x~ tiles (FieldJob::tiles) at a.in, into those at a.out
template <class T> hipError_t launch_decode_tiles(const DecArgs<T>& a, int codec, hipStream_t s);
uint64_t stage_words();  // capacity of the decoder's LDS staging buffer, in words
// min / max / non-finite count of n samples: one partial of kRangeWords words
// per workgroup at out; range_groups: how many workgroups suit n, at most
// max_groups
constexpr uint32_t kRangeWords = 3, kRangeGroups = 256;
uint32_t range_groups(uint64_t n, uint64_t max_groups);
template <class T>
hipError_t launch_range(const T* x, uint64_t n, unsigned long long* out, uint32_t groups, hipStream_t s);
hipError_t launch_fill64(unsigned long long* p, uint64_t n, unsigned long long v, hipStream_t s);
// out[0] = sum of d, out[1] = sum of d^2 in float64, d = a - b - shift (b NULL: 0);
// ws holds sum_sq_ws_bytes() bytes of partials; out may lie inside ws past them
template <class T>
hipError_t launch_sum_sq(const T* a, const T* b, double shift, uint64_t n, double* ws, double* out, hipStream_t s);
uint64_t sum_sq_ws_bytes();
// the float32-cast compressor: comps holds n components of N values each;
// linf: n zeroed bit patterns of the measured errors (raised with atomics)
template <class T>
hipError_t launch_cast_encode(const T* x, uint64_t N, int n, float* comps, unsigned long long* linf, hipStream_t s);
template <class T> hipError_t launch_cast_decode(const float* comps, uint64_t N, int k, T* out, hipStream_t s);

// capacity of one chunk in 32-bit words: 16 raw blocks (coded ones are never
// larger, the acceptance rule falls back to raw first)
inline uint64_t chunk_cap_words_host(int dtype) {
  const uint64_t raw = dtype == 1 ? 2 + 64 * 32 : 2 + 64 * 64;
  return (16 * raw + 31) / 32;
}

}  // namespace pmc
