// internal.hpp -- host-side objects shared by the C-ABI translation units
// (capi.cpp: single fields and stores; batch.cpp: batches of fields).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/pmc.h"
#include "launch.hpp"

struct ProfRec {
  int kernel;
  hipEvent_t start, stop;
};

// device fields are read and written with 16-byte row accesses
inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

struct pmc_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  std::string err;
  int fused_decode = 1;
  int sync_check = 0;
  int profile = 0;
  int codec = 0;  // the codec pmc_compress uses: 0 block transform, 1 prediction
  std::vector<std::string> prof_names;
  std::vector<uint64_t> prof_launches;
  std::vector<double> prof_ms;
  std::vector<ProfRec> prof_pending;
  std::vector<hipEvent_t> prof_pool;
  // pinned host memory for the small device-to-host reads of the calls that
  // synchronise (range, compressed sizes, decode status): a direct copy
  // instead of one staged through pageable memory; null if it could not be
  // allocated (the calls then read into pageable memory)
  void* pin = nullptr;
};
constexpr size_t kPinBytes = 16384;  // >= kMaxComps * sizeof(CompMeta), the partials of the range

struct pmc_store {
  pmc_field f{};
  pmc::Geo g{};
  int n = 0;
  int codec = 0;  // 0 block transform, 1 prediction (every component of a store)
  std::vector<double> tau, linf;
  std::vector<int> minexp;
  std::vector<uint64_t> bytes, offset, aux_offset, words, nempty, ncoded, nraw, nesc, nmiss;
  std::vector<uint64_t> max_span;  // largest payload words of a decode wave's four chunks
  std::vector<uint64_t> full;      // decode route flags (kNotHi16, ...)
  const uint8_t* d_base = nullptr;  // caller-owned device memory holding the streams
};

namespace pmc_host {

pmc_status fail(pmc_ctx* ctx, pmc_status st, const char* fmt, ...);
pmc_status hipfail(pmc_ctx* ctx, hipError_t e, const char* what);
uint64_t elem_size(const pmc_field* f);
uint64_t stream_cap_one(const pmc::Geo& g, int dtype);
// device workspace for compressing one field into n components, without the
// components' results (CompMeta), and its layout: fills the job's pointers
// into ws (bytes of them) and its sizes; false if it does not fit
uint64_t job_workspace(const pmc_field* f, const pmc::Geo& g, int n);
// resumed: for a launch that goes on from x~ of the components before it
bool job_layout(const pmc_field* f, const pmc::Geo& g, int n, bool resumed, uint8_t* ws, uint64_t bytes,
                pmc::FieldJob* job);
// the first component at or after `from` that outgrew a wave's staging slot (n: none)
int first_over(const pmc::CompMeta* hm, int from, int n);
// the job's x~ tiles taken on from component done to next, which are in place in the region
hipError_t resume_job(pmc_ctx* ctx, const pmc_field* f, const pmc::Geo& g, int n, const double* tau, const int* minexp,
                      const pmc::CompMeta* hm, int codec, int done, int next, pmc::FieldJob* job);
// a store from per-component device results (offsets relative to d_base)
pmc_store* store_from_meta(const pmc_field* f, const pmc::Geo& g, int n, const double* tau, const int* minexp,
                           const pmc::CompMeta* hm, const uint8_t* d_base, int codec);
// the decode arguments of components [i0, i1) of a store
template <class A> void fill_decode_args(const pmc_store* s, int i0, int i1, A& a) {
  for (int i = i0; i < i1; ++i) {
    a.s[i - i0] = s->d_base + s->offset[i];
    a.aux[i - i0] = (const uint32_t*)(s->d_base + s->aux_offset[i]);
    a.words[i - i0] = s->words[i];
    a.minexp[i - i0] = s->minexp[i];
    a.step[i - i0] = 2.0 * s->tau[i];
    if (i > 0) a.relmask |= 1u << (i - i0);  // residual components
  }
  a.ncomp = i1 - i0;
}

// components [i0, i1) decode on the high-half route alone (see launch_decode);
// in float64 a first component then starts from +0
inline bool high_half(const pmc_store* s, int i0, int i1) {
  if (s->codec != 0) return false;
  for (int i = i0; i < i1; ++i) {
    const uint64_t bad = i > 0 ? pmc::kNotHi16 : s->f.dtype == PMC_F32 ? 0u : pmc::kNotHi32 | pmc::kHasRaw;
    if (s->full[i] & bad) return false;
  }
  return true;
}

// The next launch [i0, i1) of a retrieval of components [i0, k), and its
// staging plan if it decodes `waves` waves of blocks with one wave per
// component (k_decode_split); false where one wave decodes all of them.  For a
// box, `waves` counts the workgroups launched, those that meet no block of it
// too.
//
// A launch takes up to eight components (float64 off the high-half routes
// four: 850 spills at the 256 registers of eight), launches of about the same
// size and as few as there can be, and asks for at most 64 KB of LDS per
// workgroup.  It is taken where few rounds of workgroups cover the field: the
// time goes in steps, one per round, and one wave for all components takes
// nearly the same time until the chip is full.  A CU holds as many workgroups
// as fit its registers' 12 waves (float32; float64 8 on the high-half routes,
// else 4), but one of five or more components alone.  Measured (us, one wave
// for all / one per component, cubes; the worse side of each line and the
// better one next to it):
//   float32  8 components, 512 waves (2 rounds) 48 / 31, 729 (3) 48 / 43, 858 (4)
//            48 / 55; 7: 729 (3) 42 / 42; 6: 512 (2) 37 / 30, 729 (3) 37 / 41
//            (off the high-half routes 50 / 45, codec 1 34 / 32, boxes 50 / 46);
//            5: 512 (2) 32 / 29, 615 (3) 33 / 41
//            4: 729 (1) 28 / 22, 858 (2) 29 / 31 (boxes 41 / 35; off the
//            high-half routes 35 / 32, codec 1 26 / 23), 1728 (3) 46 / 49
//            3: 1000 (1) 25 / 24, 1331 (2) 30 / 39
//            2: 216 (1) 19.2 / 18.6, 275 (1) 20.0 / 20.7 (off the high-half
//            routes 729 21.2 / 19.4, 858 21.5 / 22.5; boxes 1352 29 / 28)
//   float64  8: 512 (2) 48 / 41, 615 (3) 48 / 58; 6: 422 (2) 38 / 38; 5: 275
//            (2) 33 / 37; 4: 512 (1) 30 / 23, 615 (2) 31 / 36; 2: 1000 (1) 26 / 23,
//            1331 (2) 29 / 38; off the high-half routes 4: 245 (1) 37 / 22, 275
//            (2) 38 / 37; 3: 275 (2) 29 / 35; 6 in two launches: 245 (1) 52 / 40,
//            275 (2) 53 / 70
//   more components than a launch takes (one wave for all takes sixteen):
//            float32 9: 343 (2) 44 / 41, 10: 48 / 50 (codec 1 48 / 44), 12: 512 (2)
//            56 / 53, 729 (3) 56 / 76, 16: 729 (3) 75 / 82 (codec 1 75 / 69);
//            float64 12: 343 (2) 64 / 72, 16: 81 / 78
inline bool split_plan(const pmc_store* s, int i0, int k, uint64_t waves, bool box, int* i1, pmc::SplitArgs* sp) {
  const bool f32 = s->f.dtype == PMC_F32;
  int most = pmc::kMaxSplit, n = 0, launches = 0;
  bool hires = false;
  for (;;) {
    launches = (k - i0 + most - 1) / most;
    n = (k - i0 + launches - 1) / launches;
    hires = high_half(s, i0, i0 + n);
    if (f32 || hires || most == pmc::kMaxSplit64) break;
    most = pmc::kMaxSplit64;
  }
  if (n < 2) return false;
  uint64_t words = 0;
  for (int j = 0; j < n; ++j) {
    const uint64_t cap = (std::max<uint64_t>(s->max_span[i0 + j], 1) + 63) / 64 * 64;  // copies write whole 64-word rows
    if (cap > 16384) return false;
    sp->base[j] = (uint32_t)words;
    sp->cap[j] = (uint32_t)cap;
    words += cap + 3;  // the reader's look-ahead
  }
  const uint64_t lds = std::max(words * 4, (uint64_t)n * 4096);  // the words, then 4 KB of rows per component
  if (lds > 65536 - 512) return false;
  const uint64_t slots = f32 ? 12 : hires ? 8 : 4;  // waves a CU's registers hold
  const uint64_t resident = std::min<uint64_t>(n > 4 ? 1 : slots / n, 163840 / (lds + 512));
  const uint64_t rounds = (waves + 256 * resident - 1) / (256 * resident);
  uint64_t most_rounds = 1;
  if (launches > 1) {
    if (f32) most_rounds = n == 8 && !hires ? 3 : n >= 6 || !hires || k - i0 == 9 ? 2 : 1;
    else if (hires) most_rounds = n == 8 ? 2 : 1;
    else if (k - i0 < 6) return false;
  } else if (f32) {
    if (n >= 5) most_rounds = n >= 7 || (n == 6 && (box || !hires)) ? 3 : 2;
    if (n == 4 && (box || !hires)) most_rounds = 2;
    if (n == 2 && !box && waves > (hires || s->codec != 0 ? 256u : 768u)) return false;
  } else if (n >= 6) {
    most_rounds = 2;
  }
  if (rounds > most_rounds) return false;
  sp->lds_bytes = (uint32_t)lds;
  *i1 = i0 + n;
  return true;
}

inline hipEvent_t prof_event(pmc_ctx* c) {
  if (!c->prof_pool.empty()) {
    hipEvent_t e = c->prof_pool.back();
    c->prof_pool.pop_back();
    return e;
  }
  // timing only: pmc_prof_read synchronises the stream before it reads
  // them, so the events need no system-scope fence (whose cache writeback
  // and invalidation would also land between the kernels they bracket)
  hipEvent_t e = nullptr;
  if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
  return e;
}

inline int prof_kernel_id(pmc_ctx* c, const char* name) {
  for (size_t i = 0; i < c->prof_names.size(); ++i)
    if (c->prof_names[i] == name) return (int)i;
  c->prof_names.push_back(name);
  c->prof_launches.push_back(0);
  c->prof_ms.push_back(0.0);
  return (int)c->prof_names.size() - 1;
}

// brackets one kernel launch (or graph launch) with events on the context
// stream when profiling is enabled
struct ProfScope {
  pmc_ctx* c;
  ProfRec r{};
  bool on;
  ProfScope(pmc_ctx* ctx, const char* name) : c(ctx), on(ctx->profile != 0) {
    if (!on) return;
    r.kernel = prof_kernel_id(c, name);
    r.start = prof_event(c);
    r.stop = prof_event(c);
    if (!r.start || !r.stop) {
      on = false;
      return;
    }
    (void)hipEventRecord(r.start, c->stream);
  }
  ~ProfScope() {
    if (!on) return;
    (void)hipEventRecord(r.stop, c->stream);
    c->prof_pending.push_back(r);
  }
};

}  // namespace pmc_host
