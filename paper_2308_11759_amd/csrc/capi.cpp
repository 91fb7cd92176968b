// capi.cpp -- C-ABI of the progressive multi-component codec (see include/pmc.h).
// Host code only: argument checks, workspace layout, kernel sequencing, and
// the per-component metadata of the store.  Every arithmetic step of the path
// runs in the HIP kernels (the .hip sources).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "internal.hpp"

using namespace pmc;
using namespace pmc_host;

namespace pmc_host {

pmc_status fail(pmc_ctx* ctx, pmc_status st, const char* fmt, ...) {
  if (ctx) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    ctx->err = buf;
  }
  return st;
}

pmc_status hipfail(pmc_ctx* ctx, hipError_t e, const char* what) {
  return fail(ctx, PMC_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

uint64_t elem_size(const pmc_field* f) { return f->dtype == PMC_F32 ? 4 : 8; }

uint64_t job_workspace(const pmc_field* f, const Geo& g, int n) {
  const uint64_t tiles = align256((g.nblocks + 63) / 64 * 4096 * elem_size(f));
  uint64_t o = align256(g.nchunks * chunk_cap_words_host(f->dtype) * 4);  // one component, every block raw
  if (n > 1) o += tiles;
  if (n > 2) o += tiles;
  o += 2 * align256(g.nchunks * 4) + align256((g.nchunks + 1023) / 1024 * 8);
  if (n > 1) o += align256(g.nblocks * 8);
  return o;
}

// The workspace of one field: the staging slots, and at its end the records.
// A slot holds every component's span of its wave one behind the other: n
// components with every block raw for n <= 2, 96 bits per float32 and 192 per
// float64 value for more.  Data that needs more (FLAG_STAGING) has its later
// components in further launches (resumed): x~ of the components before takes a
// tile per wave in front, and the slots share the rest, 64 and 128 bits per
// value, which holds any one component with every block raw.
bool job_layout(const pmc_field* f, const Geo& g, int n, bool resumed, uint8_t* ws, uint64_t bytes, FieldJob* job) {
  const uint64_t nwaves = (g.nblocks + 63) / 64, ntiles = (g.nchunks + kPackTile - 1) / kPackTile;
  const uint64_t one = 4 * chunk_cap_words_host(f->dtype);  // words of a wave with every block raw
  if (nwaves > 0xFFFFFFFFull) return false;
  uint64_t end = bytes & ~15ull;
  auto take = [&](uint64_t size) {  // an array at the end of what is left
    size = (size + 15) & ~15ull;
    if (end < size) return (uint8_t*)nullptr;
    end -= size;
    return ws + end;
  };
  job->chunk_words = (uint32_t*)take((uint64_t)n * g.nchunks * 4);
  job->wave_linf = (double*)take((uint64_t)n * nwaves * 8);
  job->wave_stat = (uint32_t*)take((uint64_t)n * nwaves * 4);
  job->wave_start = n > 1 ? (uint32_t*)take((uint64_t)n * nwaves * 4) : nullptr;
  job->tile_recs = (TileRec*)take((uint64_t)n * ntiles * sizeof(TileRec));
  const uint64_t tiles = resumed ? align256(nwaves * 4096 * elem_size(f)) : 0;
  if (!job->tile_recs || end < tiles) return false;
  const uint64_t words = (end - tiles) / 16 * 4;
  const uint64_t slot = n <= 2 ? one * n : std::min<uint64_t>(words / nwaves / 4 * 4, 0x40000000ull);
  if (words < (nwaves - 1) * slot) return false;
  const uint64_t last = std::min(slot, (words - (nwaves - 1) * slot) / 4 * 4);
  const uint64_t need = ((g.nchunks - 4 * (nwaves - 1)) * chunk_cap_words_host(f->dtype) + 3) / 4 * 4;
  if (last < need || (nwaves > 1 && slot < one)) return false;
  job->tiles = ws;
  job->staging = (uint32_t*)(ws + tiles);
  job->slot_words = (uint32_t)slot;
  job->slot_last = (uint32_t)last;
  job->g = g;
  job->ncomp = (uint8_t)n;
  job->comp0 = 0;
  job->comp1 = (uint8_t)n;
  job->dtype = (uint8_t)f->dtype;
  return true;
}

uint64_t stream_cap_one(const Geo& g, int dtype) {
  return kStreamHeader + 4 * g.nchunks + 4 * g.nchunks * chunk_cap_words_host(dtype);
}

pmc_store* store_from_meta(const pmc_field* f, const Geo& g, int n, const double* tau, const int* minexp,
                           const CompMeta* hm, const uint8_t* d_base, int codec) {
  pmc_store* s = new pmc_store();
  s->f = *f;
  s->g = g;
  s->n = n;
  s->codec = codec;
  s->d_base = d_base;
  const uint64_t auxb = aux_bytes(g);
  for (int i = 0; i < n; ++i) {
    double l;
    std::memcpy(&l, &hm[i].linf_bits, 8);
    s->tau.push_back(tau[i]);
    s->linf.push_back(l);
    s->minexp.push_back(minexp[i]);
    s->bytes.push_back(hm[i].stream_bytes);
    s->offset.push_back(hm[i].stream_offset);
    s->aux_offset.push_back(i * auxb);
    s->words.push_back(hm[i].payload_words);
    s->nempty.push_back(hm[i].nempty);
    s->ncoded.push_back(g.nblocks - hm[i].nempty - hm[i].nraw);  // the encoder counts the others only
    s->nraw.push_back(hm[i].nraw);
    s->nesc.push_back(hm[i].nesc);
    s->nmiss.push_back(hm[i].nmiss);
    s->max_span.push_back(hm[i].max_span);
    s->full.push_back(hm[i].full);
  }
  return s;
}

int first_over(const CompMeta* hm, int from, int n) {
  while (from < n && !(hm[from].flags & FLAG_STAGING)) ++from;
  return from;
}

template <class T> static hipError_t decode_tiles(const pmc_store* s, int i0, int i1, bool first, FieldJob* job,
                                                   hipStream_t stream) {
  DecArgs<T> a{};
  fill_decode_args(s, i0, i1, a);
  a.in = first ? nullptr : (const T*)job->tiles;
  a.out = (T*)job->tiles;
  a.g = s->g;
  a.status = (unsigned int*)job->tile_recs;  // (never set on streams just written; written again before it is read)
  return launch_decode_tiles<T>(a, s->codec, stream);
}

hipError_t resume_job(pmc_ctx* ctx, const pmc_field* f, const Geo& g, int n, const double* tau, const int* minexp,
                      const CompMeta* hm, int codec, int done, int next, FieldJob* job) {
  const std::unique_ptr<pmc_store> s(store_from_meta(f, g, n, tau, minexp, hm, job->region, codec));
  ProfScope ps(ctx, f->dtype == PMC_F32 ? "k_decode_tiles_f32" : "k_decode_tiles_f64");
  hipError_t e = hipSuccess;
  for (int i0 = done, i1; i0 < next && e == hipSuccess; i0 = i1) {
    i1 = std::min(i0 + kMaxDecode, next);
    e = f->dtype == PMC_F32 ? decode_tiles<float>(s.get(), i0, i1, i0 == 0, job, ctx->stream)
                            : decode_tiles<double>(s.get(), i0, i1, i0 == 0, job, ctx->stream);
  }
  return e;
}

// pmc_compress's workspace: one field's, and its components' results
static uint64_t single_workspace(const pmc_field* f, const Geo& g, int n) {
  return job_workspace(f, g, n) + align256((uint64_t)n * sizeof(CompMeta));
}

}  // namespace pmc_host

// ---- the static workspace of pmc_compress_static --------------------------
// One buffer per GPU, held until the process ends.  Host code never uses the
// array's name as an address (on the host it names a stand-in, not device
// memory): pmc_ctx_create looks up its device address once per device with
// hipGetSymbolAddress, and only that address is passed on.
static_assert(PMC_STATIC_WS_BYTES % 256 == 0, "static workspace size");
static_assert(kPinBytes >= kRangeGroups * kRangeWords * 8, "the pinned buffer holds every partial of the range");
static_assert(kPinBytes >= kMaxComps * sizeof(CompMeta), "the pinned buffer holds every component's metadata");
static __device__ __align__(256) uint8_t scratch[PMC_STATIC_WS_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// device address of `scratch` on `device`, looked up on the first call for
// that device (with the device current; the caller's current device is
// restored afterwards)
hipError_t scratch_setup(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  int prev = 0;
  hipError_t e = hipGetDevice(&prev);
  if (e != hipSuccess) return e;
  if ((e = hipSetDevice(device)) != hipSuccess) return e;
  void* p = nullptr;
  e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  const hipError_t r = hipSetDevice(prev);
  if (e != hipSuccess) return e;
  if (r != hipSuccess) return r;
  if (!p) return hipErrorInvalidSymbol;
  g_scratch_ptr[device] = p;
  return hipSuccess;
}

void* scratch_ptr(int device) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  return device >= 0 && device < kMaxDevices ? g_scratch_ptr[device] : nullptr;
}
}  // namespace

extern "C" {

pmc_status pmc_ctx_create(int device, void* hip_stream, pmc_ctx** out) {
  if (!out) return PMC_E_ARG;
  int count = 0;
  hipError_t e = hipGetDeviceCount(&count);
  if (e != hipSuccess || device < 0 || device >= count) return PMC_E_DEVICE;
  if (scratch_setup(device) != hipSuccess) return PMC_E_DEVICE;
  pmc_ctx* c = new pmc_ctx();
  c->device = device;
  c->stream = (hipStream_t)hip_stream;
  // the pinned readback buffer, allocated with the context's device current
  // (the caller's current device is restored afterwards)
  int prev = 0;
  if (hipGetDevice(&prev) == hipSuccess && hipSetDevice(device) == hipSuccess) {
    if (hipHostMalloc(&c->pin, kPinBytes, hipHostMallocDefault) != hipSuccess) c->pin = nullptr;
    (void)hipSetDevice(prev);
  }
  *out = c;
  return PMC_OK;
}

// copy `bytes` of device memory to host `dst` on the context stream and wait
// for it, through the context's pinned buffer when it holds them
static hipError_t read_back(pmc_ctx* ctx, void* dst, const void* src, size_t bytes) {
  void* via = ctx->pin && bytes <= kPinBytes ? ctx->pin : dst;
  hipError_t e = hipMemcpyAsync(via, src, bytes, hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e == hipSuccess && via != dst) std::memcpy(dst, via, bytes);
  return e;
}

void pmc_ctx_destroy(pmc_ctx* ctx) {
  if (!ctx) return;
  if (!ctx->prof_pending.empty()) (void)hipStreamSynchronize(ctx->stream);
  for (auto& r : ctx->prof_pending) {
    (void)hipEventDestroy(r.start);
    (void)hipEventDestroy(r.stop);
  }
  for (auto e : ctx->prof_pool) (void)hipEventDestroy(e);
  if (ctx->pin) {
    (void)hipStreamSynchronize(ctx->stream);
    (void)hipHostFree(ctx->pin);
  }
  delete ctx;
}

pmc_status pmc_prof_read(pmc_ctx* ctx, pmc_prof_entry* out, int cap, int* n, int reset) {
  if (!ctx) return PMC_E_ARG;
  if (!ctx->prof_pending.empty()) {
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hipfail(ctx, e, "sync");
    for (auto& r : ctx->prof_pending) {
      float ms = 0.0f;
      if (hipEventElapsedTime(&ms, r.start, r.stop) == hipSuccess) {
        ctx->prof_ms[r.kernel] += ms;
        ctx->prof_launches[r.kernel] += 1;
      }
      ctx->prof_pool.push_back(r.start);
      ctx->prof_pool.push_back(r.stop);
    }
    ctx->prof_pending.clear();
  }
  const int k = (int)ctx->prof_names.size();
  if (n) *n = k;
  for (int i = 0; i < k && i < cap && out; ++i) {
    std::memset(&out[i], 0, sizeof(out[i]));
    std::snprintf(out[i].name, sizeof(out[i].name), "%s", ctx->prof_names[i].c_str());
    out[i].launches = ctx->prof_launches[i];
    out[i].ms = ctx->prof_ms[i];
  }
  if (reset) {
    for (int i = 0; i < k; ++i) {
      ctx->prof_launches[i] = 0;
      ctx->prof_ms[i] = 0.0;
    }
  }
  return PMC_OK;
}

const char* pmc_last_error(const pmc_ctx* ctx) { return ctx ? ctx->err.c_str() : ""; }

pmc_status pmc_ctx_set_option(pmc_ctx* ctx, int option, int value) {
  if (!ctx) return PMC_E_ARG;
  if (option == PMC_OPT_FUSED_DECODE) ctx->fused_decode = value ? 1 : 0;
  else if (option == PMC_OPT_SYNC_CHECK) ctx->sync_check = value ? 1 : 0;
  else if (option == PMC_OPT_PROFILE) ctx->profile = value ? 1 : 0;
  else if (option == PMC_OPT_CODEC) {
    if (value != 0 && value != 1) return fail(ctx, PMC_E_ARG, "codec must be 0 or 1");
    ctx->codec = value;
  }
  else return fail(ctx, PMC_E_ARG, "unknown option %d", option);
  return PMC_OK;
}

pmc_status pmc_range(pmc_ctx* ctx, const pmc_field* f, const void* d_x, void* d_ws, size_t ws_bytes,
                     double* vmin, double* vmax, uint64_t* nonfinite) {
  if (!ctx) return PMC_E_ARG;
  Geo g;
  if (!make_geo(f, &g) || !d_x) return fail(ctx, PMC_E_ARG, "bad field");
  if (!d_ws || ws_bytes < 256) return fail(ctx, PMC_E_NOMEM, "range needs 256 bytes of workspace");
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return hipfail(ctx, e, "hipSetDevice");
  const uint64_t n = g.nx * g.ny * g.nz;
  // the workgroups' partials go straight to the context's pinned buffer (the
  // device writes host memory), or into the workspace where there is none
  void* dev_pin = nullptr;
  if (!ctx->pin || hipHostGetDevicePointer(&dev_pin, ctx->pin, 0) != hipSuccess) dev_pin = nullptr;
  const uint64_t part = kRangeWords * 8;
  unsigned long long* w = (unsigned long long*)(dev_pin ? dev_pin : d_ws);
  const uint32_t groups = range_groups(n, (dev_pin ? kPinBytes : ws_bytes) / part);
  if (f->dtype == PMC_F32) e = launch_range<float>((const float*)d_x, n, w, groups, ctx->stream);
  else e = launch_range<double>((const double*)d_x, n, w, groups, ctx->stream);
  if (e != hipSuccess) return hipfail(ctx, e, "range kernel");
  std::vector<unsigned long long> hp;
  const unsigned long long* p = (const unsigned long long*)ctx->pin;
  if (!dev_pin) {
    hp.resize(kRangeWords * (size_t)groups);
    p = hp.data();
    e = hipMemcpyAsync(hp.data(), w, groups * part, hipMemcpyDeviceToHost, ctx->stream);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hipfail(ctx, e, "range read");
  unsigned long long h[3] = {~0ull, 0ull, 0ull};
  for (uint32_t i = 0; i < groups; ++i) {
    h[0] = std::min(h[0], p[kRangeWords * i]);
    h[1] = std::max(h[1], p[kRangeWords * i + 1]);
    h[2] += p[kRangeWords * i + 2];
  }
  auto unorder = [](unsigned long long o) {
    uint64_t b = (o >> 63) ? (o & 0x7FFFFFFFFFFFFFFFull) : ~o;
    double v;
    std::memcpy(&v, &b, 8);
    return v;
  };
  if (nonfinite) *nonfinite = h[2];
  if (h[2] == n) {  // nothing finite
    if (vmin) *vmin = NAN;
    if (vmax) *vmax = NAN;
  } else {
    if (vmin) *vmin = unorder(h[0]);
    if (vmax) *vmax = unorder(h[1]);
  }
  return PMC_OK;
}

size_t pmc_stats_ws_bytes(void) { return (size_t)sum_sq_ws_bytes() + 256; }

pmc_status pmc_accuracy_gain(pmc_ctx* ctx, const pmc_field* f, const void* d_x, const void* d_xt, double rate,
                             void* d_ws, size_t ws_bytes, double out[3]) {
  if (!ctx) return PMC_E_ARG;
  Geo g;
  if (!make_geo(f, &g) || !d_x || !d_xt || !out) return fail(ctx, PMC_E_ARG, "bad field or null pointer");
  if (!d_ws || ws_bytes < pmc_stats_ws_bytes())
    return fail(ctx, PMC_E_NOMEM, "accuracy gain needs %llu bytes of workspace",
                (unsigned long long)pmc_stats_ws_bytes());
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return hipfail(ctx, e, "hipSetDevice");
  const uint64_t n = g.nx * g.ny * g.nz;
  double* ws = (double*)d_ws;
  double* res = (double*)((uint8_t*)d_ws + sum_sq_ws_bytes());
  // one sum pass: (shift, with xt?) -> host pair
  auto pass = [&](const void* b, double shift, double h[2]) -> pmc_status {
    hipError_t r;
    if (f->dtype == PMC_F32)
      r = launch_sum_sq<float>((const float*)d_x, (const float*)b, shift, n, ws, res, ctx->stream);
    else
      r = launch_sum_sq<double>((const double*)d_x, (const double*)b, shift, n, ws, res, ctx->stream);
    if (r != hipSuccess) return hipfail(ctx, r, "sum kernel");
    if ((r = hipMemcpyAsync(h, res, 16, hipMemcpyDeviceToHost, ctx->stream)) != hipSuccess)
      return hipfail(ctx, r, "copy");
    if ((r = hipStreamSynchronize(ctx->stream)) != hipSuccess) return hipfail(ctx, r, "sync");
    return PMC_OK;
  };
  double h[2];
  pmc_status st;
  if ((st = pass(nullptr, 0.0, h)) != PMC_OK) return st;
  const double mean = h[0] / (double)n;
  if ((st = pass(nullptr, mean, h)) != PMC_OK) return st;  // second pass about the mean
  const double sigma = std::sqrt(h[1] / (double)n);
  if ((st = pass(d_xt, 0.0, h)) != PMC_OK) return st;
  const double rmse = std::sqrt(h[1] / (double)n);
  out[0] = sigma;
  out[1] = rmse;
  out[2] = std::log2(sigma / rmse) - rate;
  return PMC_OK;
}

pmc_status pmc_cast_compress(pmc_ctx* ctx, const pmc_field* f, const void* d_x, int n, float* d_comps, void* d_ws,
                             size_t ws_bytes, double* linf) {
  if (!ctx) return PMC_E_ARG;
  Geo g;
  if (!make_geo(f, &g) || !d_x || !d_comps) return fail(ctx, PMC_E_ARG, "bad field or null pointer");
  if (n < 1 || n > kMaxComps) return fail(ctx, PMC_E_ARG, "n must be in [1, %d]", kMaxComps);
  if (!d_ws || ws_bytes < 8 * (size_t)kMaxComps)
    return fail(ctx, PMC_E_NOMEM, "cast compression needs %d bytes of workspace", 8 * kMaxComps);
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return hipfail(ctx, e, "hipSetDevice");
  const uint64_t N = g.nx * g.ny * g.nz;
  unsigned long long* lb = (unsigned long long*)d_ws;
  if ((e = launch_fill64(lb, (uint64_t)n, 0ull, ctx->stream)) != hipSuccess) return hipfail(ctx, e, "fill");
  if (f->dtype == PMC_F32) e = launch_cast_encode<float>((const float*)d_x, N, n, d_comps, lb, ctx->stream);
  else e = launch_cast_encode<double>((const double*)d_x, N, n, d_comps, lb, ctx->stream);
  if (e != hipSuccess) return hipfail(ctx, e, "cast encode");
  if (linf) {
    std::vector<unsigned long long> h(n);
    if ((e = hipMemcpyAsync(h.data(), lb, 8 * (size_t)n, hipMemcpyDeviceToHost, ctx->stream)) != hipSuccess)
      return hipfail(ctx, e, "copy");
    if ((e = hipStreamSynchronize(ctx->stream)) != hipSuccess) return hipfail(ctx, e, "sync");
    for (int i = 0; i < n; ++i) std::memcpy(&linf[i], &h[i], 8);
  }
  return PMC_OK;
}

pmc_status pmc_cast_retrieve(pmc_ctx* ctx, const pmc_field* f, const float* d_comps, int k, void* d_out) {
  if (!ctx) return PMC_E_ARG;
  Geo g;
  if (!make_geo(f, &g) || !d_comps || !d_out) return fail(ctx, PMC_E_ARG, "bad field or null pointer");
  if (k < 0 || k > kMaxComps) return fail(ctx, PMC_E_ARG, "k must be in [0, %d]", kMaxComps);
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return hipfail(ctx, e, "hipSetDevice");
  const uint64_t N = g.nx * g.ny * g.nz;
  if (f->dtype == PMC_F32) e = launch_cast_decode<float>(d_comps, N, k, (float*)d_out, ctx->stream);
  else e = launch_cast_decode<double>(d_comps, N, k, (double*)d_out, ctx->stream);
  if (e != hipSuccess) return hipfail(ctx, e, "cast decode");
  return PMC_OK;
}

pmc_status pmc_compress_sizes(const pmc_field* f, int n, size_t* ws_bytes, size_t* stream_cap_per_comp) {
  Geo g;
  if (!make_geo(f, &g) || n < 1 || n > kMaxComps) return PMC_E_ARG;
  if (ws_bytes) *ws_bytes = single_workspace(f, g, n);
  if (stream_cap_per_comp) *stream_cap_per_comp = aux_bytes(g) + align256(stream_cap_one(g, f->dtype));
  return PMC_OK;
}

pmc_status pmc_compress(pmc_ctx* ctx, const pmc_field* f, const void* d_x, int n, const double* tau, void* d_ws,
                        size_t ws_bytes, void* d_streams, size_t streams_cap, pmc_store** out) {
  if (!ctx) return PMC_E_ARG;
  if (out) *out = nullptr;
  Geo g;
  if (!make_geo(f, &g)) return fail(ctx, PMC_E_ARG, "bad field");
  if (!d_x || !tau || !out || !d_streams) return fail(ctx, PMC_E_ARG, "null argument");
  if (!aligned16(d_x)) return fail(ctx, PMC_E_ARG, "d_x must be 16-byte aligned");
  if (n < 1 || n > kMaxComps) return fail(ctx, PMC_E_ARG, "n must be in [1, %d]", kMaxComps);
  const int codec = ctx->codec;
  for (int i = 0; i < n; ++i) {
    if (!(tau[i] > 0.0) || !std::isfinite(tau[i])) return fail(ctx, PMC_E_ARG, "tau[%d] must be > 0 and finite", i);
    if (i > 0 && !(tau[i] < tau[i - 1])) return fail(ctx, PMC_E_ARG, "tau must be strictly decreasing");
    // the prediction codec keeps every bin 2 tau 2^-d normal and 1 / (2 tau) finite
    if (codec == 1 && !(tau[i] >= std::ldexp(1.0, -960) && tau[i] <= std::ldexp(1.0, 1000)))
      return fail(ctx, PMC_E_ARG, "tau[%d] outside [2^-960, 2^1000], the prediction codec's range", i);
  }
  const uint64_t ws_need = single_workspace(f, g, n);
  if (!d_ws || ws_bytes < ws_need)
    return fail(ctx, PMC_E_NOMEM, "workspace too small: need %llu bytes", (unsigned long long)ws_need);
  // the per-block indexes sit at the front of d_streams and are written by
  // the encoder directly; the streams themselves are capacity-checked on the
  // device before they are packed
  const uint64_t min_cap = (uint64_t)n * aux_bytes(g) + (uint64_t)n * align256(kStreamHeader + 4 * g.nchunks);
  if (streams_cap < min_cap)
    return fail(ctx, PMC_E_NOMEM, "stream capacity too small: need at least %llu bytes",
                (unsigned long long)min_cap);
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return hipfail(ctx, e, "hipSetDevice");
  const uint64_t auxb = aux_bytes(g);
  FieldJob job{};
  const uint64_t meta_bytes = align256((uint64_t)n * sizeof(CompMeta));
  if (!job_layout(f, g, n, false, (uint8_t*)d_ws, ws_need - meta_bytes, &job))
    return fail(ctx, PMC_E_NOMEM, "workspace too small for its layout");
  job.meta = (CompMeta*)((uint8_t*)d_ws + ws_need - meta_bytes);
  job.x = d_x;
  job.region = (uint8_t*)d_streams;
  job.region_cap = streams_cap;
  job.aux_stride = auxb / 4;
  job.codec = (uint8_t)codec;
  std::vector<int> minexp(n);
  for (int i = 0; i < n; ++i) {
    minexp[i] = floor_log2(tau[i]);
    job.tau[i] = tau[i];
    job.minexp[i] = minexp[i];
  }
  // the per-component results also go straight to the pinned buffer
  void* dev_pin = nullptr;
  if (!ctx->pin || hipHostGetDevicePointer(&dev_pin, ctx->pin, 0) != hipSuccess) dev_pin = nullptr;
  job.host_meta = (CompMeta*)dev_pin;
  std::vector<CompMeta> hm(n);
  // components [c0, c1) in one launch of the encoder and one of each pack kernel
  auto run = [&](int c0, int c1) {
    job.comp0 = (uint8_t)c0;
    job.comp1 = (uint8_t)c1;
    hipError_t r;
    {
      ProfScope ps(ctx, f->dtype == PMC_F32 ? (codec == 0 ? "k_encode_f32" : "k_encode_pq_f32")
                                            : (codec == 0 ? "k_encode_f64" : "k_encode_pq_f64"));
      r = f->dtype == PMC_F32 ? launch_encode<float>(job, ctx->stream) : launch_encode<double>(job, ctx->stream);
    }
    if (r != hipSuccess) return r;
    ProfScope ps(ctx, f->dtype == PMC_F32 ? "k_pack_f32" : "k_pack_f64");
    return launch_pack(job, ctx->stream);
  };
  auto results = [&]() {
    hipError_t r;
    if (!dev_pin) return read_back(ctx, hm.data(), job.meta, n * sizeof(CompMeta));
    if ((r = hipStreamSynchronize(ctx->stream)) != hipSuccess) return r;
    std::memcpy(hm.data(), ctx->pin, n * sizeof(CompMeta));
    return hipSuccess;
  };
  if ((e = run(0, n)) != hipSuccess) return hipfail(ctx, e, "encode");
  if ((e = results()) != hipSuccess) return hipfail(ctx, e, "meta read");
  // Where components of some wave outgrow its slot together, those before the
  // first that does not fit stand; the next launch goes on from there, with x~
  // decoded from them.  Each launch adds to them, as a slot holds any one
  // component (28 components at 149 bits per value, 128^3 float32: 0.65 ms; all components again, one launch each,
  // took 1.52).
  for (int done = 0, next; (next = first_over(hm.data(), done, n)) < n; done = next) {
    unsigned int bad = hm[0].flags & FLAG_NONFINITE;
    for (int i = done; i < next; ++i) bad |= hm[i].flags & (FLAG_OVERFLOW | FLAG_INDEX);
    if (bad & (FLAG_NONFINITE | FLAG_INDEX)) break;
    if (!job_layout(f, g, n, true, (uint8_t*)d_ws, ws_need - meta_bytes, &job))
      return fail(ctx, PMC_E_NOMEM, "workspace too small for its layout");
    if (bad) {
      // the stream buffer is too small for the components before: one launch
      // each, for the size to report, x~ from the encoder itself
      for (int i = 0; i < n; ++i)
        if ((e = run(i, i + 1)) != hipSuccess) return hipfail(ctx, e, "encode");
      if ((e = results()) != hipSuccess) return hipfail(ctx, e, "meta read");
      break;
    }
    if (next == done) return fail(ctx, PMC_E_DEVICE, "component %d outgrew its staging slot", next);
    e = resume_job(ctx, f, g, n, tau, minexp.data(), hm.data(), codec, done, next, &job);
    if (e == hipSuccess) e = run(next, n);
    if (e != hipSuccess) return hipfail(ctx, e, "encode");
    if ((e = results()) != hipSuccess) return hipfail(ctx, e, "meta read");
  }

  unsigned int flags = 0;
  unsigned long long misses = 0;
  for (int i = 0; i < n; ++i) {
    flags |= hm[i].flags;
    misses += hm[i].nmiss;
  }
  if (flags & FLAG_NONFINITE) return fail(ctx, PMC_E_NONFINITE, "input holds NaN or Inf");
  if (flags & FLAG_INDEX) return fail(ctx, PMC_E_NOMEM, "a stream exceeds 2^32 payload words");
  if (flags & FLAG_OVERFLOW) {
    unsigned long long need = n * auxb;
    for (int i = 0; i < n; ++i) need = align256(need) + hm[i].stream_bytes;
    return fail(ctx, PMC_E_NOMEM, "stream capacity too small: need %llu bytes", need);
  }
  pmc_store* s = store_from_meta(f, g, n, tau, minexp.data(), hm.data(), (const uint8_t*)d_streams, codec);
  *out = s;
  if (misses) return fail(ctx, PMC_E_BOUND, "%llu blocks missed their tolerance", misses);
  return PMC_OK;
}

pmc_status pmc_compress_static(pmc_ctx* ctx, const pmc_field* f, const void* d_x, int n, const double* tau,
                               void* d_streams, size_t streams_cap, pmc_store** out) {
  if (!ctx) return PMC_E_ARG;
  if (out) *out = nullptr;
  Geo g;
  if (!make_geo(f, &g)) return fail(ctx, PMC_E_ARG, "bad field");
  if (n < 1 || n > kMaxComps) return fail(ctx, PMC_E_ARG, "n must be in [1, %d]", kMaxComps);
  const uint64_t need = single_workspace(f, g, n);
  if (need > PMC_STATIC_WS_BYTES)
    return fail(ctx, PMC_E_NOMEM,
                "field needs %llu bytes of workspace; the static workspace holds %llu (use pmc_compress "
                "with a caller workspace)",
                (unsigned long long)need, (unsigned long long)PMC_STATIC_WS_BYTES);
  void* ws = scratch_ptr(ctx->device);
  if (!ws) return fail(ctx, PMC_E_DEVICE, "static workspace not set up on device %d", ctx->device);
  // the same kernels as pmc_compress; every workspace word they read is
  // written first in the same call, so nothing of an earlier call carries over
  return pmc_compress(ctx, f, d_x, n, tau, ws, PMC_STATIC_WS_BYTES, d_streams, streams_cap, out);
}

pmc_status pmc_store_info(const pmc_store* s, int* n, double* tau, double* linf, uint64_t* bytes, uint64_t* nraw,
                          uint64_t* nesc) {
  if (!s) return PMC_E_ARG;
  if (n) *n = s->n;
  for (int i = 0; i < s->n; ++i) {
    if (tau) tau[i] = s->tau[i];
    if (linf) linf[i] = s->linf[i];
    if (bytes) bytes[i] = s->bytes[i];
    if (nraw) nraw[i] = s->nraw[i];
    if (nesc) nesc[i] = s->nesc[i];
  }
  return PMC_OK;
}

pmc_status pmc_store_codec(const pmc_store* s, int* codec) {
  if (!s || !codec) return PMC_E_ARG;
  *codec = s->codec;
  return PMC_OK;
}

pmc_status pmc_store_counts(const pmc_store* s, int i, uint64_t counts[5]) {
  if (!s || !counts || i < 0 || i >= s->n) return PMC_E_ARG;
  counts[0] = s->nempty[i];
  counts[1] = s->ncoded[i];
  counts[2] = s->nraw[i];
  counts[3] = s->nesc[i];
  counts[4] = s->nmiss[i];
  return PMC_OK;
}

pmc_status pmc_store_span(const pmc_store* s, int i, uint64_t* max_span_words, int* staged) {
  if (!s || i < 0 || i >= s->n) return PMC_E_ARG;
  if (max_span_words) *max_span_words = s->max_span[i];
  if (staged) *staged = s->max_span[i] <= stage_words() ? 1 : 0;
  return PMC_OK;
}

pmc_status pmc_store_decode_route(const pmc_store* s, int i, int* high_half) {
  if (!s || !high_half || i < 0 || i >= s->n) return PMC_E_ARG;
  *high_half = s->f.dtype == PMC_F32 && s->codec == 0 && s->full[i] == 0 ? 1 : 0;
  return PMC_OK;
}

pmc_status pmc_store_field(const pmc_store* s, pmc_field* f) {
  if (!s || !f) return PMC_E_ARG;
  *f = s->f;
  return PMC_OK;
}

pmc_status pmc_store_stream(const pmc_store* s, int i, const void** d_stream, uint64_t* bytes) {
  if (!s || i < 0 || i >= s->n) return PMC_E_ARG;
  if (d_stream) *d_stream = s->d_base + s->offset[i];
  if (bytes) *bytes = s->bytes[i];
  return PMC_OK;
}

pmc_status pmc_select_k(const pmc_store* s, double tol, int use_measured, int* k) {
  if (!s || !k) return PMC_E_ARG;
  for (int i = 0; i < s->n; ++i) {
    const double v = use_measured ? s->linf[i] : s->tau[i];
    if (v <= tol) {
      *k = i + 1;
      return PMC_OK;
    }
  }
  *k = 0;
  return PMC_E_UNREACHABLE;
}

size_t pmc_decode_ws_bytes(void) { return 256; }

static pmc_status decode_range(pmc_ctx* ctx, const pmc_store* s, int k0, int k1, const void* d_in, void* d_out,
                               void* d_ws, size_t ws_bytes) {
  if (!d_ws || ws_bytes < pmc_decode_ws_bytes()) return fail(ctx, PMC_E_NOMEM, "decode needs 256 bytes of workspace");
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return hipfail(ctx, e, "hipSetDevice");
  unsigned int* status = (unsigned int*)d_ws;
  // the kernels only ever set the status word; it is cleared, and read,
  // when the call checks it
  if (ctx->sync_check && (e = launch_fill64((unsigned long long*)status, 1, 0ull, ctx->stream)) != hipSuccess)
    return hipfail(ctx, e, "status init");
  const uint64_t waves = (s->g.nblocks + 63) / 64;
  const void* in = d_in;
  for (int i0 = k0, i1; i0 < k1; i0 = i1) {
    SplitArgs sp;
    const SplitArgs* psp = ctx->fused_decode && split_plan(s, i0, k1, waves, false, &i1, &sp) ? &sp : nullptr;
    if (!psp) i1 = std::min(i0 + (ctx->fused_decode ? kMaxDecode : 1), k1);
    uint64_t span = 0;
    for (int i = i0; i < i1; ++i) span = std::max(span, s->max_span[i]);
    const bool hires = high_half(s, i0, i1) && (i0 > 0 || !in);
    if (s->f.dtype == PMC_F32) {
      DecArgs<float> a{};
      fill_decode_args(s, i0, i1, a);
      a.in = (const float*)in;
      a.out = (float*)d_out;
      a.g = s->g;
      a.status = status;
      ProfScope ps(ctx, s->codec == 0 ? "k_decode_f32" : "k_decode_pq_f32");
      e = launch_decode<float>(a, span, s->codec, hires, psp, ctx->stream);
    } else {
      DecArgs<double> a{};
      fill_decode_args(s, i0, i1, a);
      a.in = (const double*)in;
      a.out = (double*)d_out;
      a.g = s->g;
      a.status = status;
      ProfScope ps(ctx, s->codec == 0 ? "k_decode_f64" : "k_decode_pq_f64");
      e = launch_decode<double>(a, span, s->codec, hires, psp, ctx->stream);
    }
    if (e != hipSuccess) return hipfail(ctx, e, "decode");
    in = d_out;
  }
  if (ctx->sync_check) {
    unsigned int h = 0;
    if ((e = read_back(ctx, &h, status, 4)) != hipSuccess) return hipfail(ctx, e, "status read");
    if (h) return fail(ctx, PMC_E_CORRUPT, "malformed stream");
  }
  return PMC_OK;
}

pmc_status pmc_retrieve_box(pmc_ctx* ctx, const pmc_store* s, int k, const uint64_t lo[3], const uint64_t hi[3],
                            void* d_out, void* d_ws, size_t ws_bytes) {
  if (!ctx) return PMC_E_ARG;
  if (!s || !d_out || !lo || !hi) return fail(ctx, PMC_E_ARG, "null argument");
  if (k < 1 || k > s->n) return fail(ctx, PMC_E_ARG, "k must be in [1, %d]", s->n);
  const uint64_t dims[3] = {s->g.nx, s->g.ny, s->g.nz};
  for (int a = 0; a < 3; ++a)
    if (!(lo[a] < hi[a] && hi[a] <= dims[a])) return fail(ctx, PMC_E_ARG, "box axis %d outside the field", a);
  if (!d_ws || ws_bytes < pmc_decode_ws_bytes()) return fail(ctx, PMC_E_NOMEM, "decode needs 256 bytes of workspace");
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return hipfail(ctx, e, "hipSetDevice");
  unsigned int* status = (unsigned int*)d_ws;
  // the kernels only ever set the status word; it is cleared, and read,
  // when the call checks it
  if (ctx->sync_check && (e = launch_fill64((unsigned long long*)status, 1, 0ull, ctx->stream)) != hipSuccess)
    return hipfail(ctx, e, "status init");
  BoxArgs b{};
  for (int a = 0; a < 3; ++a) {
    b.lo[a] = lo[a];
    b.hi[a] = hi[a];
    b.blo[a] = lo[a] / 4;
    b.bhi[a] = (hi[a] + 3) / 4;
  }
  // a row of blocks meets at most this many waves; where the field's rows
  // start on a wave's first block, as many as the first row does
  const uint64_t nbx = b.bhi[0] - b.blo[0];
  const bool whole = s->g.nbx % 64 == 0;
  b.waves_per_row = (uint32_t)(whole ? (b.blo[0] % 64 + nbx + 63) / 64 : (nbx + 63) / 64 + 1);
  const uint64_t waves = (b.bhi[1] - b.blo[1]) * (b.bhi[2] - b.blo[2]) * b.waves_per_row;
  const void* in = nullptr;
  for (int i0 = 0, i1; i0 < k; i0 = i1) {
    SplitArgs sp;
    const SplitArgs* psp = split_plan(s, i0, k, waves, true, &i1, &sp) ? &sp : nullptr;
    if (!psp) i1 = std::min(i0 + kMaxDecode, k);
    uint64_t span = 0;
    for (int i = i0; i < i1; ++i) span = std::max(span, s->max_span[i]);
    const bool hires = high_half(s, i0, i1);
    if (s->f.dtype == PMC_F32) {
      DecArgs<float> a{};
      fill_decode_args(s, i0, i1, a);
      a.in = (const float*)in;
      a.out = (float*)d_out;
      a.g = s->g;
      a.status = status;
      e = launch_decode_box<float>(a, b, span, s->codec, hires, psp, ctx->stream);
    } else {
      DecArgs<double> a{};
      fill_decode_args(s, i0, i1, a);
      a.in = (const double*)in;
      a.out = (double*)d_out;
      a.g = s->g;
      a.status = status;
      e = launch_decode_box<double>(a, b, span, s->codec, hires, psp, ctx->stream);
    }
    if (e != hipSuccess) return hipfail(ctx, e, "decode");
    in = d_out;
  }
  if (ctx->sync_check) {
    unsigned int h = 0;
    if ((e = read_back(ctx, &h, status, 4)) != hipSuccess) return hipfail(ctx, e, "status read");
    if (h) return fail(ctx, PMC_E_CORRUPT, "malformed stream");
  }
  return PMC_OK;
}

pmc_status pmc_retrieve(pmc_ctx* ctx, const pmc_store* s, int k, void* d_out, void* d_ws, size_t ws_bytes) {
  if (!ctx) return PMC_E_ARG;
  if (!s || !d_out) return fail(ctx, PMC_E_ARG, "null argument");
  if (!aligned16(d_out)) return fail(ctx, PMC_E_ARG, "d_out must be 16-byte aligned");
  if (k < 1 || k > s->n) return fail(ctx, PMC_E_ARG, "k must be in [1, %d]", s->n);
  return decode_range(ctx, s, 0, k, nullptr, d_out, d_ws, ws_bytes);
}

pmc_status pmc_refine(pmc_ctx* ctx, const pmc_store* s, int k_from, int k_to, void* d_inout, void* d_ws,
                      size_t ws_bytes) {
  if (!ctx) return PMC_E_ARG;
  if (!s || !d_inout) return fail(ctx, PMC_E_ARG, "null argument");
  if (!aligned16(d_inout)) return fail(ctx, PMC_E_ARG, "d_inout must be 16-byte aligned");
  if (k_from < 0 || k_to > s->n || k_from > k_to) return fail(ctx, PMC_E_ARG, "bad component range");
  if (k_from == k_to) return PMC_OK;
  return decode_range(ctx, s, k_from, k_to, k_from == 0 ? nullptr : d_inout, d_inout, d_ws, ws_bytes);
}

// ---- persistence -----------------------------------------------------------
pmc_status pmc_store_serialize(pmc_ctx* ctx, const pmc_store* s, void* host_buf, size_t cap, size_t* used) {
  if (!ctx) return PMC_E_ARG;
  if (!s || !used) return fail(ctx, PMC_E_ARG, "null argument");
  uint64_t region = 0;
  for (int i = 0; i < s->n; ++i) region = align256(region) + s->bytes[i];
  const uint64_t total = blob_header_bytes(s->n) + align256(region);
  *used = total;
  if (!host_buf) return PMC_OK;
  if (cap < total) return fail(ctx, PMC_E_NOMEM, "need %llu bytes", (unsigned long long)total);
  uint8_t* b = (uint8_t*)host_buf;
  std::memset(b, 0, total);
  uint32_t h32[4] = {kBlobMagic, 1u, (uint32_t)s->n, (uint32_t)s->codec};
  std::memcpy(b, h32, 16);
  uint64_t dims[3] = {s->f.nx, s->f.ny, s->f.nz};
  std::memcpy(b + 16, dims, 24);
  int32_t dt[2] = {s->f.dtype, 0};
  std::memcpy(b + 40, dt, 8);
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return hipfail(ctx, e, "hipSetDevice");
  uint64_t off = 0;
  for (int i = 0; i < s->n; ++i) {
    uint8_t* c = b + 48 + 64ull * i;
    uint64_t v[8];
    std::memcpy(&v[0], &s->tau[i], 8);
    std::memcpy(&v[1], &s->linf[i], 8);
    v[2] = s->bytes[i];
    v[3] = s->nempty[i];
    v[4] = s->ncoded[i];
    v[5] = s->nraw[i];
    v[6] = s->nesc[i];
    v[7] = s->nmiss[i];
    std::memcpy(c, v, 64);
    off = align256(off);
    e = hipMemcpyAsync(b + blob_header_bytes(s->n) + off, s->d_base + s->offset[i], s->bytes[i],
                       hipMemcpyDeviceToHost, ctx->stream);
    if (e != hipSuccess) return hipfail(ctx, e, "stream copy");
    off += s->bytes[i];
  }
  if ((e = hipStreamSynchronize(ctx->stream)) != hipSuccess) return hipfail(ctx, e, "sync");
  return PMC_OK;
}

pmc_status pmc_store_deserialize(pmc_ctx* ctx, const void* host_buf, size_t size, void* d_streams, size_t cap,
                                 pmc_store** out) {
  if (!ctx) return PMC_E_ARG;
  if (!out || !d_streams) return fail(ctx, PMC_E_ARG, "null argument");
  *out = nullptr;
  BlobView v;
  if (!parse_blob(host_buf, size, &v)) return fail(ctx, PMC_E_CORRUPT, "malformed store blob");
  Geo g;
  if (!make_geo(&v.f, &g)) return fail(ctx, PMC_E_CORRUPT, "bad field in blob");
  const uint64_t auxb = aux_bytes(g);
  const uint64_t need = blob_device_bytes(v, g);
  if (cap < need) return fail(ctx, PMC_E_NOMEM, "need %llu bytes", (unsigned long long)need);
  const uint8_t* region = (const uint8_t*)host_buf + v.region_off;
  std::vector<uint64_t> words, spans;
  if (!check_blob_streams(v, g, region, &words, &spans)) return fail(ctx, PMC_E_CORRUPT, "malformed stream");
  pmc_store* s = new pmc_store();
  s->f = v.f;
  s->g = g;
  s->n = v.n;
  s->codec = v.codec;
  s->d_base = (const uint8_t*)d_streams;
  uint64_t off = 0;
  for (int i = 0; i < v.n; ++i) {
    const uint64_t* r = &v.rec[8 * i];
    double tau, linf;
    std::memcpy(&tau, &r[0], 8);
    std::memcpy(&linf, &r[1], 8);
    off = align256(off);
    s->tau.push_back(tau);
    s->linf.push_back(linf);
    s->minexp.push_back(floor_log2(tau));
    s->bytes.push_back(r[2]);
    s->offset.push_back(v.n * auxb + off);
    s->aux_offset.push_back(i * auxb);
    s->words.push_back(words[i]);
    s->nempty.push_back(r[3]);
    s->ncoded.push_back(r[4]);
    s->nraw.push_back(r[5]);
    s->nesc.push_back(r[6]);
    s->nmiss.push_back(r[7]);
    s->max_span.push_back(spans[i]);
    off += r[2];
  }
  hipError_t e = hipSetDevice(ctx->device);
  uint8_t* base = (uint8_t*)d_streams;
  // after the streams: a status word, set by the index rebuild when a
  // chunk's payload does not parse, then one flag per component, set when a
  // coded block is outside the float32 high-half decode route
  unsigned int* status = (unsigned int*)(base + need - kBlobTrailerBytes);
  unsigned long long* full = (unsigned long long*)(base + need - kBlobTrailerBytes) + 1;
  if (e == hipSuccess) e = launch_fill64((unsigned long long*)status, 1 + (uint64_t)v.n, 0ull, ctx->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(base + v.n * auxb, region, v.region_bytes, hipMemcpyHostToDevice, ctx->stream);
  // rebuild the per-block index of every stream
  AuxArgs a{};
  uint64_t span = 0;
  for (int i = 0; i < v.n; ++i) {
    a.s[i] = base + s->offset[i];
    a.aux[i] = (uint32_t*)(base + s->aux_offset[i]);
    a.words[i] = s->words[i];
    a.minexp[i] = s->minexp[i];
    span = std::max(span, spans[i]);
  }
  a.g = g;
  a.status = status;
  a.full = full;
  if (e == hipSuccess)
    e = s->f.dtype == PMC_F32 ? launch_aux<float>(a, v.n, span, s->codec, ctx->stream)
                              : launch_aux<double>(a, v.n, span, s->codec, ctx->stream);
  unsigned long long trailer[1 + kMaxComps] = {};
  if (e == hipSuccess)
    e = hipMemcpyAsync(trailer, status, 8 * (1 + (size_t)v.n), hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  const unsigned int h = (unsigned int)(trailer[0] & 0xFFFFFFFFull);
  for (int i = 0; i < v.n; ++i) s->full.push_back(trailer[1 + i]);
  if (e != hipSuccess) {
    delete s;
    return hipfail(ctx, e, "stream upload");
  }
  if (h) {
    delete s;
    return fail(ctx, PMC_E_CORRUPT, "a chunk's payload does not parse");
  }
  *out = s;
  return PMC_OK;
}

void pmc_store_free(pmc_store* s) { delete s; }

}  // extern "C"
