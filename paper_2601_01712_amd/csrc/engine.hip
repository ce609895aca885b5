// C-ABI entry points and the host side of the relay-race path: validation, the per-call row
// plan, scratch carving and the fixed kernel sequence of a layer.  Declarations and argument
// contracts are in include/relaygr.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/relaygr.h"
#include "attention.h"
#include "common.h"
#include "errors.h"
#include "fp32.h"
#include "gemm.h"
#include "gemm_bf16.h"
#include "kv_pool.h"
#include "rowwise.h"
#include "staging.h"

using namespace relaygr;

// ---- errors -----------------------------------------------------------------------------------
static thread_local char g_err[512] = "";

int relaygr::fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

#define HIP_TRY(expr)                                                                          \
  do {                                                                                         \
    hipError_t e_ = (expr);                                                                    \
    if (e_ != hipSuccess) return fail(RELAYGR_EHIP, "%s: %s", #expr, hipGetErrorString(e_));   \
  } while (0)

#define LAUNCH_CHECK(name)                                                                     \
  do {                                                                                         \
    hipError_t e_ = hipGetLastError();                                                         \
    if (e_ != hipSuccess) return fail(RELAYGR_EHIP, "launch %s: %s", name, hipGetErrorString(e_)); \
  } while (0)

extern "C" const char* relaygr_last_error(void) { return g_err; }

// ---- config -----------------------------------------------------------------------------------
static inline bool is_half16(const relaygr_model_config& c) { return c.dtype == RELAYGR_DTYPE_BF16 || c.dtype == RELAYGR_DTYPE_FP16; }

static bool config_ok(const relaygr_model_config* c) {
  if (!c) return false;
  if (c->n_layers < 1 || c->n_heads < 1 || c->d_model < 64) return false;
  if (c->dtype != RELAYGR_DTYPE_FP32 && c->dtype != RELAYGR_DTYPE_BF16 && c->dtype != RELAYGR_DTYPE_FP16) return false;
  int d = c->d_model;
  if (d != 64 && d != 128 && d != 256 && d != 512 && d != 1024) return false;
  if (d % c->n_heads) return false;
  int dh = d / c->n_heads;
  if (dh != 32 && dh != 64 && dh != 128) return false;
  if (dh < d / 64) return false;                       // a head must span at least one lane in row-wise kernels
  if (is_half16(*c) && d < 128) return false;  // the MFMA GEMM tiles 128 output columns
  if (!(c->ln_eps > 0.f)) return false;
  return true;
}

static inline size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

extern "C" size_t relaygr_kv_footprint_bytes(const relaygr_model_config* cfg, int32_t prefix_len) {
  if (!config_ok(cfg) || prefix_len < 0) return 0;
  return (size_t)2 * cfg->n_layers * (size_t)prefix_len * cfg->d_model * elem_bytes(*cfg);
}

extern "C" size_t relaygr_kv_pool_bytes_for(const relaygr_model_config* cfg, int32_t prefix_len, int32_t page_tokens) {
  if (!config_ok(cfg) || prefix_len < 0 || page_tokens < kTile || page_tokens % kTile) return 0;
  size_t pages = ((size_t)prefix_len + page_tokens - 1) / page_tokens;
  return pages * (size_t)2 * cfg->n_layers * page_tokens * cfg->d_model * elem_bytes(*cfg);
}

// ---- per-call plan ----------------------------------------------------------------------------
struct Plan {
  int n_users = 0;
  int n_prows = 0, n_nrows = 0, n_rows = 0;
  int64_t sfx_tiles = 0, kvs_tiles = 0;   // suffix tiles / recomputed-prefix tiles held in scratch
  int n_tiles = 0;      // attention work items (16-bit: pieces, the last layer's list by itself)
  int nsplit = 1;       // attention partial sums a row can have (fp32: has)
  // byte offsets into scratch
  size_t off_x, off_xh, off_u, off_q, off_knew, off_vnew, off_sfx, off_kvs, off_part, off_ml, off_rows, off_blob;
  size_t blob_bytes = 0;
  size_t total = 0;
};

// Rows per attention work item: 32 (fp32: one wavefront), or 128 * nq for the 16-bit kernel, nq in {1, 2}.
static int rows_per_attn_tile(const relaygr_model_config& c, int nq) { return c.dtype == RELAYGR_DTYPE_FP32 ? 32 : 128 * nq; }

// Lays the call's buffers out in scratch.  Everything is a function of the counts already in p.
// Bytes at the start of scratch that hold the weights re-packed into MFMA panels (bf16 only).
static size_t wpack_bytes(const relaygr_model_config& c) {
  if (!is_half16(c)) return 0;
  const size_t d = c.d_model;
  return align_up((size_t)c.n_layers * 5 * d * d * 2);
}

// Prefix rows of a user start at a multiple of this in the row space (bf16: GEMM tiles of 256 rows
// never straddle users, and 32-row MFMA blocks coincide with 32-token halves of K/V tiles).
static int prefix_row_align(const relaygr_model_config& c) { return is_half16(c) ? kPrefixRowAlign : 1; }

static void carve(const relaygr_model_config& c, Plan& p) {
  const size_t d = c.d_model, e = elem_bytes(c), R = p.n_rows;
  const size_t Rp = (R + 255) / 256 * 256;     // the bf16 GEMMs read whole 256-row tiles of xh
  size_t o = 0;   // offsets are relative to the call scratch, which follows the packed weights in a context's buffer
  auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
  p.off_x = take(R * d * 4);
  p.off_xh = take(Rp * d * e);
  p.off_u = take(R * d * e);
  p.off_q = take(R * d * e);
  p.off_knew = take((size_t)p.n_nrows * d * e);
  p.off_vnew = take((size_t)p.n_nrows * d * e);
  p.off_sfx = take((size_t)p.sfx_tiles * 2 * kTile * d * e);
  p.off_kvs = take((size_t)p.kvs_tiles * 2 * kTile * d * e);
  p.off_part = take((size_t)p.nsplit * R * d * 4);
  p.off_ml = take((size_t)p.nsplit * R * c.n_heads * 2 * 4);   // softmax form: (m, l) per row, head and split
  p.off_rows = take(6 * align_up(R * 4));
  p.blob_bytes = align_up((size_t)p.n_users * sizeof(UserDesc)) + 2 * align_up((size_t)(p.n_users + 1) * 4) +
                 align_up((size_t)p.n_tiles * sizeof(AttnTile));
  p.off_blob = take(p.blob_bytes);
  p.total = o;
}

// fp32: a work item is one wavefront over its part of the keys, and 2048 of them (two a SIMD) fill the chip.  As long as the
// items alone leave SIMDs idle (under 1024), a workgroup's eight wavefronts share an item's keys (gs = 8), and what is
// still missing comes from splits of the key range (at most 8, at least one 32-key half tile per wavefront in the mean).
static void fp32_splits(int64_t items, int64_t half_tiles, int* nsplit, int* gs) {
  *nsplit = 1;
  *gs = items < 1024 ? kF32Team : 1;
  if (items <= 0 || *gs == 1) return;
  const int64_t by_chip = 2048 / (items * kF32Team), by_keys = half_tiles / (items * kF32Team);
  *nsplit = (int)std::max<int64_t>(1, std::min<int64_t>({by_chip, by_keys, 8}));
}

extern "C" size_t relaygr_scratch_bytes(const relaygr_model_config* cfg, int32_t max_users,
                                        int64_t max_prefix_tokens, int64_t max_new_tokens) {
  if (!config_ok(cfg) || max_users < 1 || max_prefix_tokens < 0 || max_new_tokens < 0) return 0;
  if (max_prefix_tokens + max_new_tokens >= (1ll << 31)) return 0;
  Plan p;
  p.n_users = max_users;
  int64_t padded = max_prefix_tokens + (int64_t)max_users * (prefix_row_align(*cfg) - 1);
  if (padded + max_new_tokens >= (1ll << 31)) return 0;
  p.n_prows = (int)padded;
  p.n_nrows = (int)max_new_tokens;
  p.n_rows = p.n_prows + p.n_nrows;
  p.sfx_tiles = max_new_tokens / kTile + max_users;
  p.kvs_tiles = max_prefix_tokens / kTile + max_users;
  int rpt = rows_per_attn_tile(*cfg, 1);
  const int tiles_new = (int)(max_new_tokens / rpt) + max_users, tiles_prefix = (int)(padded / rpt) + max_users;
  p.n_tiles = 2 * tiles_new + tiles_prefix + 2 * max_cut_items(cfg->n_heads);   // the last layer's list too, and room for the items that are cut into pieces
  p.nsplit = 1;
  carve(*cfg, p);
  size_t base = wpack_bytes(*cfg) + p.total;
  // head-room so that small calls may split their key range 8 ways
  size_t small_rows = std::min<size_t>((size_t)p.n_rows, 8192);
  return base + align_up(small_rows * 7 * ((size_t)cfg->d_model * 4 + (size_t)cfg->n_heads * 8));
}

// ---- scratch that lives in the library (for callers that cannot allocate) ----------------------
// relaygr_rank_with_cache_static lays its call out here instead of in the context's buffer.  Each GPU holds
// its own copy of the array at its own address; in host code the array's name is only a stand-in, so the
// device address is looked up once per device (hipGetSymbolAddress, with that device current) and that
// pointer is what kernels, copies and fills are given.
constexpr size_t kStaticScratchBytes = RELAYGR_STATIC_SCRATCH_BYTES;
// Room beside it for the descriptors (64-byte work items, in two lists, and six row tables: at most 132 bytes a row), so that
// they take nothing from what a call's rows may use: 16-bit d = 128, where rows are smallest, fits 30 000 rows in 64 MiB.
constexpr size_t kStaticDescriptorBytes = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kStaticDescriptorBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_static_mu;
static char* g_static_ptr[kMaxDevices] = {};
// Calls on the shared array are kept apart on the GPU like a context's calls on its own scratch: a call on another
// stream than the last one waits for what that stream holds (order_behind; the event is created with the address).
static hipEvent_t g_static_done[kMaxDevices] = {};
static hipStream_t g_static_last_stream[kMaxDevices] = {};
static bool g_static_has_call[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up on that device's first use.
static int static_scratch(char** out, int* dev_out = nullptr) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(RELAYGR_EINVAL, "static scratch: device index %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_static_mu);
  if (!g_static_ptr[dev]) {
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(RELAYGR_EHIP, "static scratch: hipGetSymbolAddress returned a null address");
    HIP_TRY(hipEventCreateWithFlags(&g_static_done[dev], hipEventDisableTiming));
    g_static_ptr[dev] = (char*)ptr;
  }
  *out = g_static_ptr[dev];
  if (dev_out) *dev_out = dev;
  return RELAYGR_OK;
}

// ---- context ----------------------------------------------------------------------------------
constexpr int kStagingSlots = 4;
constexpr size_t kInlineBlobBytes = 128 << 10, kSlotFlagBytes = 256;   // batches whose descriptors the first kernel fetches itself
static_assert(kInlineBlobBytes / kBlobChunk * 4 <= kSlotFlagBytes, "a flag per chunk");

// Whether a stream has work left, asked in a way that is safe next to another stream's capture.
static StreamState stream_state(hipStream_t st) {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) { (void)hipGetLastError(); return StreamState::kBusy; }
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(st, &cap);
  const bool captured = e == hipSuccess && cap != hipStreamCaptureStatusNone;   // (a question would end the capture)
  if (e == hipSuccess && !captured) e = hipStreamQuery(st);
  if (e != hipSuccess) (void)hipGetLastError();      // the answer, not an error of the call that asks
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (captured) return StreamState::kBusy;
  switch (e) {
    case hipErrorNotReady: case hipErrorStreamCaptureUnsupported: case hipErrorStreamCaptureImplicit: return StreamState::kBusy;
    case hipSuccess: case hipErrorInvalidHandle: case hipErrorContextIsDestroyed: case hipErrorInvalidValue: return StreamState::kDrained;   // (the others: destroyed by its owner)
    default: return StreamState::kFailed;
  }
}

struct StagingSlot {
  void* host = nullptr;       // pinned: flags of the kernel that reads the slot, then the descriptors
  size_t bytes = 0;           // of descriptors
  hipEvent_t done = nullptr;
  bool pending = false;       // a copy command may still read it: `done` follows
  uint32_t seq = 0;           // calls whose first kernel has read (or will read) it
  int chunks = 0;             // workgroups of the last of them, each of which sets its flag to seq
  uint32_t* flags() const { return (uint32_t*)host; }
  hipStream_t stream = nullptr;   // where that kernel is
  // Waits for that kernel: it is on its stream (chunks is 0 otherwise).  False: it will not come (wait_for_flags).
  bool wait_read() {
    if (chunks == 0) return true;
    const hipStream_t st = stream;
    if (!wait_for_flags(flags(), chunks, seq, [st] { return stream_state(st); })) return false;
    chunks = 0;
    return true;
  }
  char* blob() const { return (char*)host + kSlotFlagBytes; }
};

struct ProfRec { int cls; hipEvent_t a, b; };

struct relaygr_ctx {
  uint32_t prof_mask = 0;
  int prof_every = 1;                   // time the launches of every n-th call only
  int64_t prof_calls = 0;
  bool prof_this_call = true;
  std::vector<ProfRec> prof_recs;       // recorded, not yet resolved
  std::vector<hipEvent_t> prof_free;    // events ready for reuse
  double prof_ms[RELAYGR_K_COUNT] = {};
  int64_t prof_n[RELAYGR_K_COUNT] = {};
  relaygr_model_config cfg;
  int attn_form = RELAYGR_ATTN_SILU;
  std::vector<relaygr_layer_weights> layers;
  const void *ln_out_g, *ln_out_b, *w_score;
  float b_score;
  char* scratch;                        // the caller's buffer: [packed weights | call scratch]
  size_t scratch_bytes;
  std::vector<const uint16_t*> w1_packed, w2_packed;   // bf16: panels at the start of scratch
  int n_cus = 256;                      // compute units of the device the context was created on
  StagingSlot staging[kStagingSlots];   // pinned, allocated once at creation
  void* staging_mem = nullptr;          // of all slots
  int next_slot = 0;
  // A context's calls share its scratch, so they must not overlap on the GPU.  On one stream they cannot; a call
  // on another stream than the one before it is made to wait for what that stream holds (order_behind).
  hipEvent_t call_done = nullptr;
  hipStream_t last_stream = nullptr;
  bool has_call = false;
  std::mutex mu;                        // one host thread at a time plans and enqueues a call of this context
};

// Device memory one call lays its buffers out in (the part of a context's buffer behind the packed weights).
struct CallScratch { char* base; size_t bytes; };

extern "C" int relaygr_ctx_create(const relaygr_model_config* cfg, const relaygr_weights* w, void* scratch_dev,
                                  size_t scratch_bytes, relaygr_ctx** out) {
  if (!out) return fail(RELAYGR_EINVAL, "ctx_create: out is null");
  *out = nullptr;
  if (!config_ok(cfg)) return fail(RELAYGR_EINVAL, "ctx_create: unsupported model config");
  if (!w || !w->layers || !w->ln_out_g || !w->ln_out_b || !w->w_score) return fail(RELAYGR_EINVAL, "ctx_create: null weights");
  if (!scratch_dev || ((uintptr_t)scratch_dev & 255)) return fail(RELAYGR_EINVAL, "ctx_create: scratch null or not 256-byte aligned");
  for (int l = 0; l < cfg->n_layers; ++l) {
    const relaygr_layer_weights& lw = w->layers[l];
    if (!lw.ln_in_g || !lw.ln_in_b || !lw.w1 || !lw.b1 || !lw.ln_at_g || !lw.ln_at_b || !lw.w2 || !lw.b2)
      return fail(RELAYGR_EINVAL, "ctx_create: layer %d has a null parameter", l);
  }
  relaygr_ctx* c = new (std::nothrow) relaygr_ctx();
  if (!c) return fail(RELAYGR_EINVAL, "ctx_create: out of host memory");
  c->cfg = *cfg;
  c->layers.assign(w->layers, w->layers + cfg->n_layers);
  c->ln_out_g = w->ln_out_g; c->ln_out_b = w->ln_out_b; c->w_score = w->w_score; c->b_score = w->b_score;
  c->scratch = (char*)scratch_dev;
  c->scratch_bytes = scratch_bytes;
  {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
      c->n_cus = cus;
  }
  if (scratch_bytes < wpack_bytes(*cfg)) { delete c; return fail(RELAYGR_ENOSPC, "ctx_create: scratch smaller than the packed weights"); }
  if (is_half16(*cfg)) {
    // re-pack W1 and W2 of every layer into MFMA panels, once
    const size_t d = cfg->d_model;
    uint16_t* wp = (uint16_t*)scratch_dev;
    for (int l = 0; l < cfg->n_layers; ++l) {
      uint16_t* w1p = wp + (size_t)l * 5 * d * d;
      uint16_t* w2p = w1p + 4 * d * d;
      int c1 = (int)(4 * d * d / 8), c2 = (int)(d * d / 8);
      hipLaunchKernelGGL(pack_weight_kernel, dim3((c1 + 255) / 256), dim3(256), 0, 0, (const uint16_t*)c->layers[l].w1,
                         (uint16_t*)w1p, (int)(4 * d), (int)d);
      hipLaunchKernelGGL(pack_weight16_kernel, dim3((c2 + 255) / 256), dim3(256), 0, 0, (const uint16_t*)c->layers[l].w2,
                         (uint16_t*)w2p, (int)d);
      c->w1_packed.push_back(w1p);
      c->w2_packed.push_back(w2p);
    }
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) { delete c; return fail(RELAYGR_EHIP, "ctx_create: packing weights: %s", hipGetErrorString(e)); }
  }
  // Pinned staging for the per-call descriptor blob, sized once from what the scratch buffer can hold: a call
  // has at most one row per d*(8 + 3e) bytes of call scratch (residual stream, one partial sum, normalised row, u and q), one
  // attention work item per 32 (16-bit: 128, in two lists, and the pieces of a cut list) rows plus two per user, and a buffer sized by relaygr_scratch_bytes for max_users holds
  // two K/V tiles per user; calls beyond that are refused (RELAYGR_ENOSPC), so no compute call allocates.
  {
    const size_t call_bytes = scratch_bytes - wpack_bytes(*cfg);
    const size_t d = cfg->d_model, e = elem_bytes(*cfg);
    const size_t rows_est = call_bytes / (d * (8 + 3 * e)) + 1;
    const size_t users_est = std::min<size_t>(call_bytes / (4 * kTile * d * e) + 1, 1 << 16);
    const size_t cut = max_cut_items(cfg->n_heads);
    const size_t tiles_est = is_half16(*cfg) ? std::max(rows_est / 128 + 2 * users_est, cut) + std::max(rows_est / 128 + users_est, cut) : rows_est / 32 + 2 * users_est;
    const size_t want = align_up(users_est * sizeof(UserDesc)) + 2 * align_up((users_est + 1) * 4) + align_up(tiles_est * sizeof(AttnTile));
    // (one allocation for all slots: each costs a few hundred microseconds)
    const size_t each = align_up(kSlotFlagBytes + want);
    hipError_t e1 = hipHostMalloc(&c->staging_mem, kStagingSlots * each, hipHostMallocDefault);
    for (int k = 0; k < kStagingSlots && e1 == hipSuccess; ++k) {
      StagingSlot& sl = c->staging[k];
      sl.host = (char*)c->staging_mem + k * each;
      sl.bytes = want;
      memset(sl.host, 0, kSlotFlagBytes);
      e1 = hipEventCreateWithFlags(&sl.done, hipEventDisableTiming);
    }
    if (e1 != hipSuccess) {
      relaygr_ctx_destroy(c);
      return fail(RELAYGR_EHIP, "ctx_create: pinned staging of %d x %zu bytes: %s", kStagingSlots, each, hipGetErrorString(e1));
    }
  }
  {
    hipError_t e = hipEventCreateWithFlags(&c->call_done, hipEventDisableTiming);
    if (e != hipSuccess) { relaygr_ctx_destroy(c); return fail(RELAYGR_EHIP, "ctx_create: event: %s", hipGetErrorString(e)); }
  }
  {   // set-up for relaygr_rank_with_cache_static: this device's address of the library's own scratch
    char* unused = nullptr;
    int rc = static_scratch(&unused);
    if (rc != RELAYGR_OK) { relaygr_ctx_destroy(c); return rc; }
  }
  *out = c;
  return RELAYGR_OK;
}

extern "C" int relaygr_ctx_set_attention(relaygr_ctx* c, int32_t form) {
  if (!c) return fail(RELAYGR_EINVAL, "ctx_set_attention: null context");
  if (form != RELAYGR_ATTN_SILU && form != RELAYGR_ATTN_SOFTMAX) return fail(RELAYGR_EINVAL, "ctx_set_attention: unknown form %d", form);
  c->attn_form = form;
  return RELAYGR_OK;
}

extern "C" void relaygr_ctx_destroy(relaygr_ctx* c) {
  if (!c) return;
  for (auto& r : c->prof_recs) { (void)hipEventSynchronize(r.b); (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
  for (auto e : c->prof_free) (void)hipEventDestroy(e);
  bool read = true;   // (memory that a kernel may still read is not given back)
  for (auto& s : c->staging) {
    read = s.wait_read() && read;
    if (s.done) { if (s.pending) (void)hipEventSynchronize(s.done); (void)hipEventDestroy(s.done); }
  }
  if (c->staging_mem && read) (void)hipHostFree(c->staging_mem);
  if (c->call_done) (void)hipEventDestroy(c->call_done);
  delete c;
}

// Pinned staging for the descriptor blob: a ring of slots allocated at context creation, each guarded by an
// event, or by flags that the kernel reading it sets, so that a slot is not rewritten while an earlier call may still read it.
// The only host wait of a compute call is here: when the call kStagingSlots calls ago has not read its slot yet.
static int staging_acquire(relaygr_ctx* c, size_t bytes, StagingSlot** out) {
  StagingSlot& s = c->staging[c->next_slot];
  if (s.bytes < bytes)
    return fail(RELAYGR_ENOSPC, "batch descriptors need %zu bytes of staging, the context holds %zu (sized from its scratch buffer: "
                "too many users or row tiles for one call)", bytes, s.bytes);
  c->next_slot = (c->next_slot + 1) % kStagingSlots;
  if (s.pending) { HIP_TRY(hipEventSynchronize(s.done)); s.pending = false; }
  if (!s.wait_read())
    return fail(RELAYGR_EHIP, "the kernel that reads an earlier call's descriptors has not run: the stream it was put on failed");
  *out = &s;
  return RELAYGR_OK;
}

// ---- per-kernel timing ------------------------------------------------------------------------
struct ProfScope {
  relaygr_ctx* c; int cls; hipStream_t st; hipEvent_t a = nullptr, b = nullptr;
  ProfScope(relaygr_ctx* c_, int cls_, hipStream_t st_) : c(c_), cls(cls_), st(st_) {
    if (!(c->prof_mask & (1u << cls)) || !c->prof_this_call) return;
    auto get = [&]() -> hipEvent_t {
      hipEvent_t e = nullptr;
      if (!c->prof_free.empty()) { e = c->prof_free.back(); c->prof_free.pop_back(); }
      else if (hipEventCreate(&e) != hipSuccess) e = nullptr;
      return e;
    };
    a = get(); b = get();
    if (a && b) (void)hipEventRecord(a, st);
  }
  ~ProfScope() {
    if (!a || !b) return;
    (void)hipEventRecord(b, st);
    c->prof_recs.push_back({cls, a, b});
  }
};

static int prof_resolve(relaygr_ctx* c) {
  for (auto& r : c->prof_recs) {
    HIP_TRY(hipEventSynchronize(r.b));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, r.a, r.b));
    c->prof_ms[r.cls] += ms;
    c->prof_n[r.cls] += 1;
    c->prof_free.push_back(r.a);
    c->prof_free.push_back(r.b);
  }
  c->prof_recs.clear();
  return RELAYGR_OK;
}

extern "C" int relaygr_ctx_profile_enable(relaygr_ctx* c, uint32_t class_mask) {
  if (!c) return fail(RELAYGR_EINVAL, "profile_enable: null context");
  int rc = prof_resolve(c);
  if (rc != RELAYGR_OK) return rc;
  c->prof_mask = class_mask & ((1u << RELAYGR_K_COUNT) - 1);
  for (int k = 0; k < RELAYGR_K_COUNT; ++k) { c->prof_ms[k] = 0.0; c->prof_n[k] = 0; }
  return RELAYGR_OK;
}

extern "C" int relaygr_ctx_profile_sample(relaygr_ctx* c, int32_t every_n_calls) {
  if (!c || every_n_calls < 1) return fail(RELAYGR_EINVAL, "profile_sample: null context or every_n_calls < 1");
  c->prof_every = every_n_calls;
  c->prof_calls = 0;
  return RELAYGR_OK;
}

extern "C" int relaygr_ctx_profile_read(relaygr_ctx* c, int32_t cls, double* total_ms, int64_t* launches) {
  if (!c || cls < 0 || cls >= RELAYGR_K_COUNT) return fail(RELAYGR_EINVAL, "profile_read: bad argument");
  int rc = prof_resolve(c);
  if (rc != RELAYGR_OK) return rc;
  if (total_ms) *total_ms = c->prof_ms[cls];
  if (launches) *launches = c->prof_n[cls];
  return RELAYGR_OK;
}

// ---- pool ABI ---------------------------------------------------------------------------------
extern "C" int relaygr_kv_pool_create(const relaygr_model_config* cfg, void* slab_dev, size_t slab_bytes,
                                      int32_t page_tokens, relaygr_kv_pool** out) {
  if (!out) return fail(RELAYGR_EINVAL, "kv_pool_create: out is null");
  *out = nullptr;
  if (!config_ok(cfg)) return fail(RELAYGR_EINVAL, "kv_pool_create: unsupported model config");
  if (!slab_dev || ((uintptr_t)slab_dev & 255)) return fail(RELAYGR_EINVAL, "kv_pool_create: slab null or not 256-byte aligned");
  if (page_tokens < kTile || page_tokens % kTile) return fail(RELAYGR_EINVAL, "kv_pool_create: page_tokens must be a positive multiple of 64");
  size_t page_bytes = (size_t)2 * cfg->n_layers * page_tokens * cfg->d_model * elem_bytes(*cfg);
  int64_t n_pages = (int64_t)(slab_bytes / page_bytes);
  if (n_pages < 1) return fail(RELAYGR_ENOSPC, "kv_pool_create: slab smaller than one page (%zu bytes)", page_bytes);
  if (n_pages * (int64_t)page_tokens >= (1ll << 31)) return fail(RELAYGR_EINVAL, "kv_pool_create: slab holds 2^31 tokens or more");
  KvPool* p = new (std::nothrow) KvPool();
  if (!p) return fail(RELAYGR_EINVAL, "kv_pool_create: out of host memory");
  p->cfg = *cfg;
  p->slab = slab_dev;
  p->slab_bytes = slab_bytes;
  p->page_tokens = page_tokens;
  p->n_pages = n_pages;
  p->layer_stride = (int64_t)2 * kTile * cfg->d_model;
  p->tile_stride = p->layer_stride * cfg->n_layers;
  p->free_extents[0] = n_pages;
  *out = reinterpret_cast<relaygr_kv_pool*>(p);
  return RELAYGR_OK;
}

extern "C" void relaygr_kv_pool_destroy(relaygr_kv_pool* pool) { delete reinterpret_cast<KvPool*>(pool); }

extern "C" int relaygr_kv_pool_alloc(relaygr_kv_pool* pool, uint64_t user_id, int32_t prefix_len, relaygr_kv_handle* out) {
  if (!pool || !out) return fail(RELAYGR_EINVAL, "kv_pool_alloc: null argument");
  int rc = reinterpret_cast<KvPool*>(pool)->alloc(user_id, prefix_len, out);
  if (rc == RELAYGR_ENOSPC) return fail(rc, "kv_pool_alloc: no free extent for %d tokens", prefix_len);
  if (rc != RELAYGR_OK) return fail(rc, "kv_pool_alloc: prefix_len < 1 or user %llu already has a live entry", (unsigned long long)user_id);
  return rc;
}

extern "C" int relaygr_kv_pool_free(relaygr_kv_pool* pool, relaygr_kv_handle h) {
  if (!pool) return fail(RELAYGR_EINVAL, "kv_pool_free: null pool");
  int rc = reinterpret_cast<KvPool*>(pool)->release(h);
  if (rc != RELAYGR_OK) return fail(rc, "kv_pool_free: stale or unknown handle");
  return rc;
}

extern "C" int relaygr_kv_pool_lookup(relaygr_kv_pool* pool, uint64_t user_id, relaygr_kv_handle* out) {
  if (!pool || !out) return fail(RELAYGR_EINVAL, "kv_pool_lookup: null argument");
  int rc = reinterpret_cast<KvPool*>(pool)->lookup(user_id, out);
  if (rc != RELAYGR_OK) return fail(rc, "kv_pool_lookup: user %llu has no live entry", (unsigned long long)user_id);
  return rc;
}

extern "C" int relaygr_kv_pool_entry_len(relaygr_kv_pool* pool, relaygr_kv_handle h, int32_t* prefix_len) {
  if (!pool || !prefix_len) return fail(RELAYGR_EINVAL, "kv_pool_entry_len: null argument");
  PoolEntry e;
  int rc = reinterpret_cast<KvPool*>(pool)->resolve(h, &e);
  if (rc != RELAYGR_OK) return fail(rc, "kv_pool_entry_len: stale or unknown handle");
  *prefix_len = e.prefix_len;
  return RELAYGR_OK;
}

extern "C" int relaygr_kv_pool_stats(relaygr_kv_pool* pool, int64_t* total, int64_t* free_pages, int64_t* live, int64_t* largest) {
  if (!pool) return fail(RELAYGR_EINVAL, "kv_pool_stats: null pool");
  reinterpret_cast<KvPool*>(pool)->stats(total, free_pages, live, largest);
  return RELAYGR_OK;
}

extern "C" int relaygr_kv_pool_locate(relaygr_kv_pool* pool, relaygr_kv_handle h, int32_t layer, int32_t token,
                                      int32_t feature, int64_t* k_index, int64_t* v_index) {
  if (!pool || !k_index || !v_index) return fail(RELAYGR_EINVAL, "kv_pool_locate: null argument");
  KvPool* p = reinterpret_cast<KvPool*>(pool);
  PoolEntry e;
  int rc = p->resolve(h, &e);
  if (rc != RELAYGR_OK) return fail(rc, "kv_pool_locate: stale or unknown handle");
  if (layer < 0 || layer >= p->cfg.n_layers || token < 0 || token >= e.prefix_len || feature < 0 || feature >= p->cfg.d_model)
    return fail(RELAYGR_EINVAL, "kv_pool_locate: index out of range");
  int dh = p->cfg.d_model / p->cfg.n_heads;
  int head = feature / dh, f = feature % dh;
  int64_t tile = e.page0 * (p->page_tokens / kTile) + token / kTile;
  int r = token % kTile;
  int64_t base = tile * p->tile_stride + (int64_t)layer * p->layer_stride + (int64_t)head * 2 * kTile * dh;
  if (p->cfg.dtype == RELAYGR_DTYPE_FP32) {
    *k_index = base + KvLayout<float>::k_off(r, f, dh);
    *v_index = base + KvLayout<float>::v_off(r, f, dh);
  } else {
    *k_index = base + KvLayout16::k_off(r, f, dh);
    *v_index = base + KvLayout16::v_off(r, f, dh);
  }
  return RELAYGR_OK;
}

// ---- the layer sequence -----------------------------------------------------------------------
enum Mode { kPrefill, kRankCached, kRankFull };

template <typename F>
static inline bool dispatch_e(int d, F&& f) {
  switch (d / 64) {
    case 1: f(std::integral_constant<int, 1>()); return true;
    case 2: f(std::integral_constant<int, 2>()); return true;
    case 4: f(std::integral_constant<int, 4>()); return true;
    case 8: f(std::integral_constant<int, 8>()); return true;
    case 16: f(std::integral_constant<int, 16>()); return true;
  }
  return false;
}

template <typename T>
static int launch_attention(const relaygr_model_config& cfg, const AttnParams& ap, int n_tiles, int nq, bool softmax, hipStream_t st);   // ap.gs: groups per workgroup

template <bool SM>
static int launch_attention_f32(const relaygr_model_config& cfg, const AttnParams& ap, int n_tiles, hipStream_t st) {
  const int items = n_tiles * cfg.n_heads * ap.nsplit, wgs = ap.gs > 1 ? items : (items + kF32Team - 1) / kF32Team;
  dim3 grid((wgs + 7) / 8 * 8);
  switch (cfg.d_model / cfg.n_heads) {
    case 32: hipLaunchKernelGGL((attn_f32_kernel<32, SM>), grid, dim3(kF32Team * 64), 0, st, ap); break;
    case 64: hipLaunchKernelGGL((attn_f32_kernel<64, SM>), grid, dim3(kF32Team * 64), 0, st, ap); break;
    case 128: hipLaunchKernelGGL((attn_f32_kernel<128, SM>), grid, dim3(kF32Team * 64), 0, st, ap); break;
    default: return fail(RELAYGR_EINVAL, "attention: unsupported d_head");
  }
  LAUNCH_CHECK("attn_f32");
  return RELAYGR_OK;
}
template <>
int launch_attention<float>(const relaygr_model_config& cfg, const AttnParams& ap, int n_tiles, int, bool softmax, hipStream_t st) {
  return softmax ? launch_attention_f32<true>(cfg, ap, n_tiles, st) : launch_attention_f32<false>(cfg, ap, n_tiles, st);
}

template <typename H, bool SM>
static int launch_attention16(const relaygr_model_config& cfg, const AttnParams& ap, int n_tiles, int nq, hipStream_t st) {
  const int nh = cfg.n_heads;
  dim3 grid(nh >= 8 ? n_tiles * nh : (n_tiles + 8 / nh - 1) / (8 / nh) * 8);   // the kernel's order of heads and items
  switch (cfg.d_model / cfg.n_heads) {
    case 32: hipLaunchKernelGGL((attn_bf16_kernel<H, 32, 1, 4, SM>), grid, dim3(256), 0, st, ap); break;
    case 64:
      if (nq == 2 && ap.gs == 2) hipLaunchKernelGGL((attn_bf16_kernel<H, 64, 2, 4, SM, 2>), grid, dim3(512), 0, st, ap);
      else if (ap.gs == 2) hipLaunchKernelGGL((attn_bf16_kernel<H, 64, 1, 4, SM, 2>), grid, dim3(512), 0, st, ap);
      else if (nq == 2) hipLaunchKernelGGL((attn_bf16_kernel<H, 64, 2, 4, SM>), grid, dim3(256), 0, st, ap);
      else hipLaunchKernelGGL((attn_bf16_kernel<H, 64, 1, 4, SM>), grid, dim3(256), 0, st, ap);
      break;
    case 128:
      // 256-row items: eight wavefronts of 32 rows.  With four of 64 rows a lane needs 458 registers, so that the scores come out of accumulation
      // registers one move each and a SIMD has one wavefront; with eight it needs 212, without moves, and two share a SIMD: 262 -> 240 k cycles.  The
      // fragments are read from LDS twice as often, and the clock sinks with the load, so that less of it shows (us a call at d = 1024, 512 candidates
      // each, four / eight wavefronts: 16 users of 1000 keys 1381 / 1367, of 4096 2069 / 2058 and 2144 / 2159 on another card, of 8000 3070 / 3033; 24 of
      // 4000 3437 / 3351, of 12 000 6646 / 6679; 40 of 1000 3655 / 3569, of 2000 in the softmax form 4414 / 4285; full recompute of 12 000 keys 3962 / 3854).
      if (nq == 2) hipLaunchKernelGGL((attn_bf16_kernel<H, 128, 1, 8, SM>), grid, dim3(512), 0, st, ap);
      else hipLaunchKernelGGL((attn_bf16_kernel<H, 128, 1, 4, SM>), grid, dim3(256), 0, st, ap);
      break;
    default: return fail(RELAYGR_EINVAL, "attention: unsupported d_head");
  }
  LAUNCH_CHECK("attn (16-bit)");
  return RELAYGR_OK;
}
template <>
int launch_attention<__hip_bfloat16>(const relaygr_model_config& cfg, const AttnParams& ap, int n_tiles, int nq, bool softmax, hipStream_t st) {
  return softmax ? launch_attention16<Bf16, true>(cfg, ap, n_tiles, nq, st) : launch_attention16<Bf16, false>(cfg, ap, n_tiles, nq, st);
}
template <>
int launch_attention<__half>(const relaygr_model_config& cfg, const AttnParams& ap, int n_tiles, int nq, bool softmax, hipStream_t st) {
  return softmax ? launch_attention16<F16, true>(cfg, ap, n_tiles, nq, st) : launch_attention16<F16, false>(cfg, ap, n_tiles, nq, st);
}

static int check_offsets(const int32_t* off, int n, const char* what) {
  if (!off) return RELAYGR_OK;
  if (off[0] != 0) return fail(RELAYGR_EINVAL, "%s offsets must start at 0", what);
  for (int i = 0; i < n; ++i)
    if (off[i + 1] < off[i]) return fail(RELAYGR_EINVAL, "%s offsets not monotone at user %d", what, i);
  return RELAYGR_OK;
}

template <typename T>
static int run_typed(relaygr_ctx* c, KvPool* pool, const relaygr_batch* b, Mode mode, float* scores, const CallScratch& cs, hipStream_t st, bool capturing) {
  const relaygr_model_config& cfg = c->cfg;
  const int d = cfg.d_model, H = cfg.n_heads, dh = d / H, NL = cfg.n_layers, n = b->n_users;
  const bool bf16 = is_half16(cfg);   // either 16-bit type: the MFMA path
  using HT = typename HalfOf<T>::type;
  const int palign = prefix_row_align(cfg);

  // -- per-user shapes and K/V sources
  std::vector<UserDesc> users(n);
  std::vector<int32_t> pstart(n + 1, 0), nstart(n + 1, 0);
  Plan p;
  p.n_users = n;
  int64_t prow = 0, nrow = 0, sfx_tiles = 0, kvs_tiles = 0;
  for (int u = 0; u < n; ++u) {
    UserDesc& ud = users[u];
    memset(&ud, 0, sizeof(ud));
    int L = b->prefix_off ? b->prefix_off[u + 1] - b->prefix_off[u] : 0;
    int S = (mode != kPrefill && b->suffix_off) ? b->suffix_off[u + 1] - b->suffix_off[u] : 0;
    int M = (mode != kPrefill && b->cand_off) ? b->cand_off[u + 1] - b->cand_off[u] : 0;
    ud.L = L; ud.S = S; ud.M = M;
    ud.prefix_src0 = b->prefix_off ? b->prefix_off[u] : 0;
    ud.suffix_src0 = b->suffix_off ? b->suffix_off[u] : 0;
    ud.cand_src0 = b->cand_off ? b->cand_off[u] : 0;
    relaygr_kv_handle h = (mode == kRankFull || !b->handles) ? RELAYGR_NO_CACHE : b->handles[u];
    bool compute_prefix;
    if (h != RELAYGR_NO_CACHE) {
      if (!pool) return fail(RELAYGR_EINVAL, "user %d has a handle but no pool was given", u);
      PoolEntry e;
      if (pool->resolve(h, &e) != RELAYGR_OK) return fail(RELAYGR_ENOENT, "user %d: stale or unknown handle", u);
      if (e.prefix_len != L) return fail(RELAYGR_EINVAL, "user %d: prefix length %d differs from the cached entry's %d", u, L, e.prefix_len);
      ud.kv = pool->slab;
      ud.kv_tile0 = e.page0 * (pool->page_tokens / kTile) * pool->tile_stride;
      ud.kv_tile_stride = pool->tile_stride;
      ud.kv_layer_stride = pool->layer_stride;
      compute_prefix = (mode == kPrefill);
    } else {
      if (mode == kPrefill) {
        if (L > 0) return fail(RELAYGR_EINVAL, "prefill: user %d has no handle", u);
        compute_prefix = false;
      } else {
        compute_prefix = L > 0;
        ud.kv_tile0 = kvs_tiles * (int64_t)(2 * kTile * d);   // pointer filled in once scratch is carved
        ud.kv_tile_stride = (int64_t)2 * kTile * d;
        ud.kv_layer_stride = 0;
        kvs_tiles += (L + kTile - 1) / kTile;
      }
    }
    pstart[u] = (int32_t)prow;
    ud.prow0 = compute_prefix ? (int32_t)prow : -1;
    if (compute_prefix) {
      if (!b->prefix_emb) return fail(RELAYGR_EINVAL, "user %d needs prefix_emb", u);
      prow += ((int64_t)L + palign - 1) / palign * palign;   // filler rows up to the next aligned start
    }
    nstart[u] = (int32_t)nrow;
    ud.nrow0 = (mode != kPrefill) ? (int32_t)nrow : -1;
    ud.sfx_tile0 = sfx_tiles * (int64_t)(2 * kTile * d);
    if (mode != kPrefill) { nrow += S + M; sfx_tiles += (S + kTile - 1) / kTile; }
    if (prow + nrow >= (1ll << 31) - 1) return fail(RELAYGR_EINVAL, "batch has 2^31 rows or more");
  }
  if (mode == kPrefill && b->handles) {   // two users writing one pool entry would race
    std::vector<relaygr_kv_handle> hs;
    for (int u = 0; u < n; ++u) if (b->handles[u] != RELAYGR_NO_CACHE) hs.push_back(b->handles[u]);
    std::sort(hs.begin(), hs.end());
    if (std::adjacent_find(hs.begin(), hs.end()) != hs.end()) return fail(RELAYGR_EINVAL, "prefill: two users of the batch carry the same handle");
  }
  pstart[n] = (int32_t)prow;
  p.n_prows = (int)prow; p.n_nrows = (int)nrow; p.n_rows = (int)(prow + nrow);
  p.sfx_tiles = sfx_tiles; p.kvs_tiles = kvs_tiles;
  for (int u = 0; u <= n; ++u) nstart[u] = (u < n ? nstart[u] : (int32_t)nrow) + p.n_prows;
  for (int u = 0; u < n; ++u) if (users[u].nrow0 >= 0) users[u].nrow0 += p.n_prows;
  if (p.n_rows == 0) return RELAYGR_OK;
  if (mode != kPrefill && nrow > 0) {
    if ((sfx_tiles > 0 && !b->suffix_emb)) return fail(RELAYGR_EINVAL, "suffix tokens present but suffix_emb is null");
    if (!b->cand_emb && b->cand_off && b->cand_off[n] > 0) return fail(RELAYGR_EINVAL, "candidates present but cand_emb is null");
    if (!scores && b->cand_off && b->cand_off[n] > 0) return fail(RELAYGR_EINVAL, "scores_dev is null");
  }

  const int nq = bf16 ? attn_row_blocks(users, H, dh) : 1;
  const int rpt = rows_per_attn_tile(cfg, nq);

  // -- attention row tiles, and the launch lists made of them (all layers but the last; the last): longest items first
  std::vector<AttnTile> rows_new, rows_prefix;
  attn_row_tiles(users, rpt, rows_new, rows_prefix);
  AttnCut cut;
  if (!bf16) {
    int64_t half_tiles = 0;
    for (auto* rows : {&rows_new, &rows_prefix})
      for (const AttnTile& a : *rows) half_tiles += 2 * key_tiles(a) * H;
    fp32_splits((int64_t)(rows_new.size() + rows_prefix.size()) * H, half_tiles, &cut.nsplit, &cut.gs);
    cut.all = rows_new;
    cut.all.insert(cut.all.end(), rows_prefix.begin(), rows_prefix.end());
    auto longer = [](const AttnTile& a, const AttnTile& b2) { return key_tiles(a) > key_tiles(b2); };
    std::stable_sort(cut.all.begin(), cut.all.begin() + rows_new.size(), longer);
    std::stable_sort(cut.all.begin() + rows_new.size(), cut.all.end(), longer);
  } else {
    cut_attention(rows_new, rows_prefix, H, dh, rpt, c->n_cus, cut, [&](const AttnCut& k) {
      p.nsplit = k.nsplit; p.n_tiles = (int)(k.all.size() + k.last.size());
      carve(cfg, p);
      return p.total <= cs.bytes;
    });
    set_user_parts(users, cut);
  }
  p.nsplit = cut.nsplit;
  p.n_tiles = (int)(cut.all.size() + cut.last.size());

  // -- scratch
  carve(cfg, p);
  while (!bf16 && p.total > cs.bytes && p.nsplit > 1) { p.nsplit -= 1; carve(cfg, p); }   // (16-bit: cut to fit above)
  if (p.total > cs.bytes)
    return fail(RELAYGR_ENOSPC, "scratch too small: call needs %zu bytes, %zu are available", p.total, cs.bytes);
  char* S0 = cs.base;
  float* x = (float*)(S0 + p.off_x);
  T* xh = (T*)(S0 + p.off_xh);
  T* ubuf = (T*)(S0 + p.off_u);
  T* qbuf = (T*)(S0 + p.off_q);
  T* knew = (T*)(S0 + p.off_knew);
  T* vnew = (T*)(S0 + p.off_vnew);
  T* sfx = (T*)(S0 + p.off_sfx);
  T* kvs = (T*)(S0 + p.off_kvs);
  float* part = (float*)(S0 + p.off_part);
  float* ml = (float*)(S0 + p.off_ml);
  const bool softmax = c->attn_form == RELAYGR_ATTN_SOFTMAX;
  RowTables rt;
  {
    size_t rb = align_up((size_t)p.n_rows * 4);
    char* r0 = S0 + p.off_rows;
    rt.user = (int32_t*)r0; rt.kind = (int32_t*)(r0 + rb); rt.idx = (int32_t*)(r0 + 2 * rb);
    rt.lim = (int32_t*)(r0 + 3 * rb); rt.src = (int32_t*)(r0 + 4 * rb); rt.parts = (int32_t*)(r0 + 5 * rb);
  }
  for (int u = 0; u < n; ++u)
    if (!users[u].kv) users[u].kv = kvs;
  for (auto* list : {&cut.all, &cut.last})
    for (AttnTile& a : *list) a.kv = (const char*)users[a.user].kv + users[a.user].kv_tile0 * (int64_t)sizeof(T);

  // -- descriptor blob: users | pstart | nstart | tiles(new, prefix)
  StagingSlot* slot;
  int rc = staging_acquire(c, p.blob_bytes, &slot);
  if (rc != RELAYGR_OK) return rc;
  size_t o_users = 0, o_ps = align_up((size_t)n * sizeof(UserDesc)), o_ns = o_ps + align_up((size_t)(n + 1) * 4),
         o_tiles = o_ns + align_up((size_t)(n + 1) * 4);
  char* hb = slot->blob();
  memcpy(hb + o_users, users.data(), (size_t)n * sizeof(UserDesc));
  memcpy(hb + o_ps, pstart.data(), (size_t)(n + 1) * 4);
  memcpy(hb + o_ns, nstart.data(), (size_t)(n + 1) * 4);
  if (!cut.all.empty()) memcpy(hb + o_tiles, cut.all.data(), cut.all.size() * sizeof(AttnTile));
  if (!cut.last.empty()) memcpy(hb + o_tiles + cut.all.size() * sizeof(AttnTile), cut.last.data(), cut.last.size() * sizeof(AttnTile));
  char* db = S0 + p.off_blob;
  // few users: the first kernel fetches the descriptors itself; many, or a stream under capture: a copy command brings them
  const bool inline_batch = n <= kInlineUsers && p.blob_bytes <= kInlineBlobBytes && !capturing;
  BlobCopy bc = {};
  InlineBatch ib = {};
  int copy_blocks = 0;
  if (inline_batch) {
    memcpy(ib.users, users.data(), (size_t)n * sizeof(UserDesc));
    memcpy(ib.pstart, pstart.data(), (size_t)(n + 1) * 4);
    memcpy(ib.nstart, nstart.data(), (size_t)(n + 1) * 4);
    copy_blocks = (int)((p.blob_bytes + kBlobChunk - 1) / kBlobChunk);
    bc = {(const uint4*)hb, (uint4*)db, slot->flags(), ++slot->seq, (int)(p.blob_bytes / 16)};
  } else {
    HIP_TRY(hipMemcpyAsync(db, hb, p.blob_bytes, hipMemcpyHostToDevice, st));
    HIP_TRY(hipEventRecord(slot->done, st));
    slot->pending = true;
  }
  const UserDesc* d_users = (const UserDesc*)(db + o_users);
  const int32_t* d_ps = (const int32_t*)(db + o_ps);
  const int32_t* d_ns = (const int32_t*)(db + o_ns);
  const AttnTile* d_tiles = (const AttnTile*)(db + o_tiles);

  const float alpha = 1.0f / sqrtf((float)dh);
  const float kLog2e = 1.4426950408889634f;
  const float q_mul = bf16 ? alpha * kLog2e : 1.0f;       // what f1 multiplies q by before storing it
  const float score_mul = bf16 ? 1.0f : alpha;            // what the attention kernel still applies
  const T* emb_p = (const T*)b->prefix_emb;
  const T* emb_s = (const T*)b->suffix_emb;
  const T* emb_c = (const T*)b->cand_emb;
  const int R = p.n_rows;
  constexpr bool kPanel = !std::is_same<T, float>::value;   // bf16: xh / y are written as MFMA panels

  const int shared_tiles = bf16 ? attn_shared_tiles(softmax, H, dh, !rows_prefix.empty(), cut, c->n_cus) : kNoneShared;

  for (int l = 0; l < NL; ++l) {
    const relaygr_layer_weights& lw = c->layers[l];
    const bool last = (l == NL - 1);
    // rows whose layer output is still needed: in the last layer prefix rows only supply K and V
    const int a0 = last ? p.n_prows : 0;
    const bool have_active = a0 < R;

    // step 1: input LayerNorm of the first layer, with the gather of the embeddings into the residual stream, the row
    // tables and the cleared tail tiles; later layers get theirs from the previous layer's tail kernel
    if (l == 0) {
      ProfScope ps(c, RELAYGR_K_LN, st);
      const RowBuild rb = {d_users, d_ps, d_ns, n, p.n_prows, rpt, cut.piece_all};
      TailClear tc = {(R + kRowsPerBlock - 1) / kRowsPerBlock, 0, H, dh, 0, p.sfx_tiles ? (void*)sfx : nullptr};
      if (!bf16 && p.n_prows) tc.kv_layers = NL;   // the 16-bit projection fills a prefix's ragged tail itself
      if (tc.kv_layers > 0 || tc.sfx != nullptr) tc.jobs = n * (tc.kv_layers + 1) * H;
      dim3 grid(tc.row_blocks + tc.jobs + copy_blocks);
      bool ok = dispatch_e(d, [&](auto e) {
        constexpr int E = decltype(e)::value;
        if (inline_batch)
          hipLaunchKernelGGL((ln_in_kernel<T, E, kPanel, true>), grid, dim3(256), 0, st, x, xh, (const T*)lw.ln_in_g, (const T*)lw.ln_in_b,
                             emb_p, emb_s, emb_c, rt, rb, tc, bc, ib, R, cfg.ln_eps);
        else
          hipLaunchKernelGGL((ln_in_kernel<T, E, kPanel, false>), grid, dim3(256), 0, st, x, xh, (const T*)lw.ln_in_g, (const T*)lw.ln_in_b,
                             emb_p, emb_s, emb_c, rt, rb, tc, bc, ib, R, cfg.ln_eps);
      });
      if (!ok) return fail(RELAYGR_EINVAL, "unsupported d_model");
      LAUNCH_CHECK("ln_in");
      if (inline_batch) { slot->chunks = copy_blocks; slot->stream = st; }   // now the kernel that will set the flags is on its stream
    }
    // step 2: projections
    ColMap all4 = {4, {0, 1, 2, 3}, d}, kv_only = {2, {1, 3, 0, 0}, d};
    auto run_f1 = [&](int r0, int r1, const ColMap& cm) {
      if constexpr (std::is_same<T, float>::value) {
        F1F32Params fp;
        fp.A = xh; fp.W = (const float*)lw.w1; fp.bias = (const float*)lw.b1; fp.u = ubuf; fp.q = qbuf; fp.knew = knew; fp.vnew = vnew; fp.sfx = sfx;
        fp.users = d_users; fp.rt = rt; fp.d = d; fp.dh = dh; fp.n_prows = p.n_prows; fp.layer = l; fp.row_begin = r0; fp.row_end = r1; fp.cm = cm;
        // 128 x 128 tiles once they give every compute unit two, 64 x 64 while those do, 32 x 32 with k cut in four below
        const int64_t cols = (int64_t)cm.nblk * d;
        auto tiles = [&](int t) { return (int64_t)((r1 - r0 + t - 1) / t) * (cols / t); };
        const int tile = (d % 128 == 0 && tiles(128) >= 2 * c->n_cus) ? 128 : tiles(64) >= 2 * c->n_cus ? 64 : 32;
        fp.n_mtiles = (r1 - r0 + tile - 1) / tile;
        const dim3 grid((tiles(tile) + 7) / 8 * 8);
        if (tile == 128) hipLaunchKernelGGL((f1_f32_kernel<2, 0>), grid, dim3(256), 0, st, fp);
        else if (tile == 64) hipLaunchKernelGGL((f1_f32_kernel<1, 0>), grid, dim3(256), 0, st, fp);
        else dispatch_e(d, [&](auto e) { hipLaunchKernelGGL((f1_f32_kernel<1, 16 * decltype(e)::value>), grid, dim3(256), 0, st, fp); });
      } else {
        F1Params fp;
        fp.A = (const uint16_t*)xh; fp.W = c->w1_packed[l]; fp.bias = (const uint16_t*)lw.b1;
        fp.u = (uint16_t*)ubuf; fp.q = (uint16_t*)qbuf; fp.knew = (uint16_t*)knew; fp.vnew = (uint16_t*)vnew; fp.sfx = (uint16_t*)sfx;
        fp.users = d_users; fp.rt = rt; fp.d = d; fp.dh = dh; fp.n_prows = p.n_prows; fp.layer = l;
        fp.row_begin = r0; fp.row_end = r1;           // (r0: a multiple of kPrefixRowAlign)
        fp.cm = cm; fp.q_mul = q_mul; fp.octets = softmax ? 0 : 1; fp.stream_out = (r1 - r0) >= kF1StreamMinRows ? 1 : 0;
        const int cols = cm.nblk * (d / 128);
        auto launch = [&](auto kernel, int tile_rows, int tile_cols) {
          fp.n_mtiles = (r1 - r0 + tile_rows - 1) / tile_rows;
          hipLaunchKernelGGL(kernel, dim3((fp.n_mtiles * tile_cols + 7) / 8 * 8), dim3(256), 0, st, fp);
        };
        auto launch_d = [&](auto dim) {               // (no tile that f1_tile does not take at a width is built for it)
          constexpr int D = decltype(dim)::value, KT = D / kGemmKTile;
          switch (f1_tile(D, cm.nblk, r1 - r0, c->n_cus)) {
            case F1Tile::k64x64: launch(f1_gemm_bf16_kernel<HT, 1, 1, (KT <= 16 ? KT : 18), KT>, 64, 2 * cols); break;
            case F1Tile::k64x128: launch(f1_gemm_bf16_kernel<HT, 1, 2, (KT < 6 ? KT : 6), KT>, 64, cols); break;
            case F1Tile::k128x128: if constexpr (D >= 256) launch(f1_gemm_bf16_kernel<HT, 2, 2, 4, KT>, 128, cols); break;
            case F1Tile::k128x128x3: if constexpr (D >= 256 && D <= 512) launch(f1_gemm_bf16_kernel<HT, 2, 2, 3, KT>, 128, cols); break;
            case F1Tile::kStationary:
              if constexpr (D <= 512) hipLaunchKernelGGL((f1_ws_bf16_kernel<HT, D>), dim3(cols * f1_row_groups(D, cm.nblk, c->n_cus)), dim3(512), 0, st, fp);
              break;
            default: launch(f1_gemm_bf16_kernel<HT, kF1TM, kF1TN, kF1Stages, 0>, 64 * kF1TM, cols); break;
          }
        };
        switch (d) {
          case 128: launch_d(std::integral_constant<int, 128>()); break;
          case 256: launch_d(std::integral_constant<int, 256>()); break;
          case 512: launch_d(std::integral_constant<int, 512>()); break;
          default: launch_d(std::integral_constant<int, 1024>()); break;
        }
      }
    };
    if (last && p.n_prows) {
      ProfScope ps(c, RELAYGR_K_F1, st);
      run_f1(0, p.n_prows, kv_only);
      LAUNCH_CHECK("f1 (k,v only)");
    }
    if (have_active) {
      ProfScope ps(c, RELAYGR_K_F1, st);
      run_f1(a0, R, all4);
      LAUNCH_CHECK("f1");
    }
    if (!have_active) continue;
    // step 3: attention partial sums
    AttnParams ap;
    ap.tiles = d_tiles; ap.q = qbuf; ap.sfx = sfx; ap.part = part;
    ap.split_stride = (size_t)R * d; ap.nsplit = p.nsplit; ap.d = d; ap.n_heads = H; ap.layer = l; ap.score_mul = score_mul;
    ap.ml = ml; ap.ml_stride = (size_t)R * H * 2; ap.gs = shared_tiles < kNoneShared ? 2 : cut.gs;
    ap.shared_tiles = shared_tiles;
    // 16-bit SiLU form: the attention kernel adds the candidates' own keys, so the layer tail does not read q, k, v again
    const bool self_in_attn = bf16 && !softmax;
    ap.knew = self_in_attn ? (const void*)knew : nullptr; ap.vnew = vnew; ap.n_prows = p.n_prows; ap.n_rows = R;
    const bool own_list = bf16 && last && p.n_prows > 0;
    const int nt = (int)(own_list ? cut.last.size() : !bf16 && last ? rows_new.size() : cut.all.size());   // (fp32: new rows first)
    ap.n_tiles = nt;
    if (own_list) ap.tiles = d_tiles + cut.all.size();
    if (nt > 0) {
      ProfScope ps(c, RELAYGR_K_ATTN, st);
      rc = launch_attention<T>(cfg, ap, nt, nq, softmax, st);
      if (rc != RELAYGR_OK) return rc;
    }
    // steps 3-4: combine, self term, 1/n, LayerNorm, gate, output projection, residual, next LayerNorm or score head
    {
      ProfScope ps(c, RELAYGR_K_F2, st);
      if constexpr (std::is_same<T, float>::value) {
        TailF32Params fp;
        fp.part = part; fp.nsplit = p.nsplit; fp.split_stride = (size_t)R * d; fp.ml = ml; fp.ml_stride = (size_t)R * H * 2; fp.n_heads = H;
        fp.u = ubuf; fp.q = qbuf; fp.knew = knew; fp.vnew = vnew; fp.gate_gain = (const float*)lw.ln_at_g; fp.gate_offs = (const float*)lw.ln_at_b;
        fp.W = (const float*)lw.w2; fp.bias = (const float*)lw.b2; fp.x = x; fp.xh = last ? nullptr : xh;
        fp.gain = (const float*)(last ? c->ln_out_g : c->layers[l + 1].ln_in_g);
        fp.offs = (const float*)(last ? c->ln_out_b : c->layers[l + 1].ln_in_b);
        fp.rt = rt; fp.n_prows = p.n_prows; fp.dh = dh; fp.row_begin = a0; fp.row_end = R; fp.alpha = alpha; fp.eps = cfg.ln_eps;
        fp.w_score = (const float*)c->w_score; fp.b_score = c->b_score; fp.scores = last && mode != kPrefill ? scores : nullptr;
        const dim3 grid((R - a0 + 15) / 16);
        dispatch_e(d, [&](auto e) {
          constexpr int D = 64 * decltype(e)::value;
          if (softmax) hipLaunchKernelGGL((tail_f32_kernel<D, true>), grid, dim3(1024), 0, st, fp);
          else hipLaunchKernelGGL((tail_f32_kernel<D, false>), grid, dim3(1024), 0, st, fp);
        });
      } else {
        {
          F2LnParams fp;
          fp.W = c->w2_packed[l]; fp.bias = (const uint16_t*)lw.b2; fp.x = x; fp.rt = rt;
          // the last layer of a ranking call ends in the score head instead of the next layer's LayerNorm
          const bool score_here = last && mode != kPrefill && scores != nullptr;
          fp.xh = last ? nullptr : (uint16_t*)xh;
          fp.gain = last ? (const uint16_t*)c->ln_out_g : (const uint16_t*)c->layers[l + 1].ln_in_g;
          fp.offs = last ? (const uint16_t*)c->ln_out_b : (const uint16_t*)c->layers[l + 1].ln_in_b;
          fp.w_score = (const uint16_t*)c->w_score; fp.b_score = c->b_score; fp.scores = score_here ? scores : nullptr;
          fp.row_begin = a0; fp.row_end = R; fp.eps = cfg.ln_eps;
          fp.part = part; fp.parts_shift = last ? 8 : 0; fp.parts_all = last ? cut.parts_last : cut.parts_all; fp.split_stride = (size_t)R * d;
          fp.u = (const uint16_t*)ubuf; fp.q = self_in_attn ? nullptr : (const uint16_t*)qbuf; fp.knew = (const uint16_t*)knew; fp.vnew = (const uint16_t*)vnew;
          fp.gate_gain = (const uint16_t*)lw.ln_at_g; fp.gate_offs = (const uint16_t*)lw.ln_at_b;
          fp.n_prows = p.n_prows; fp.dh = dh;
          fp.ml = softmax ? ml : nullptr; fp.ml_stride = (size_t)R * H * 2; fp.n_heads = H;
          const int wg_rows = tail_rows(d, R - a0);
          const bool rb2 = wg_rows == 64, vr8 = wg_rows == 8, vr16 = wg_rows == 16;
          const dim3 grid((R - a0 + wg_rows - 1) / wg_rows);
          auto launch_tail = [&](auto sm, auto sums) {
            constexpr bool SM = decltype(sm)::value;
            constexpr int NB = decltype(sums)::value, NB2 = NB < 2 ? NB : 2;
            switch (d) {
              case 128:
                if (rb2) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 128, 4, 4, SM, 1, 64, 0, NB2>), grid, dim3(256), 0, st, fp);
                else hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 128, 4, 2, SM, 1, 32, 0, NB2>), grid, dim3(256), 0, st, fp);
                break;
              case 256:
                if (rb2) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 256, 8, 4, SM, 1, 64, 0, NB2>), grid, dim3(512), 0, st, fp);
                else if (vr8) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 256, 8, 1, SM, 1, 8, 4, NB>), grid, dim3(512), 0, st, fp);
                else if (vr16) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 256, 8, 1, SM, 1, 16, 4, NB>), grid, dim3(512), 0, st, fp);
                else hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 256, 8, 2, SM, 1, 32, 0, NB2>), grid, dim3(512), 0, st, fp);
                break;
              case 512:
                if (rb2) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 512, 8, 4, SM, 2, 64, 0, NB2>), grid, dim3(512), 0, st, fp);
                else if (vr8) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 512, 8, 1, SM, 1, 8, 4, NB>), grid, dim3(512), 0, st, fp);
                else if (vr16) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 512, 8, 1, SM, 1, 16, 4, NB>), grid, dim3(512), 0, st, fp);
                else hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 512, 8, 2, SM, 1, 32, 0, NB2>), grid, dim3(512), 0, st, fp);
                break;
              default:
                if (vr8) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 1024, 8, 1, SM, 1, 8, 0, NB>), grid, dim3(512), 0, st, fp);
                else if (vr16) hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 1024, 8, 1, SM, 1, 16, 0, 1>), grid, dim3(512), 0, st, fp);
                else hipLaunchKernelGGL((f2_ln_bf16_kernel<HT, 1024, 8, 2, SM, 1, 32, 0, 1>), grid, dim3(512), 0, st, fp);
                break;
            }
          };
          auto launch_sums = [&](auto sm) {
            switch (sums_at_once(fp.parts_all, p.nsplit)) {
              case 1: launch_tail(sm, std::integral_constant<int, 1>()); break;
              case 2: launch_tail(sm, std::integral_constant<int, 2>()); break;
              case 4: launch_tail(sm, std::integral_constant<int, 4>()); break;
              default: launch_tail(sm, std::integral_constant<int, kMaxPieces>()); break;
            }
          };
          if (softmax) launch_sums(std::true_type());
          else launch_sums(std::false_type());
        }
      }
    }
    LAUNCH_CHECK("f2");
  }

  return RELAYGR_OK;
}

static bool stream_is_capturing(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) { (void)hipGetLastError(); return false; }
  return cap != hipStreamCaptureStatusNone;
}

// Makes stream `st` wait for everything enqueued so far on `prev` (the stream of the previous call on the same
// scratch): the event is recorded on `prev` only now, when a call arrives on another stream, so that calls that
// stay on one stream pay nothing.  If `prev` can no longer take an event (destroyed by its owner while its work may
// still be running) the device is synchronised instead.
static hipError_t order_behind(hipStream_t st, hipStream_t prev, hipEvent_t ev) {
  hipError_t e = hipEventRecord(ev, prev);
  if (e == hipSuccess) e = hipStreamWaitEvent(st, ev, 0);
  if (e == hipSuccess) return e;
  (void)hipGetLastError();
  return hipDeviceSynchronize();
}

static int run(relaygr_ctx* c, relaygr_kv_pool* pool, const relaygr_batch* b, Mode mode, float* scores, void* stream,
               const CallScratch* other = nullptr) {
  if (!c || !b) return fail(RELAYGR_EINVAL, "null context or batch");
  if (b->n_users < 0) return fail(RELAYGR_EINVAL, "n_users < 0");
  if (b->n_users == 0) return RELAYGR_OK;
  std::lock_guard<std::mutex> call_lock(c->mu);
  c->prof_this_call = (c->prof_calls++ % c->prof_every) == 0;
  int rc;
  if ((rc = check_offsets(b->prefix_off, b->n_users, "prefix")) != RELAYGR_OK) return rc;
  if ((rc = check_offsets(b->suffix_off, b->n_users, "suffix")) != RELAYGR_OK) return rc;
  if ((rc = check_offsets(b->cand_off, b->n_users, "candidate")) != RELAYGR_OK) return rc;
  KvPool* kp = reinterpret_cast<KvPool*>(pool);
  if (kp) {
    const relaygr_model_config &a = kp->cfg, &m = c->cfg;
    if (a.n_layers != m.n_layers || a.d_model != m.d_model || a.n_heads != m.n_heads || a.dtype != m.dtype)
      return fail(RELAYGR_EINVAL, "pool and context were created for different model shapes");
  }
  hipStream_t st = (hipStream_t)stream;
  (void)hipGetLastError();   // a failure the caller's own HIP calls left behind is not this call's: launch checks below start clean
  const size_t wp = wpack_bytes(c->cfg);
  const CallScratch own = {c->scratch + wp, c->scratch_bytes - wp};
  const CallScratch& cs = other ? *other : own;
  // (a stream under graph capture takes neither the wait nor the event: the captured work is ordered by its graph,
  // and against the context's other calls by whoever launches that graph)
  const bool capturing = stream_is_capturing(st);
  if (!capturing && c->has_call && c->last_stream != st) HIP_TRY(order_behind(st, c->last_stream, c->call_done));
  if (c->cfg.dtype == RELAYGR_DTYPE_FP32) rc = run_typed<float>(c, kp, b, mode, scores, cs, st, capturing);
  else if (c->cfg.dtype == RELAYGR_DTYPE_FP16) rc = run_typed<__half>(c, kp, b, mode, scores, cs, st, capturing);
  else rc = run_typed<__hip_bfloat16>(c, kp, b, mode, scores, cs, st, capturing);
  if (!capturing) { c->last_stream = st; c->has_call = true; }
  return rc;
}

extern "C" int relaygr_prefill_prefix(relaygr_ctx* ctx, relaygr_kv_pool* pool, const relaygr_batch* batch, void* hip_stream) {
  if (!pool) return fail(RELAYGR_EINVAL, "prefill_prefix: null pool");
  if (batch && !batch->handles) return fail(RELAYGR_EINVAL, "prefill_prefix: null handles");
  return run(ctx, pool, batch, kPrefill, nullptr, hip_stream);
}

extern "C" int relaygr_rank_with_cache(relaygr_ctx* ctx, relaygr_kv_pool* pool, const relaygr_batch* batch, float* scores_dev,
                                       void* hip_stream) {
  return run(ctx, pool, batch, kRankCached, scores_dev, hip_stream);
}

extern "C" int relaygr_rank_with_cache_static(relaygr_ctx* ctx, relaygr_kv_pool* pool, const relaygr_batch* batch, float* scores_dev,
                                              void* hip_stream) {
  char* base = nullptr;
  int dev = 0;
  int rc = static_scratch(&base, &dev);      // a table lookup after the first call on this device
  if (rc != RELAYGR_OK) return rc;
  const CallScratch cs = {base, kStaticScratchBytes + kStaticDescriptorBytes};
  {
    // one caller at a time enqueues on the shared array, behind the call that used it last
    std::lock_guard<std::mutex> lk(g_static_mu);
    hipStream_t st = (hipStream_t)hip_stream;
    const bool capturing = stream_is_capturing(st);
    if (!capturing && g_static_has_call[dev] && g_static_last_stream[dev] != st) HIP_TRY(order_behind(st, g_static_last_stream[dev], g_static_done[dev]));
    rc = run(ctx, pool, batch, kRankCached, scores_dev, hip_stream, &cs);
    if (!capturing) { g_static_last_stream[dev] = st; g_static_has_call[dev] = true; }
  }
  if (rc == RELAYGR_ENOSPC)
    return fail(rc, "rank_with_cache_static: the call does not fit the library's %zu-byte scratch (%s); use relaygr_rank_with_cache",
                kStaticScratchBytes, std::string(relaygr_last_error()).c_str());
  return rc;
}

extern "C" size_t relaygr_static_scratch_bytes(void) { return kStaticScratchBytes; }

extern "C" int relaygr_rank_full_recompute(relaygr_ctx* ctx, const relaygr_batch* batch, float* scores_dev, void* hip_stream) {
  return run(ctx, nullptr, batch, kRankFull, scores_dev, hip_stream);
}
