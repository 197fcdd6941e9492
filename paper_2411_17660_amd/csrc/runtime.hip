// runtime.hip -- host side of libgsr.so: context, workspace, validation and
// the launch sequences behind the C ABI (include/gsr.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstddef>
#include <map>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/gsr.h"
#include "launch.h"



using namespace gsr;

namespace {

struct DBuf {
  void* p = nullptr;
  size_t bytes = 0;
};

struct Saved {
  bool valid = false;
  gsr_settings set{};
  int64_t n = 0;
  int F = 0;
  const float *means = nullptr, *log_scales = nullptr, *quats = nullptr, *opac = nullptr,
              *sh = nullptr, *poses = nullptr;
  const float *rgb = nullptr, *depth = nullptr;
  int64_t T = 0, P = 0, max_hw = 0;
  uint64_t K = 0;          // exact count (grow mode) or capacity bound (fixed mode)
  bool k_known = false;
  bool sorted_in_b = false;   // tile sort result buffer
  bool keys16 = false;        // tile keys stored as 16 bits
  bool surfel = false;        // the forward rendered 2D surfels
  bool has_backward = false;  // a backward of this forward has filled grad2d
};

}  // namespace

struct gsr_context {
  int device = 0;
  std::string err;
  // workspace
  DBuf rec, trect, trect_s, keyoff, dkey_a, dval_a, dkey_b, dval_b, ntiles, cnt_sorted, offsets, scan_tmp, hist,
      counters;
  DBuf keys_a, vals_a, keys_b, vals_b, partial, stamp, grad2d;
  DBuf ranges, nproc, t_final, n_last, frames, twist_part, loss_part, loss_scale;
  DBuf ssim_rgb, ssim_tiles, ssim_scale;  // rendering loss with SSIM
  DBuf med_pos;                     // per pixel: list position of the median-depth entry
  DBuf dist_aux, spart, sgrad;      // surfels: distortion sums per pixel, per-key and
                                    // per-record gradient sums
  DBuf nc_part;                     // normal consistency: per-block loss partials
  DBuf reloc_cnt, reloc_rule;       // MCMC relocation scratch
  DBuf up_rgb, up_depth, up_alpha;  // upstream gradients for gsr_step_l1
  DBuf tune_out;                    // scratch outputs of the autotuner
  DBuf order_f, order_b;            // compositing tile schedules (forward, backward)
  DBuf bwd_maps;   // compositing backward in segments: state changes per pixel
  DBuf cls_order;  // records ordered by key count (per-record reduction)
  // layout (tile shape and frame sizes) whose processed-entry counts nproc
  // holds, so that the next forward over the same tiles can order its queue
  // by them; empty when nproc holds none
  std::vector<int32_t> nproc_layout;
  std::map<std::string, gsr_settings> tune_cache;
  uint64_t key_cap = 0;             // allocated key slots
  // pinned host staging
  uint64_t* h_count = nullptr;
  void* loss_scratch = nullptr;     // this device's static scratch of gsr_loss_l1_noalloc
  std::vector<FrameDesc> last_frames;
  uint32_t epoch = 0;
  Saved s;
  // GSR_FLAG_TIMING: event pairs per stage, read by gsr_debug_timings
  struct Timed { int stage; hipEvent_t a, b; };
  std::vector<Timed> timed;
  std::vector<hipEvent_t> ev_pool;
  int64_t n_pairs = -1;
};

namespace {

gsr_status fail(gsr_context* c, gsr_status code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (c) c->err = buf;
  return code;
}

gsr_status hip_check(gsr_context* c, hipError_t e, const char* what) {
  if (e == hipSuccess) return GSR_OK;
  return fail(c, GSR_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define GSR_HIP(expr)                                            \
  do {                                                           \
    gsr_status _s = hip_check(ctx, (expr), #expr);               \
    if (_s != GSR_OK) return _s;                                 \
  } while (0)

// Grow-only device buffer.  Growing synchronises the stream first so that no
// queued kernel still uses the old allocation; it is refused while the stream
// is being captured into a graph (a capture must follow an uncaptured call of
// the same sizes).  `zero` clears a new buffer with a fill kernel.
gsr_status ensure(gsr_context* ctx, DBuf& b, size_t bytes, hipStream_t st, bool zero = false) {
  if (bytes == 0) bytes = 16;
  if (b.bytes >= bytes) return GSR_OK;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  GSR_HIP(hipStreamIsCapturing(st, &cap));
  if (cap != hipStreamCaptureStatusNone)
    return fail(ctx, GSR_ERR_STATE,
                "workspace must grow to %zu bytes during graph capture; run the call once "
                "uncaptured with the same sizes first", bytes);
  const size_t want = bytes + bytes / 4;
  if (b.p) {
    GSR_HIP(hipStreamSynchronize(st));
    GSR_HIP(hipFree(b.p));
    b.p = nullptr;
    b.bytes = 0;
  }
  void* p = nullptr;
  if (hipMalloc(&p, want) != hipSuccess) {
    (void)hipGetLastError();
    return fail(ctx, GSR_ERR_OUT_OF_MEMORY, "hipMalloc of %zu bytes failed", want);
  }
  b.p = p;
  b.bytes = want;
  if (zero) launch_fill_u32(st, static_cast<uint32_t*>(p), want / 4, 0u);
  return GSR_OK;
}

template <typename T>
T* P(const DBuf& b) { return static_cast<T*>(b.p); }

gsr_status validate(gsr_context* ctx, const gsr_settings* s, int64_t n, const float* means,
                    const float* log_scales, const float* quats, const float* opac,
                    const float* sh, int32_t F, const gsr_camera* cams, const float* poses,
                    const float* rgb, const float* depth, const float* alpha) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  char msg[256];
  const gsr_status rc = check_forward(s, n, means, log_scales, quats, opac, sh, F, cams, poses,
                                      rgb, depth, alpha, msg, sizeof msg);
  if (rc) return fail(ctx, rc, "%s", msg);
  return GSR_OK;
}

// Frame descriptors to the device (re-uploaded only when they change).
// The frame table goes to the device as kernel arguments (by value), so
// every forward writes its own table on its stream, also inside a captured
// graph that holds several forwards with different tables; no host staging
// buffer has to outlive the call.
gsr_status upload_frames(gsr_context* ctx, const std::vector<FrameDesc>& fr, hipStream_t st) {
  gsr_status rc = ensure(ctx, ctx->frames, fr.size() * sizeof(FrameDesc), st);
  if (rc) return rc;
  launch_set_frames(st, fr.data(), (int)fr.size(), P<FrameDesc>(ctx->frames));
  ctx->last_frames = fr;
  return GSR_OK;
}

hipEvent_t take_event(gsr_context* ctx) {
  if (!ctx->ev_pool.empty()) {
    hipEvent_t e = ctx->ev_pool.back();
    ctx->ev_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Brackets one stage with events on the call's stream when timing is on.
struct StageTimer {
  gsr_context* ctx;
  hipStream_t st;
  int stage;
  hipEvent_t a = nullptr;
  StageTimer(gsr_context* c, hipStream_t s, bool on, int id) : ctx(c), st(s), stage(id) {
    if (!on) return;
    a = take_event(ctx);
    if (a) (void)hipEventRecord(a, st);
  }
  ~StageTimer() {
    if (!a) return;
    hipEvent_t b = take_event(ctx);
    if (!b) return;
    (void)hipEventRecord(b, st);
    ctx->timed.push_back({stage, a, b});
  }
};

}  // namespace

extern "C" {

gsr_status gsr_create(gsr_context** out, int32_t device) {
  if (!out) return GSR_ERR_INVALID_ARGUMENT;
  *out = nullptr;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || device < 0 || device >= count)
    return GSR_ERR_INVALID_ARGUMENT;
  if (hipSetDevice(device) != hipSuccess) return GSR_ERR_HIP;
  gsr_context* ctx = new (std::nothrow) gsr_context();
  if (!ctx) return GSR_ERR_OUT_OF_MEMORY;
  ctx->device = device;
  if (loss_scratch_init(device, &ctx->loss_scratch) != hipSuccess ||
      // (coherent: the host watches a kernel's store)
      hipHostMalloc((void**)&ctx->h_count, sizeof(uint64_t) * 8,
                    hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
    delete ctx;
    return GSR_ERR_HIP;
  }
  *out = ctx;
  return GSR_OK;
}

gsr_status gsr_destroy(gsr_context* ctx) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  (void)hipSetDevice(ctx->device);
  (void)hipDeviceSynchronize();
  DBuf* bufs[] = {&ctx->rec, &ctx->trect, &ctx->trect_s, &ctx->keyoff, &ctx->dkey_a, &ctx->dval_a, &ctx->dkey_b, &ctx->dval_b,
                  &ctx->ntiles, &ctx->cnt_sorted, &ctx->offsets, &ctx->scan_tmp, &ctx->hist,
                  &ctx->counters,
                  &ctx->keys_a, &ctx->vals_a, &ctx->keys_b, &ctx->vals_b, &ctx->partial,
                  &ctx->grad2d,
                  &ctx->stamp, &ctx->ranges, &ctx->nproc, &ctx->t_final, &ctx->n_last,
                  &ctx->frames, &ctx->twist_part, &ctx->loss_part, &ctx->loss_scale,
                  &ctx->ssim_rgb, &ctx->ssim_tiles, &ctx->ssim_scale, &ctx->med_pos,
                  &ctx->reloc_cnt, &ctx->reloc_rule,
                  &ctx->up_rgb, &ctx->up_depth, &ctx->up_alpha, &ctx->tune_out,
                  &ctx->order_f, &ctx->order_b, &ctx->bwd_maps, &ctx->cls_order, &ctx->dist_aux, &ctx->spart,
                  &ctx->sgrad, &ctx->nc_part};
  for (DBuf* b : bufs)
    if (b->p) (void)hipFree(b->p);
  if (ctx->h_count) (void)hipHostFree(ctx->h_count);
  for (auto& t : ctx->timed) {
    (void)hipEventDestroy(t.a);
    (void)hipEventDestroy(t.b);
  }
  for (hipEvent_t e : ctx->ev_pool) (void)hipEventDestroy(e);
  delete ctx;
  return GSR_OK;
}

const char* gsr_last_error(const gsr_context* ctx) { return ctx ? ctx->err.c_str() : ""; }

}  // extern "C"

namespace {

// h_count[kMailbox]: the key count posted by the forward's scan.  Watching it
// saves the copy behind the scan and the runtime's wait (about 10 us per
// forward); the stream is asked now and then, so that an error ends the wait.
// Every return comes after the post, or once the stream has nothing left that
// could post: a count that arrived later would be taken for the next forward's.
constexpr int kMailbox = 7;
constexpr uint64_t kNoCount = ~0ull;

gsr_status await_count(gsr_context* ctx, hipStream_t st, uint64_t* out) {
  const hipError_t before = hipGetLastError();  // of the launches, or of an earlier call
  const uint64_t* box = ctx->h_count + kMailbox;
  uint64_t v;
  for (uint32_t i = 1; (v = __atomic_load_n(box, __ATOMIC_ACQUIRE)) == kNoCount; ++i) {
    if (i % 4096 != 0) continue;
    // (a stream in capture runs nothing: its synchronisation says so)
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(st, &cap);
    if (e != hipSuccess || cap == hipStreamCaptureStatusNone) e = hipStreamQuery(st);
    (void)hipGetLastError();  // ("not ready" is no error of this call)
    if (e == hipErrorNotReady) continue;
    GSR_HIP(hipStreamSynchronize(st));
    v = __atomic_load_n(box, __ATOMIC_ACQUIRE);
    GSR_HIP(before);
    if (v == kNoCount) return fail(ctx, GSR_ERR_HIP, "the key count did not arrive");
    break;
  }
  GSR_HIP(before);
  *out = v;
  return GSR_OK;
}

// The forward of either primitive: 3D Gaussians (normal == NULL) or 2D
// surfels (log_scales [n,2], normal [sum 3HW], dist [sum HW]); they differ
// in the preprocess and the compositing kernels only.
gsr_status forward_impl(gsr_context* ctx, const gsr_settings* s, int64_t n, const float* means,
                        const float* log_scales, const float* quats, const float* opac,
                        const float* sh, int32_t F, const gsr_camera* cams, const float* poses,
                        float* rgb, float* depth, float* alpha, float* normal, float* dist,
                        bool surfel, void* stream) {
  gsr_status rc = validate(ctx, s, n, means, log_scales, quats, opac, sh, F, cams, poses, rgb,
                           depth, alpha);
  if (rc) return rc;
  if (surfel && (s->flags & GSR_FLAG_MEDIAN_DEPTH))
    return fail(ctx, GSR_ERR_UNSUPPORTED, "surfels: median depth not built");
  if (surfel && (!normal || !dist))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "normal or dist is NULL");
  if (surfel && ((((uintptr_t)normal) | ((uintptr_t)dist)) & 3u))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer not 4-aligned");
  ctx->err.clear();
  ctx->s.valid = false;
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  const int tw = s->tile_w, th = s->tile_h;
  // A0: frame descriptors
  std::vector<FrameDesc> fr;
  int64_t T = 0, Px = 0, max_hw = 0;
  {
    char msg[256];
    if ((rc = build_frames(F, cams, tw, th, fr, &T, &Px, &max_hw, msg, sizeof msg)))
      return fail(ctx, rc, "%s", msg);
  }
  if ((rc = upload_frames(ctx, fr, st))) return rc;
  const uint64_t M = (uint64_t)n * F;
  // workspace sized by M, T, P
  const size_t rec_bytes = surfel ? surfel_record_bytes() : sizeof(Record);
  if ((rc = ensure(ctx, ctx->rec, M * rec_bytes, st))) return rc;
  if ((rc = ensure(ctx, ctx->trect, M * sizeof(uint2), st))) return rc;
  if ((rc = ensure(ctx, ctx->trect_s, M * sizeof(uint2), st))) return rc;
  if ((rc = ensure(ctx, ctx->keyoff, M * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->dkey_a, M * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->dval_a, M * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->dkey_b, M * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->dval_b, M * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->ntiles, M * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->cnt_sorted, M * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->offsets, M * 8, st))) return rc;
  if ((rc = ensure(ctx, ctx->counters, 64, st, true))) return rc;
  if ((rc = ensure(ctx, ctx->ranges, (size_t)T * 8, st))) return rc;
  std::vector<int32_t> layout = {tw, th};
  for (int f = 0; f < F; ++f) {
    layout.push_back(cams[f].width);
    layout.push_back(cams[f].height);
  }
  const void* nproc_before = ctx->nproc.p;
  if ((rc = ensure(ctx, ctx->nproc, (size_t)T * 4, st))) return rc;
  const bool have_prev = ctx->nproc.p == nproc_before && ctx->nproc_layout == layout;
  if ((rc = ensure(ctx, ctx->order_f, (size_t)T * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->order_b, (size_t)T * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->t_final, (size_t)Px * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->n_last, (size_t)Px * 4, st))) return rc;
  const bool median = (s->flags & GSR_FLAG_MEDIAN_DEPTH) != 0;
  if (median && (rc = ensure(ctx, ctx->med_pos, (size_t)Px * 4, st))) return rc;
  if (surfel && (rc = ensure(ctx, ctx->dist_aux, (size_t)Px * 16, st))) return rc;
  uint64_t* d_count = P<uint64_t>(ctx->counters);               // [0] = K
  uint32_t* d_overflow = (uint32_t*)(P<uint64_t>(ctx->counters) + 1);
  const bool timing = (s->flags & GSR_FLAG_TIMING) != 0;
  // grow mode: the host waits for the key count, which the scan posts to it
  uint64_t* mailbox = nullptr;
  if (s->key_capacity == 0) {
    mailbox = ctx->h_count + kMailbox;
    __atomic_store_n(mailbox, kNoCount, __ATOMIC_SEQ_CST);
  }
  // A1 preprocess: the keys go where the depth sort ends in (.._a) after it
  const bool few = rank_records(M);
  uint32_t* dkey = P<uint32_t>(few ? ctx->dkey_b : ctx->dkey_a);
  uint32_t* dval = P<uint32_t>(few ? ctx->dval_b : ctx->dval_a);
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_PREPROCESS);
    if (surfel)
      launch_surfel_preprocess(st, n, F, P<FrameDesc>(ctx->frames), poses, means, log_scales,
                               quats, opac, sh, s->sh_degree, tw, th, ctx->rec.p,
                               P<uint2>(ctx->trect), dkey,
                               dval, P<uint32_t>(ctx->ntiles));
    else
      launch_preprocess_fwd(st, n, F, P<FrameDesc>(ctx->frames), poses, means, log_scales,
                            quats, opac, sh, s->sh_degree, tw, th, P<Record>(ctx->rec),
                            P<uint2>(ctx->trect), dkey,
                            dval, P<uint32_t>(ctx->ntiles));
  }
  // depth sort of the records (32-bit keys)
  const uint64_t kcap_guess = std::max<uint64_t>(ctx->key_cap, s->key_capacity);
  const int tile_bits = bits_for((uint64_t)T + 1);
  const size_t hist_need = std::max(radix_hist_elems(M, 0),
                                    radix_hist_elems(std::max<uint64_t>(kcap_guess, 1), tile_bits));
  if ((rc = ensure(ctx, ctx->hist, hist_need * 4, st))) return rc;
  const size_t scan_need =
      std::max({scan_block_elems(M) * 8, radix_scan_elems(M, 0) * 4,
                radix_scan_elems(std::max<uint64_t>(kcap_guess, 1), tile_bits) * 4});
  if ((rc = ensure(ctx, ctx->scan_tmp, scan_need, st))) return rc;
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_DEPTH_SORT);
    if (few)
      launch_rank_records(st, dkey, dval, M, P<uint2>(ctx->trect), P<uint32_t>(ctx->dkey_a),
                          P<uint32_t>(ctx->dval_a), P<uint32_t>(ctx->cnt_sorted),
                          P<uint2>(ctx->trect_s));
    else
      launch_depth_sort(st, P<uint32_t>(ctx->dkey_a), P<uint32_t>(ctx->dval_a),
                        P<uint32_t>(ctx->dkey_b), P<uint32_t>(ctx->dval_b), M,
                        P<uint32_t>(ctx->hist), P<uint32_t>(ctx->scan_tmp));
  }
  const uint32_t* perm = P<uint32_t>(ctx->dval_a);
  // A2 offsets over the depth-ordered records, K on the device
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_OFFSETS);
    if (few)
      launch_ranked_scan(st, P<uint32_t>(ctx->cnt_sorted), M, P<uint64_t>(ctx->offsets), d_count,
                         mailbox);
    else
      launch_offsets_scan(st, P<uint32_t>(ctx->dkey_a), perm, P<uint2>(ctx->trect), M,
                          P<uint32_t>(ctx->cnt_sorted), P<uint2>(ctx->trect_s),
                          P<uint64_t>(ctx->offsets), P<uint64_t>(ctx->scan_tmp), d_count, mailbox);
  }
  // key capacity
  uint64_t K = 0, cap = 0;
  bool k_known = false;
  if (s->key_capacity == 0) {
    if (M > 0 && (rc = await_count(ctx, st, &K))) return rc;
    if (K >= (1ull << 32) - 1) return fail(ctx, GSR_ERR_CAPACITY, "%llu keys exceed 2^32",
                                           (unsigned long long)K);
    cap = K;
    k_known = true;
  } else {
    cap = (uint64_t)s->key_capacity;
    K = cap;
  }
  if (cap > ctx->key_cap || !ctx->keys_a.p) {
    const uint64_t c2 = std::max<uint64_t>(cap, 1);
    if ((rc = ensure(ctx, ctx->keys_a, c2 * 4, st))) return rc;
    if ((rc = ensure(ctx, ctx->vals_a, c2 * 4, st))) return rc;
    if ((rc = ensure(ctx, ctx->keys_b, c2 * 4, st))) return rc;
    if ((rc = ensure(ctx, ctx->vals_b, c2 * 4, st))) return rc;
    if ((rc = ensure(ctx, ctx->partial, c2 * kNG * 4, st))) return rc;
    if ((rc = ensure(ctx, ctx->stamp, c2 * 4, st, true))) return rc;
    ctx->key_cap = std::min({ctx->keys_a.bytes / 4, ctx->keys_b.bytes / 4, ctx->vals_a.bytes / 4,
                             ctx->vals_b.bytes / 4, ctx->partial.bytes / (kNG * 4),
                             ctx->stamp.bytes / 4});
  }
  if ((rc = ensure(ctx, ctx->hist, radix_hist_elems(ctx->key_cap, tile_bits) * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->scan_tmp, radix_scan_elems(ctx->key_cap, tile_bits) * 4, st)))
    return rc;
  const uint64_t use_cap = s->key_capacity ? std::min<uint64_t>(cap, ctx->key_cap) : ctx->key_cap;
  // A3 keygen
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_KEYGEN);
    launch_keygen(st, M, (uint64_t)n, perm, P<uint32_t>(ctx->cnt_sorted),
                  P<uint64_t>(ctx->offsets), P<uint32_t>(ctx->keyoff), P<uint2>(ctx->trect_s),
                  P<FrameDesc>(ctx->frames), use_cap, tile_bits, ctx->keys_a.p,
                  P<uint32_t>(ctx->vals_a), d_overflow);
  }
  // A4 stable sort by tile id
  const uint64_t sort_n = k_known ? K : use_cap;
  bool keys_in_b = false;
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_TILE_SORT);
    keys_in_b = launch_tile_sort(st, ctx->keys_a.p, P<uint32_t>(ctx->vals_a), ctx->keys_b.p,
                                 P<uint32_t>(ctx->vals_b), k_known ? nullptr : d_count, sort_n,
                                 tile_bits, P<uint32_t>(ctx->hist), P<uint32_t>(ctx->scan_tmp));
  }
  const void* skeys = (keys_in_b ? ctx->keys_b : ctx->keys_a).p;
  const uint32_t* svals = P<uint32_t>(keys_in_b ? ctx->vals_b : ctx->vals_a);
  // A5 ranges
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_RANGES);
    launch_ranges(st, skeys, tile_bits, d_count, sort_n, use_cap, P<uint2>(ctx->ranges),
                  (uint64_t)T);
  }
  // A6 compositing
  const bool remap = !(s->flags & GSR_FLAG_NO_XCD_REMAP);
  unsigned long long* d_pairs = (unsigned long long*)(P<uint64_t>(ctx->counters) + 2);
  const bool count = (s->flags & GSR_FLAG_COUNT_PAIRS) != 0;
  if (count) launch_fill_u32(st, (uint32_t*)d_pairs, 2, 0u);
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_COMPOSITE_FWD);
    if (surfel)
      launch_surfel_fwd(st, tw, th, (int)T, F, P<FrameDesc>(ctx->frames), P<uint2>(ctx->ranges),
                        svals, ctx->rec.p, s->background, rgb, depth, alpha, normal, dist,
                        P<float>(ctx->t_final), P<int32_t>(ctx->n_last), P<float>(ctx->dist_aux),
                        P<uint32_t>(ctx->nproc), have_prev ? P<uint32_t>(ctx->nproc) : nullptr,
                        P<uint32_t>(ctx->order_f), remap, count ? d_pairs : nullptr);
    else
      launch_composite_fwd(st, tw, th, (int)T, F,
                           P<FrameDesc>(ctx->frames),
                           P<uint2>(ctx->ranges), svals, P<Record>(ctx->rec), s->background,
                           rgb, depth, alpha, P<float>(ctx->t_final), P<int32_t>(ctx->n_last),
                           P<uint32_t>(ctx->nproc),
                           have_prev ? P<uint32_t>(ctx->nproc) : nullptr,
                           P<uint32_t>(ctx->order_f), remap, count ? d_pairs : nullptr,
                           median ? P<int32_t>(ctx->med_pos) : nullptr);
  }
  ctx->nproc_layout = layout;
  ctx->n_pairs = count ? -2 : -1;  // -2: count pending on the device
  GSR_HIP(hipGetLastError());
  Saved& sv = ctx->s;
  sv.valid = true;
  sv.has_backward = false;
  sv.set = *s;
  sv.n = n;
  sv.F = F;
  sv.means = means; sv.log_scales = log_scales; sv.quats = quats; sv.opac = opac; sv.sh = sh;
  sv.poses = poses;
  sv.rgb = rgb;
  sv.depth = depth;
  sv.T = T;
  sv.P = Px;
  sv.max_hw = max_hw;
  sv.K = sort_n;
  sv.k_known = k_known;
  sv.sorted_in_b = keys_in_b;
  sv.keys16 = tile_keys_16bit(tile_bits);
  sv.surfel = surfel;
  return GSR_OK;
}

}  // namespace

extern "C" {

gsr_status gsr_forward(gsr_context* ctx, const gsr_settings* s, int64_t n, const float* means,
                       const float* log_scales, const float* quats, const float* opac,
                       const float* sh, int32_t F, const gsr_camera* cams, const float* poses,
                       float* rgb, float* depth, float* alpha, void* stream) {
  return forward_impl(ctx, s, n, means, log_scales, quats, opac, sh, F, cams, poses, rgb, depth,
                      alpha, nullptr, nullptr, false, stream);
}

gsr_status gsr_forward_surfel(gsr_context* ctx, const gsr_settings* s, int64_t n,
                              const float* means, const float* log_scales, const float* quats,
                              const float* opac, const float* sh, int32_t F,
                              const gsr_camera* cams, const float* poses, float* rgb,
                              float* depth, float* alpha, float* normal, float* dist,
                              void* stream) {
  return forward_impl(ctx, s, n, means, log_scales, quats, opac, sh, F, cams, poses, rgb, depth,
                      alpha, normal, dist, true, stream);
}

gsr_status gsr_normal_consistency(gsr_context* ctx, int32_t F, const gsr_camera* cams,
                                  const float* depth, const float* alpha, const float* normal,
                                  float weight, float* loss, float* g_depth, float* g_alpha,
                                  float* g_normal, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  {
    char msg[256];
    gsr_status rc0 = check_image_cameras(F, cams, msg, sizeof msg);
    if (rc0) return fail(ctx, rc0, "%s", msg);
  }
  if (!depth || !alpha || !normal || !loss || !g_depth || !g_alpha || !g_normal)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer is NULL");
  const void* ptrs[] = {depth, alpha, normal, loss, g_depth, g_alpha, g_normal};
  for (const void* p : ptrs)
    if (((uintptr_t)p) & 3u) return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer not 4-aligned");
  int64_t blocks = 0;
  for (int f = 0; f < F; ++f) blocks += normal_consistency_blocks(cams[f].width, cams[f].height);
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  gsr_status rc;
  if ((rc = ensure(ctx, ctx->nc_part, (size_t)blocks * 8, st))) return rc;
  launch_normal_consistency(st, F, cams, depth, alpha, normal, weight, P<double>(ctx->nc_part),
                            loss, g_depth, g_alpha, g_normal);
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_backward_surfel(gsr_context* ctx, const float* g_rgb, const float* g_depth,
                               const float* g_alpha, const float* g_normal,
                               const float* g_dist, float* g_means, float* g_log_scales,
                               float* g_quats, float* g_opac, float* g_sh, float* g_twist,
                               void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  Saved& sv = ctx->s;
  if (!sv.valid) return fail(ctx, GSR_ERR_STATE, "backward without a preceding forward");
  if (!sv.surfel) return fail(ctx, GSR_ERR_STATE, "the last forward rendered 3D Gaussians");
  if (!g_rgb || !g_depth || !g_alpha || !g_normal || !g_dist || !g_twist)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "gradient pointer is NULL");
  if (sv.n > 0 && (!g_means || !g_log_scales || !g_quats || !g_opac || !g_sh))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "gradient pointer is NULL");
  const void* ptrs[] = {g_rgb, g_depth, g_alpha, g_normal, g_dist, g_means, g_log_scales,
                        g_quats, g_opac, g_sh, g_twist};
  for (const void* p : ptrs)
    if (((uintptr_t)p) & 3u) return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer not 4-aligned");
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  const gsr_settings& s = sv.set;
  gsr_status rc;
  const size_t ng = (size_t)surfel_grad_values();
  const uint64_t M = (uint64_t)sv.n * sv.F;
  // slots of this forward's keys only (sv.K: its key count, or the fixed
  // capacity it ran with); records past it are marked as overflowed
  const uint64_t kcap = std::min<uint64_t>(sv.K, ctx->key_cap);
  if ((rc = ensure(ctx, ctx->spart, std::max<uint64_t>(kcap, 1) * ng * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->sgrad, std::max<uint64_t>(M, 1) * ng * 8, st))) return rc;
  if ((rc = ensure(ctx, ctx->cls_order, M * 4, st))) return rc;
  const int segments = bwd_segments(sv.K, sv.T, s.tile_w, s.tile_h);
  if ((rc = ensure(ctx, ctx->bwd_maps, bwd_map_bytes(), st))) return rc;
  const int64_t waves = sv.n > 0 ? surfel_preprocess_bwd_waves(sv.n) : 0;
  if ((rc = ensure(ctx, ctx->twist_part, (size_t)std::max<int64_t>(waves, 1) * sv.F * 6 * 8, st)))
    return rc;
  ++ctx->epoch;
  uint32_t* d_epoch = (uint32_t*)(P<uint64_t>(ctx->counters) + 3);
  launch_bump_epoch(st, d_epoch);
  const uint32_t* svals = P<uint32_t>(sv.sorted_in_b ? ctx->vals_b : ctx->vals_a);
  const bool timing = (s.flags & GSR_FLAG_TIMING) != 0;
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_COMPOSITE_BWD);
    launch_surfel_bwd(st, s.tile_w, s.tile_h, (int)sv.T, sv.F, P<FrameDesc>(ctx->frames),
                      P<uint2>(ctx->ranges), svals, ctx->rec.p,
                      P<uint32_t>(ctx->keyoff), s.background, g_rgb, g_depth, g_alpha, g_normal,
                      g_dist, P<float>(ctx->t_final), P<int32_t>(ctx->n_last),
                      P<float>(ctx->dist_aux), P<float>(ctx->spart), P<uint32_t>(ctx->stamp),
                      d_epoch, P<uint32_t>(ctx->nproc), P<uint32_t>(ctx->order_b),
                      !(s.flags & GSR_FLAG_NO_XCD_REMAP), segments, P<double2>(ctx->bwd_maps));
  }
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_PREPROCESS_BWD);
    launch_class_order(st, M, P<uint32_t>(ctx->ntiles), P<uint32_t>(ctx->cls_order), 0, nullptr,
                       P<uint32_t>(ctx->hist), P<uint32_t>(ctx->scan_tmp));
    launch_surfel_slot_reduce(st, M, P<uint32_t>(ctx->cls_order),
                              P<uint32_t>(ctx->keyoff), P<uint32_t>(ctx->ntiles),
                              P<float>(ctx->spart), P<uint32_t>(ctx->stamp), d_epoch,
                              kcap, P<double>(ctx->sgrad));
    launch_surfel_preprocess_bwd(st, sv.n, sv.F, P<FrameDesc>(ctx->frames), sv.poses, sv.means,
                                 sv.log_scales, sv.quats, sv.opac, sv.sh, s.sh_degree,
                                 P<uint32_t>(ctx->ntiles), P<uint32_t>(ctx->keyoff),
                                 P<double>(ctx->sgrad), kcap, g_means, g_log_scales,
                                 g_quats, g_opac, g_sh, P<double>(ctx->twist_part), g_twist);
  }
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_backward(gsr_context* ctx, const float* g_rgb, const float* g_depth,
                        const float* g_alpha, float* g_means, float* g_log_scales,
                        float* g_quats, float* g_opac, float* g_sh, float* g_twist,
                        void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  Saved& sv = ctx->s;
  if (!sv.valid) return fail(ctx, GSR_ERR_STATE, "backward without a preceding forward");
  if (sv.surfel) return fail(ctx, GSR_ERR_STATE, "the last forward rendered surfels");
  if (!g_rgb || !g_depth || !g_alpha || !g_twist)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "gradient pointer is NULL");
  if (sv.n > 0 && (!g_means || !g_log_scales || !g_quats || !g_opac || !g_sh))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "gradient pointer is NULL");
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  const gsr_settings& s = sv.set;
  gsr_status rc;
  // The epoch lives in device memory (counters[3]) and is advanced by a
  // kernel, so a captured step stamps with a new epoch on every replay.  A
  // stale stamp could only alias after 2^32 - 1 backward calls.
  ++ctx->epoch;
  uint32_t* d_epoch = (uint32_t*)(P<uint64_t>(ctx->counters) + 3);
  launch_bump_epoch(st, d_epoch);
  const uint32_t* svals = P<uint32_t>(sv.sorted_in_b ? ctx->vals_b : ctx->vals_a);
  const bool remap = !(s.flags & GSR_FLAG_NO_XCD_REMAP);
  const bool timing = (s.flags & GSR_FLAG_TIMING) != 0;
  // A8 reverse compositing -> per-key partials
  const int segments = bwd_segments(sv.K, sv.T, s.tile_w, s.tile_h);
  if ((rc = ensure(ctx, ctx->bwd_maps, bwd_map_bytes(), st))) return rc;
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_COMPOSITE_BWD);
    launch_composite_bwd(st, s.tile_w, s.tile_h, (int)sv.T, sv.F,
                         P<FrameDesc>(ctx->frames),
                         P<uint2>(ctx->ranges), svals, P<Record>(ctx->rec),
                         P<uint32_t>(ctx->keyoff), P<uint32_t>(ctx->nproc), s.background, g_rgb,
                         g_depth, g_alpha,
                         P<float>(ctx->t_final), P<int32_t>(ctx->n_last),
                         P<float>(ctx->partial), P<uint32_t>(ctx->stamp), d_epoch,
                         P<uint32_t>(ctx->order_b), remap,
                         (s.flags & GSR_FLAG_MEDIAN_DEPTH) ? P<int32_t>(ctx->med_pos) : nullptr,
                         segments, P<double2>(ctx->bwd_maps));
  }
  // A9-A11 per-record reduce, chain rule, twist
  const int64_t waves = sv.n > 0 ? preprocess_bwd_waves(sv.n) : 0;
  if ((rc = ensure(ctx, ctx->twist_part, (size_t)std::max<int64_t>(waves, 1) * sv.F * 6 * 8, st)))
    return rc;
  if ((rc = ensure(ctx, ctx->grad2d, (size_t)sv.n * sv.F * kNG * 8, st))) return rc;
  const uint64_t M = (uint64_t)sv.n * sv.F;
  if ((rc = ensure(ctx, ctx->cls_order, M * 4, st))) return rc;
  {
    StageTimer t(ctx, st, timing, GSR_STAGE_PREPROCESS_BWD);
    uint32_t* first_wide = (uint32_t*)(P<uint64_t>(ctx->counters) + 6);
    launch_class_order(st, M, P<uint32_t>(ctx->ntiles), P<uint32_t>(ctx->cls_order),
                       wide_class(), first_wide, P<uint32_t>(ctx->hist),
                       P<uint32_t>(ctx->scan_tmp));
    launch_preprocess_bwd(st, sv.n, sv.F, P<FrameDesc>(ctx->frames), sv.poses, sv.means,
                          sv.log_scales, sv.quats, sv.opac, sv.sh, s.sh_degree,
                          P<Record>(ctx->rec),
                          P<uint32_t>(ctx->cls_order), first_wide,
                          P<uint32_t>(ctx->keyoff), P<uint32_t>(ctx->ntiles), P<float>(ctx->partial),
                          P<uint32_t>(ctx->stamp), d_epoch, ctx->key_cap,
                          P<double>(ctx->grad2d), g_means, g_log_scales, g_quats, g_opac, g_sh,
                          P<double>(ctx->twist_part), g_twist);
  }
  GSR_HIP(hipGetLastError());
  sv.has_backward = true;
  return GSR_OK;
}

gsr_status gsr_densify_stats(gsr_context* ctx, float* grad_accum, float* count, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  const Saved& sv = ctx->s;
  if (!sv.valid || !sv.has_backward)
    return fail(ctx, GSR_ERR_STATE, "densify statistics need a forward and its backward");
  if (sv.n > 0 && (!grad_accum || !count))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer is NULL");
  if ((((uintptr_t)grad_accum) | ((uintptr_t)count)) & 3u)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer not 4-aligned");
  GSR_HIP(hipSetDevice(ctx->device));
  launch_densify_stats((hipStream_t)stream, sv.n, sv.F, P<uint32_t>(ctx->ntiles),
                       P<double>(ctx->grad2d), grad_accum, count);
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_mcmc_noise(gsr_context* ctx, int64_t n, float* means, const float* log_scales,
                          const float* quats, const float* opacity_logits, const float* eps,
                          float scale, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  if (n < 0) return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "n < 0");
  if (n > 0 && (!means || !log_scales || !quats || !opacity_logits || !eps))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer is NULL");
  const void* ptrs[] = {means, log_scales, quats, opacity_logits, eps};
  for (const void* p : ptrs)
    if (((uintptr_t)p) & 3u) return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer not 4-aligned");
  if (!std::isfinite(scale)) return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "scale not finite");
  GSR_HIP(hipSetDevice(ctx->device));
  launch_mcmc_noise((hipStream_t)stream, n, means, log_scales, quats, opacity_logits, eps, scale);
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_mcmc_relocate(gsr_context* ctx, int64_t n, int32_t sh_degree, float* means,
                             float* log_scales, float* quats, float* opacity_logits, float* sh,
                             const int32_t* src, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  if (n < 0 || sh_degree < 0 || sh_degree > 3)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "n < 0 or sh_degree outside 0..3");
  if (n > 0 && (!means || !log_scales || !quats || !opacity_logits || !sh || !src))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer is NULL");
  const void* ptrs[] = {means, log_scales, quats, opacity_logits, sh, src};
  for (const void* p : ptrs)
    if (((uintptr_t)p) & 3u) return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer not 4-aligned");
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  gsr_status rc;
  if ((rc = ensure(ctx, ctx->reloc_cnt, (size_t)n * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->reloc_rule, (size_t)n * 32, st))) return rc;
  const int ksh3 = 3 * (sh_degree + 1) * (sh_degree + 1);
  launch_mcmc_relocate(st, n, ksh3, means, log_scales, quats, opacity_logits, sh, src,
                       P<uint32_t>(ctx->reloc_cnt), P<double>(ctx->reloc_rule));
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_loss_l1(gsr_context* ctx, const float* target_rgb, const float* target_depth,
                       float depth_weight, float* loss, float* g_rgb, float* g_depth,
                       float* g_alpha, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  Saved& sv = ctx->s;
  if (!sv.valid) return fail(ctx, GSR_ERR_STATE, "loss without a preceding forward");
  if (!target_rgb || !target_depth || !loss || !g_rgb || !g_depth || !g_alpha)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer is NULL");
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  const int bx = loss_blocks_x(sv.max_hw);
  gsr_status rc;
  if ((rc = ensure(ctx, ctx->loss_part, (size_t)bx * sv.F * 3 * 8, st))) return rc;
  if ((rc = ensure(ctx, ctx->loss_scale, (size_t)sv.F * 2 * 4, st))) return rc;
  {
    StageTimer t(ctx, st, (sv.set.flags & GSR_FLAG_TIMING) != 0, GSR_STAGE_LOSS);
    launch_loss_l1(st, sv.F, bx, P<FrameDesc>(ctx->frames), sv.rgb, sv.depth, target_rgb,
                   target_depth, depth_weight, P<double>(ctx->loss_part),
                   P<float>(ctx->loss_scale), loss, g_rgb, g_depth, g_alpha);
  }
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_loss_l1_noalloc(gsr_context* ctx, const float* target_rgb,
                               const float* target_depth, float depth_weight, float* loss,
                               float* g_rgb, float* g_depth, float* g_alpha, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  Saved& sv = ctx->s;
  if (!sv.valid) return fail(ctx, GSR_ERR_STATE, "loss without a preceding forward");
  if (!target_rgb || !target_depth || !loss || !g_rgb || !g_depth || !g_alpha)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer is NULL");
  if (!ctx->loss_scratch) return fail(ctx, GSR_ERR_STATE, "static scratch not resolved");
  const int bx = loss_blocks_x(sv.max_hw);
  // [F][bx][3] doubles, then [F][2] floats
  const size_t part_bytes = (size_t)bx * sv.F * 3 * 8;
  const size_t need = part_bytes + (size_t)sv.F * 2 * 4;
  if (need > loss_scratch_bytes())
    return fail(ctx, GSR_ERR_UNSUPPORTED,
                "%d frames of up to %lld pixels need %zu bytes of loss scratch; the static "
                "buffer holds %zu (use gsr_loss_l1)",
                sv.F, (long long)sv.max_hw, need, loss_scratch_bytes());
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  unsigned char* base = static_cast<unsigned char*>(ctx->loss_scratch);
  launch_loss_l1(st, sv.F, bx, P<FrameDesc>(ctx->frames), sv.rgb, sv.depth, target_rgb,
                 target_depth, depth_weight, reinterpret_cast<double*>(base),
                 reinterpret_cast<float*>(base + part_bytes), loss, g_rgb, g_depth, g_alpha);
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_loss_render(gsr_context* ctx, const float* rgb, const float* depth,
                           const float* target_rgb, const float* target_depth, float lambda1,
                           float lambda2, float* loss, float* ssim, float* g_rgb, float* g_depth,
                           float* g_alpha, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  Saved& sv = ctx->s;
  if (!sv.valid) return fail(ctx, GSR_ERR_STATE, "loss without a preceding forward");
  if (!rgb || !depth || !target_rgb || !target_depth || !loss || !g_rgb || !g_depth || !g_alpha)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer is NULL");
  if (!(lambda1 >= 0.0f && lambda1 <= 1.0f) || !(lambda2 >= 0.0f && lambda2 <= 1.0f))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "lambda1/lambda2 outside [0, 1]");
  const void* ptrs[] = {rgb, depth, target_rgb, target_depth, loss, ssim, g_rgb, g_depth, g_alpha};
  for (const void* p : ptrs)
    if (((uintptr_t)p) & 3u) return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer not 4-aligned");
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  const SsimPlan plan = ssim_plan(ctx->last_frames.data(), sv.F);
  if (sv.F > 65535) return fail(ctx, GSR_ERR_UNSUPPORTED, "more than 65535 frames");
  gsr_status rc;
  // the gradient of one pixel needs its neighbours' colours: a g_rgb in the
  // place of an image is written beside it first (a buffer that every call
  // reserves: a capture in place may follow a call that was not)
  const bool in_place = g_rgb == rgb || g_rgb == target_rgb;
  if ((rc = ensure(ctx, ctx->ssim_rgb, (size_t)sv.P * 3 * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->ssim_tiles, (size_t)sv.F * 3 * plan.units_max * 4 * 8, st)))
    return rc;
  if ((rc = ensure(ctx, ctx->ssim_scale, (size_t)sv.F * 2 * 8, st))) return rc;
  {
    StageTimer t(ctx, st, (sv.set.flags & GSR_FLAG_TIMING) != 0, GSR_STAGE_LOSS);
    launch_loss_render(st, sv.F, plan, P<FrameDesc>(ctx->frames), rgb, depth, target_rgb,
                       target_depth, lambda1, lambda2, P<double>(ctx->ssim_tiles),
                       P<double>(ctx->ssim_scale), loss, ssim,
                       in_place ? P<float>(ctx->ssim_rgb) : g_rgb, g_depth, g_alpha);
    if (in_place)
      GSR_HIP(hipMemcpyAsync(g_rgb, ctx->ssim_rgb.p, (size_t)sv.P * 3 * 4,
                             hipMemcpyDeviceToDevice, st));
  }
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_step_render(gsr_context* ctx, const gsr_settings* s, int64_t n, const float* means,
                           const float* log_scales, const float* quats, const float* opac,
                           const float* sh, int32_t F, const gsr_camera* cams, const float* poses,
                           const float* target_rgb, const float* target_depth, float lambda1,
                           float lambda2, float* rgb, float* depth, float* alpha, float* loss,
                           float* ssim, float* g_means, float* g_log_scales, float* g_quats,
                           float* g_opac, float* g_sh, float* g_twist, void* stream) {
  gsr_status rc = gsr_forward(ctx, s, n, means, log_scales, quats, opac, sh, F, cams, poses,
                              rgb, depth, alpha, stream);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  const size_t npix = (size_t)ctx->s.P;
  if ((rc = ensure(ctx, ctx->up_rgb, npix * 3 * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->up_depth, npix * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->up_alpha, npix * 4, st))) return rc;
  rc = gsr_loss_render(ctx, rgb, depth, target_rgb, target_depth, lambda1, lambda2, loss, ssim,
                       P<float>(ctx->up_rgb), P<float>(ctx->up_depth), P<float>(ctx->up_alpha),
                       stream);
  if (rc) return rc;
  return gsr_backward(ctx, P<float>(ctx->up_rgb), P<float>(ctx->up_depth),
                      P<float>(ctx->up_alpha), g_means, g_log_scales, g_quats, g_opac, g_sh,
                      g_twist, stream);
}

gsr_status gsr_step_l1(gsr_context* ctx, const gsr_settings* s, int64_t n, const float* means,
                       const float* log_scales, const float* quats, const float* opac,
                       const float* sh, int32_t F, const gsr_camera* cams, const float* poses,
                       const float* target_rgb, const float* target_depth, float depth_weight,
                       float* rgb, float* depth, float* alpha, float* loss, float* g_means,
                       float* g_log_scales, float* g_quats, float* g_opac, float* g_sh,
                       float* g_twist, void* stream) {
  gsr_status rc = gsr_forward(ctx, s, n, means, log_scales, quats, opac, sh, F, cams, poses,
                              rgb, depth, alpha, stream);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  const size_t npix = (size_t)ctx->s.P;
  if ((rc = ensure(ctx, ctx->up_rgb, npix * 3 * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->up_depth, npix * 4, st))) return rc;
  if ((rc = ensure(ctx, ctx->up_alpha, npix * 4, st))) return rc;
  rc = gsr_loss_l1(ctx, target_rgb, target_depth, depth_weight, loss, P<float>(ctx->up_rgb),
                   P<float>(ctx->up_depth), P<float>(ctx->up_alpha), stream);
  if (rc) return rc;
  return gsr_backward(ctx, P<float>(ctx->up_rgb), P<float>(ctx->up_depth),
                      P<float>(ctx->up_alpha), g_means, g_log_scales, g_quats, g_opac, g_sh,
                      g_twist, stream);
}

gsr_status gsr_autotune(gsr_context* ctx, const gsr_settings* base, int64_t n, const float* means,
                        const float* log_scales, const float* quats, const float* opac,
                        const float* sh, int32_t F, const gsr_camera* cams, const float* poses,
                        const float* target_rgb, const float* target_depth, float depth_weight,
                        int32_t reps, int32_t force, gsr_settings* chosen, float* ms_out,
                        void* stream) {
  static const int kShapes[GSR_TUNE_TILES][2] = {{16, 16}, {8, 8}, {32, 8}, {16, 8}, {32, 16}};
  constexpr int kConfigs = GSR_TUNE_TILES * GSR_TUNE_BATCHES;
  if (!ctx || !base || !chosen || !cams || F < 1) return GSR_ERR_INVALID_ARGUMENT;
  if (reps < 1) reps = 1;
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  // cache key: the multiset of frame sizes, n rounded up to a power of two,
  // SH degree
  std::vector<std::pair<int, int>> sizes;
  for (int f = 0; f < F; ++f) sizes.push_back({cams[f].width, cams[f].height});
  std::sort(sizes.begin(), sizes.end());
  std::string key = "d" + std::to_string(base->sh_degree) + ":n";
  int64_t nb = 1;
  while (nb < n) nb <<= 1;
  key += std::to_string(nb);
  for (const auto& wh : sizes) key += ":" + std::to_string(wh.first) + "x" + std::to_string(wh.second);
  if (!force) {
    auto it = ctx->tune_cache.find(key);
    if (it != ctx->tune_cache.end()) {
      *chosen = it->second;
      if (ms_out)
        for (int i = 0; i < kConfigs; ++i) ms_out[i] = -1.0f;
      return GSR_OK;
    }
  }
  int64_t npx = 0;
  for (int f = 0; f < F; ++f) npx += (int64_t)cams[f].width * cams[f].height;
  const int nbasis = (base->sh_degree + 1) * (base->sh_degree + 1);
  // scratch: rgb 3P, depth P, alpha P, loss 1, grads 3n + 3n + 4n + n + 3 nb n, twist 6F
  const size_t floats = (size_t)5 * npx + 1 + (size_t)n * (11 + 3 * nbasis) + 6 * F + 64;
  gsr_status rc = ensure(ctx, ctx->tune_out, floats * 4, st);
  if (rc) return rc;
  float* o = P<float>(ctx->tune_out);
  float *rgb = o, *depth = rgb + 3 * npx, *alpha = depth + npx, *loss = alpha + npx;
  float *gm = loss + 1, *gl = gm + 3 * n, *gq = gl + 3 * n, *go = gq + 4 * n;
  float *gsh = go + n, *gt = gsh + 3 * nbasis * n;
  hipEvent_t e0, e1;
  GSR_HIP(hipEventCreate(&e0));
  GSR_HIP(hipEventCreate(&e1));
  float best = 1e30f;
  gsr_settings best_s = *base;
  for (int i = 0; i < GSR_TUNE_TILES && !rc; ++i) {
    gsr_settings s = *base;
    s.tile_w = kShapes[i][0];
    s.tile_h = kShapes[i][1];
    s.lds_batch = kWave;
    s.key_capacity = 0;
    s.flags &= ~(uint32_t)(GSR_FLAG_TIMING | GSR_FLAG_COUNT_PAIRS);
    // one sizing run per tile shape
    rc = gsr_step_l1(ctx, &s, n, means, log_scales, quats, opac, sh, F, cams, poses, target_rgb,
                     target_depth, depth_weight, rgb, depth, alpha, loss, gm, gl, gq, go, gsh, gt,
                     stream);
    if (rc) break;
    s.key_capacity = (int64_t)(ctx->s.K + ctx->s.K / 20 + 1024);
    std::vector<float> t(reps);
    for (int r = 0; r < reps && !rc; ++r) {
      GSR_HIP(hipEventRecord(e0, st));
      rc = gsr_step_l1(ctx, &s, n, means, log_scales, quats, opac, sh, F, cams, poses,
                       target_rgb, target_depth, depth_weight, rgb, depth, alpha, loss, gm, gl,
                       gq, go, gsh, gt, stream);
      GSR_HIP(hipEventRecord(e1, st));
      GSR_HIP(hipEventSynchronize(e1));
      GSR_HIP(hipEventElapsedTime(&t[r], e0, e1));
    }
    if (rc) break;
    if ((rc = gsr_check_overflow(ctx, stream))) break;
    std::sort(t.begin(), t.end());
    const float med = t[reps / 2];
    // the time does not depend on lds_batch
    for (int j = 0; ms_out && j < GSR_TUNE_BATCHES; ++j) ms_out[i * GSR_TUNE_BATCHES + j] = med;
    if (med < best) {
      best = med;
      best_s = s;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc) return rc;
  ctx->s.valid = false;  // the scratch outputs are not the caller's
  *chosen = best_s;
  ctx->tune_cache[key] = best_s;
  return GSR_OK;
}

gsr_status gsr_adam_step(gsr_context* ctx, int64_t n, int32_t sh_degree, float* means,
                         const float* g_means, float* m_means, float* v_means, float* sh,
                         const float* g_sh, float* m_sh, float* v_sh, int32_t F, float* poses,
                         const float* g_twist, float* m_twist, float* v_twist, float lr_means,
                         float lr_sh, float lr_pose, float beta1, float beta2, float eps,
                         int32_t* step, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  if (n < 0 || F < 0 || F > 1024 || sh_degree < 0 || sh_degree > 3 || !step)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "adam: bad sizes or NULL step");
  if (n > 0 && (!means || !g_means || !m_means || !v_means || !sh || !g_sh || !m_sh || !v_sh))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "adam: Gaussian buffer is NULL");
  if (F > 0 && (!poses || !g_twist || !m_twist || !v_twist))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "adam: pose buffer is NULL");
  if (!(beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f && beta2 < 1.0f && eps >= 0.0f))
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "adam: bad hyper-parameters");
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  const uint64_t nb = (uint64_t)(sh_degree + 1) * (sh_degree + 1);
  launch_adam(st, (uint64_t)n * 3, (uint64_t)n * nb * 3, means, g_means, m_means, v_means, sh,
              g_sh, m_sh, v_sh, F, poses, g_twist, m_twist, v_twist, lr_means, lr_sh, lr_pose,
              beta1, beta2, eps, step);
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_check_overflow(gsr_context* ctx, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  if (!ctx->counters.p) return GSR_OK;
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  GSR_HIP(hipMemcpyAsync(ctx->h_count, ctx->counters.p, 16, hipMemcpyDeviceToHost, st));
  GSR_HIP(hipStreamSynchronize(st));
  const uint32_t flag = (uint32_t)(ctx->h_count[1] & 0xffffffffu);
  if (flag) {
    launch_fill_u32(st, (uint32_t*)(P<uint64_t>(ctx->counters) + 1), 1, 0u);
    GSR_HIP(hipStreamSynchronize(st));
    return fail(ctx, GSR_ERR_CAPACITY, "%llu keys exceeded the fixed key capacity",
                (unsigned long long)ctx->h_count[0]);
  }
  return GSR_OK;
}

gsr_status gsr_debug_stats(gsr_context* ctx, gsr_stats* out, void* stream) {
  if (!ctx || !out) return GSR_ERR_INVALID_ARGUMENT;
  const Saved& sv = ctx->s;
  if (!sv.valid) return fail(ctx, GSR_ERR_STATE, "no forward");
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  unsigned long long* cull = (unsigned long long*)(P<uint64_t>(ctx->counters) + 4);
  launch_fill_u32(st, (uint32_t*)cull, 4, 0u);
  const int nb3 = 3 * (sv.set.sh_degree + 1) * (sv.set.sh_degree + 1);
  launch_cull_stats(st, (uint64_t)sv.n * sv.F, P<uint32_t>(ctx->ntiles), sv.n, sv.means,
                    sv.log_scales, sv.surfel ? 2 : 3, sv.quats, sv.opac, sv.sh, nb3, cull);
  GSR_HIP(hipGetLastError());
  GSR_HIP(hipMemcpyAsync(ctx->h_count, ctx->counters.p, 48, hipMemcpyDeviceToHost, st));
  GSR_HIP(hipStreamSynchronize(st));
  out->n_pairs = ctx->n_pairs == -2 ? (int64_t)ctx->h_count[2] : -1;
  out->n_culled = (int64_t)ctx->h_count[4];
  out->n_nonfinite = (int64_t)ctx->h_count[5];
  out->n_records = sv.n * sv.F;
  out->n_keys = (int64_t)ctx->h_count[0];
  out->n_tiles = sv.T;
  out->n_pixels = sv.P;
  out->key_capacity = (int64_t)ctx->key_cap;
  out->epoch = ctx->epoch;
  out->tile_w = sv.set.tile_w;
  out->tile_h = sv.set.tile_h;
  return GSR_OK;
}

gsr_status gsr_debug_timings(gsr_context* ctx, double* ms, int64_t* calls) {
  if (!ctx || !ms || !calls) return GSR_ERR_INVALID_ARGUMENT;
  for (int i = 0; i < GSR_N_STAGES; ++i) {
    ms[i] = 0.0;
    calls[i] = 0;
  }
  GSR_HIP(hipSetDevice(ctx->device));
  gsr_status rc = GSR_OK;
  for (auto& t : ctx->timed) {
    float e = 0.0f;
    if (rc == GSR_OK) {
      hipError_t err = hipEventSynchronize(t.b);
      if (err == hipSuccess) err = hipEventElapsedTime(&e, t.a, t.b);
      if (err != hipSuccess) rc = hip_check(ctx, err, "hipEventElapsedTime");
    }
    if (t.stage >= 0 && t.stage < GSR_N_STAGES) {
      ms[t.stage] += e;
      calls[t.stage] += 1;
    }
    ctx->ev_pool.push_back(t.a);
    ctx->ev_pool.push_back(t.b);
  }
  ctx->timed.clear();
  return rc;
}

gsr_status gsr_debug_lists(gsr_context* ctx, uint32_t* ntiles, uint32_t* depth_key,
                           uint32_t* square, uint32_t* tile_keys, uint32_t* tile_vals,
                           uint32_t* ranges, int32_t* n_last, float* t_final, void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  const Saved& sv = ctx->s;
  if (!sv.valid) return fail(ctx, GSR_ERR_STATE, "no forward");
  hipStream_t st = (hipStream_t)stream;
  GSR_HIP(hipSetDevice(ctx->device));
  GSR_HIP(hipStreamSynchronize(st));
  const size_t M = (size_t)sv.n * sv.F;
  uint64_t K = 0;
  GSR_HIP(hipMemcpy(&K, ctx->counters.p, 8, hipMemcpyDeviceToHost));
  K = std::min<uint64_t>(K, ctx->key_cap);
  if (ntiles && M) GSR_HIP(hipMemcpy(ntiles, ctx->ntiles.p, M * 4, hipMemcpyDeviceToHost));
  if (depth_key && M) {
    // the depth keys were sorted in place; rebuild the per-record view
    std::vector<uint32_t> k(M), v(M);
    const DBuf& kb = ctx->dkey_a;
    const DBuf& vb = ctx->dval_a;
    GSR_HIP(hipMemcpy(k.data(), kb.p, M * 4, hipMemcpyDeviceToHost));
    GSR_HIP(hipMemcpy(v.data(), vb.p, M * 4, hipMemcpyDeviceToHost));
    for (size_t i = 0; i < M; ++i) depth_key[v[i]] = k[i];
  }
  if (square && M) {
    const size_t rb = sv.surfel ? surfel_record_bytes() : sizeof(Record);
    const size_t off = sv.surfel ? surfel_square_offset() : offsetof(Record, sqx);
    std::vector<uint8_t> r(M * rb);
    GSR_HIP(hipMemcpy(r.data(), ctx->rec.p, M * rb, hipMemcpyDeviceToHost));
    for (size_t i = 0; i < M; ++i) {
      std::memcpy(&square[2 * i], &r[i * rb + off], 8);  // sqx, sqy
    }
  }
  const DBuf& kb = sv.sorted_in_b ? ctx->keys_b : ctx->keys_a;
  const DBuf& vb = sv.sorted_in_b ? ctx->vals_b : ctx->vals_a;
  if (tile_keys && K) {
    if (sv.keys16) {  // widened, the 16-bit sentinel to the 32-bit one
      std::vector<uint16_t> k16(K);
      GSR_HIP(hipMemcpy(k16.data(), kb.p, K * 2, hipMemcpyDeviceToHost));
      for (uint64_t i = 0; i < K; ++i)
        tile_keys[i] = k16[i] == 0xffffu ? 0xffffffffu : (uint32_t)k16[i];
    } else {
      GSR_HIP(hipMemcpy(tile_keys, kb.p, K * 4, hipMemcpyDeviceToHost));
    }
  }
  if (tile_vals && K) GSR_HIP(hipMemcpy(tile_vals, vb.p, K * 4, hipMemcpyDeviceToHost));
  if (ranges && sv.T) GSR_HIP(hipMemcpy(ranges, ctx->ranges.p, sv.T * 8, hipMemcpyDeviceToHost));
  if (n_last && sv.P) GSR_HIP(hipMemcpy(n_last, ctx->n_last.p, sv.P * 4, hipMemcpyDeviceToHost));
  if (t_final && sv.P) GSR_HIP(hipMemcpy(t_final, ctx->t_final.p, sv.P * 4, hipMemcpyDeviceToHost));
  return GSR_OK;
}

gsr_status gsr_debug_copy(gsr_context* ctx, const void* src, void* dst, uint64_t bytes,
                          void* stream) {
  if (!ctx) return GSR_ERR_INVALID_ARGUMENT;
  if (bytes == 0) return GSR_OK;
  if (!src || !dst) return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointer is NULL");
  if ((((uintptr_t)src) | ((uintptr_t)dst) | bytes) & 15u)
    return fail(ctx, GSR_ERR_INVALID_ARGUMENT, "pointers and size must be 16-byte multiples");
  GSR_HIP(hipSetDevice(ctx->device));
  launch_copy16((hipStream_t)stream, src, dst, bytes / 16);
  GSR_HIP(hipGetLastError());
  return GSR_OK;
}

gsr_status gsr_debug_grad2d(gsr_context* ctx, double* out, void* stream) {
  if (!ctx || !out) return GSR_ERR_INVALID_ARGUMENT;
  const Saved& sv = ctx->s;
  if (!sv.valid) return fail(ctx, GSR_ERR_STATE, "no forward");
  const size_t bytes = (size_t)sv.n * sv.F * kNG * 8;
  if (bytes == 0) return GSR_OK;
  if (ctx->grad2d.bytes < bytes) return fail(ctx, GSR_ERR_STATE, "no backward");
  GSR_HIP(hipSetDevice(ctx->device));
  GSR_HIP(hipStreamSynchronize((hipStream_t)stream));
  std::vector<double> parts(bytes / 8);
  GSR_HIP(hipMemcpy(parts.data(), ctx->grad2d.p, bytes, hipMemcpyDeviceToHost));
  const uint64_t m = (uint64_t)sv.n * sv.F;
  for (uint64_t r = 0; r < m; ++r)
    for (int j = 0; j < kNG; ++j) out[r * kNG + j] = parts[grad2d_at(r, j, m)];
  return GSR_OK;
}

}  // extern "C"
