// Host side of the C ABI declared in lococo.h: argument validation, the
// integer plan of the scan (Alg. 2 loop and IF), path selection and kernel
// sequencing.  No arithmetic of the method happens here.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "lococo_internal.h"

using namespace lococo;

// The library's own scratch array (see lococo_segment_step_noalloc): device memory that exists from
// the moment the code object is loaded.  On the host this name is only a handle for
// hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[LOCOCO_NOALLOC_SCRATCH_BYTES];

namespace {
DebugOptions g_debug = {0, 0, 0, 0, 0, 0, 0};
}
namespace lococo {
const DebugOptions& debug_options() { return g_debug; }
int cu_count() {
  static int n = 0;
  if (!n) {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
      n = prop.multiProcessorCount;
    if (n <= 0) n = 256;
  }
  return n;
}
}  // namespace lococo

namespace {

thread_local char g_err[512] = "";

lococo_status fail(lococo_status st, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return st;
}

lococo_status hip_fail(hipError_t e, const char* what) {
  return fail(LOCOCO_EHIP, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(expr, what)                         \
  do {                                              \
    hipError_t e_ = (expr);                         \
    if (e_ != hipSuccess) return hip_fail(e_, what); \
  } while (0)

// ---- optional per-kernel timing with HIP events (lococo_timing_begin / _end)
enum KernelId { K_ATTN_GENERIC, K_FILL, K_CONV_GENERIC, K_NORM_GENERIC, K_MIX_GENERIC,
                K_REPACK, K_COMPRESS_MFMA, K_ATTN_MFMA, K_ATTN_DECODE, K_ATTN_COLSUM, K_CONV_MFMA, K_MIX_MFMA,
                K_COMPRESS_SMALL, K_BWD_WALK, K_COUNT };
const char* const kKernelNames[K_COUNT] = {"attn_generic", "fill", "conv_logits_generic",
                                           "normalise_generic", "mix_generic", "repack_filters",
                                           "compress_mfma", "attn_mfma", "attn_decode", "attn_colsum",
                                           "conv_logits_mfma", "mix_mfma", "compress_small", "bwd_walk"};
struct TimedLaunch { int id; hipEvent_t start, stop; };
std::mutex g_timing_mu;
bool g_timing_on = false;
std::vector<TimedLaunch> g_timed;

// Records an event pair around the launches made while it is alive.
struct KTimer {
  int id;
  hipStream_t s;
  hipEvent_t start = nullptr, stop = nullptr;
  KTimer(int id_, hipStream_t s_) : id(id_), s(s_) {
    if (!g_timing_on) return;
    if (hipEventCreate(&start) != hipSuccess || hipEventCreate(&stop) != hipSuccess) {
      start = stop = nullptr;
      return;
    }
    (void)hipEventRecord(start, s);
  }
  void drop() {                            // nothing was launched after all
    if (!start) return;
    (void)hipEventDestroy(start);
    (void)hipEventDestroy(stop);
    start = stop = nullptr;
  }
  ~KTimer() {
    if (!start) return;
    (void)hipEventRecord(stop, s);
    std::lock_guard<std::mutex> lk(g_timing_mu);
    g_timed.push_back(TimedLaunch{id, start, stop});
  }
};

size_t esize(int dtype) { return dtype == LOCOCO_F32 ? 4 : 2; }
size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

lococo_status check_config(const lococo_config* c) {
  if (!c) return fail(LOCOCO_EINVAL, "config is NULL");
  if (c->struct_size != sizeof(lococo_config))
    return fail(LOCOCO_EINVAL, "config.struct_size is %u, this library expects %zu", c->struct_size,
                sizeof(lococo_config));
  if (c->dtype != LOCOCO_F32 && c->dtype != LOCOCO_BF16)
    return fail(LOCOCO_EINVAL, "config.dtype %d is neither LOCOCO_F32 nor LOCOCO_BF16", c->dtype);
  if (c->batch <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0 || c->head_dim <= 0 || c->M <= 0)
    return fail(LOCOCO_EINVAL, "batch, head counts, head_dim and M must be positive");
  if (c->n_q_heads % c->n_kv_heads)
    return fail(LOCOCO_EINVAL, "n_q_heads (%d) is not a multiple of n_kv_heads (%d)", c->n_q_heads,
                c->n_kv_heads);
  if (c->conv_width < 1) return fail(LOCOCO_EINVAL, "conv_width must be >= 1");
  if (c->conv_width % 2 == 0)
    return fail(LOCOCO_EUNSUPPORTED, "conv_width %d is even; only odd widths have a centred "
                "same-length convolution", c->conv_width);
  if (c->conv_in != 0 && c->conv_in != 1) return fail(LOCOCO_EINVAL, "conv_in must be 0 or 1");
  if (c->norm < 0 || c->norm > 2) return fail(LOCOCO_EINVAL, "norm must be 0, 1 or 2");
  if (c->impl < LOCOCO_IMPL_AUTO || c->impl > LOCOCO_IMPL_MFMA)
    return fail(LOCOCO_EINVAL, "impl must be one of LOCOCO_IMPL_*");
  if (c->flags & ~LOCOCO_FLAG_FILTERS_PREPARED) return fail(LOCOCO_EINVAL, "config.flags has unknown bits set");
  if (c->w_head_stride < 0 || c->b_head_stride < 0)
    return fail(LOCOCO_EINVAL, "filter head strides must be >= 0");
  if (!(c->attn_scale >= 0.f) || !(c->norm_eps >= 0.f) || std::isinf(c->attn_scale))
    return fail(LOCOCO_EINVAL, "attn_scale and norm_eps must be finite and >= 0");
  if (c->head_dim > 1024) return fail(LOCOCO_EUNSUPPORTED, "head_dim > 1024");
  if (c->n_q_heads > 65535 || c->batch > 65535 || c->M > 65535 ||
      (int64_t)c->batch * c->n_kv_heads > 65535)
    return fail(LOCOCO_EUNSUPPORTED, "batch, heads, M or batch*n_kv_heads above 65535");
  return LOCOCO_OK;
}

lococo_status check_tensor(const lococo_config* c, const lococo_tensor& t, const char* name,
                           int64_t tokens) {
  if (!t.p) return fail(LOCOCO_EINVAL, "%s pointer is NULL", name);
  if (t.stride_t < c->head_dim)
    return fail(LOCOCO_EINVAL, "%s.stride_t (%lld) is below head_dim", name, (long long)t.stride_t);
  if (t.stride_h < 0 || t.stride_b < 0)
    return fail(LOCOCO_EINVAL, "%s strides must be non-negative", name);
  if (c->dtype == LOCOCO_BF16 &&
      ((t.stride_t | t.stride_h | t.stride_b) % 8 || ((uintptr_t)t.p & 15)))
    return fail(LOCOCO_EINVAL, "%s: bf16 tensors need 16-byte aligned pointers and strides that "
                "are multiples of 8 elements", name);
  if (c->dtype == LOCOCO_F32 && ((uintptr_t)t.p & 3))
    return fail(LOCOCO_EINVAL, "%s pointer is not 4-byte aligned", name);
  (void)tokens;
  return LOCOCO_OK;
}

lococo_status check_cache(const lococo_config* c, const lococo_cache* ca) {
  if (!ca) return fail(LOCOCO_EINVAL, "cache is NULL");
  for (int i = 0; i < 2; ++i) {
    if (!ca->k[i] || !ca->v[i]) return fail(LOCOCO_EINVAL, "cache buffer pointer is NULL");
    if (((uintptr_t)ca->k[i] | (uintptr_t)ca->v[i]) & 15)
      return fail(LOCOCO_EINVAL, "cache buffers must be 16-byte aligned");
  }
  const void* p[4] = {ca->k[0], ca->k[1], ca->v[0], ca->v[1]};
  for (int i = 0; i < 4; ++i)
    for (int j = i + 1; j < 4; ++j)
      if (p[i] == p[j]) return fail(LOCOCO_EINVAL, "cache buffers alias each other");
  if (ca->cur != 0 && ca->cur != 1) return fail(LOCOCO_ESTATE, "cache.cur is %d", ca->cur);
  if (ca->len < 0 || ca->len > c->M)
    return fail(LOCOCO_ESTATE, "cache.len %d is outside [0, M=%d]", ca->len, c->M);
  if (ca->protect) {
    if ((uintptr_t)ca->protect & 3) return fail(LOCOCO_EINVAL, "cache.protect is not 4-byte aligned");
    if (ca->protect_chain_stride != 0 && ca->protect_chain_stride < (c->M + 31) / 32)
      return fail(LOCOCO_EINVAL, "cache.protect_chain_stride must be 0 or at least ceil(M / 32) words");
  }
  if ((uintptr_t)ca->attn_colsum & 3) return fail(LOCOCO_EINVAL, "cache.attn_colsum is not 4-byte aligned");
  return LOCOCO_OK;
}

lococo_status check_qkvo(const lococo_config* c, const lococo_qkvo* x, int64_t tokens,
                         bool need_q_o) {
  if (!x) return fail(LOCOCO_EINVAL, "qkvo is NULL");
  lococo_status st;
  if (need_q_o) {
    if ((st = check_tensor(c, x->q, "q", tokens))) return st;
    if ((st = check_tensor(c, x->o, "o", tokens))) return st;
    if (x->o.p == x->q.p || x->o.p == x->k.p || x->o.p == x->v.p)
      return fail(LOCOCO_EINVAL, "o aliases an input");
  }
  if ((st = check_tensor(c, x->k, "k", tokens))) return st;
  if ((st = check_tensor(c, x->v, "v", tokens))) return st;
  return LOCOCO_OK;
}

// PATH_MFMA: the fused compression kernel.  PATH_MFMA_UNFUSED: shapes it does not take (other filter
// widths, [K | V] filters, M not a multiple of 32) with bf16 storage and head_dim 128: attention on
// MFMA, Eq. 5 and Eq. 4 as two MFMA kernels around the shape-agnostic normalisation, the logits
// passing through the workspace in fp32.
enum Path { PATH_GENERIC = 0, PATH_MFMA = 1, PATH_MFMA_UNFUSED = 2 };

// Which kernels take this shape.  *why is set when the fused kernel is refused.
Path choose_path(const lococo_config* c, int32_t B, const char** why) {
  (void)B;
  const char* ignore = "";
  if (!attn_mfma_supports(c->dtype, c->head_dim, why)) return PATH_GENERIC;
  if (compress_mfma_supports(c->dtype, c->head_dim, c->M, c->conv_width, c->conv_in, c->norm, why) &&
      !(c->conv_in && g_debug.unfused_kv))
    return PATH_MFMA;
  if (c->norm != 2 &&                 // the input-side rectifier exists in the shape-agnostic kernels only
      conv_logits_mfma_supports(c->dtype, c->head_dim, c->conv_width) && attn_mfma_supports(c->dtype, c->head_dim, &ignore))
    return PATH_MFMA_UNFUSED;
  return PATH_GENERIC;
}

int filter_banks(const lococo_config* c) { return c->w_head_stride ? c->n_kv_heads : 1; }

lococo_status resolve_path(const lococo_config* c, int32_t B, Path* out) {
  const char* why = "";
  Path p = c->impl == LOCOCO_IMPL_GENERIC ? PATH_GENERIC : choose_path(c, B, &why);
  if (c->impl == LOCOCO_IMPL_MFMA && p != PATH_MFMA)     // MFMA means the fused kernel, nothing less
    return fail(LOCOCO_EUNSUPPORTED, "impl = MFMA requested but %s", why);
  *out = p;
  return LOCOCO_OK;
}

// Workspace of one step.  Generic: fp32 logits [chains, M, T], T <= M + B.
// MFMA: the repacked filter bank.
size_t filter_ws_bytes(const lococo_config* c) {
  return align_up(compress_mfma_filter_bytes(c->M, c->conv_width, c->conv_in, filter_banks(c)), 256);
}
// chain sync counters + status word of the one-launch scan
size_t scan_sync_bytes(const lococo_config* c) {
  return align_up(compress_scan_sync_bytes(c->batch, c->n_kv_heads, c->M), 256);
}
// softmax statistics of `rows` query rows per head (what the column sums of the MFMA attention need)
size_t stats_bytes(const lococo_config* c, int64_t rows) {
  return align_up((size_t)c->batch * c->n_q_heads * (size_t)rows * 2 * sizeof(float), 256);
}
// filters packed per tap for the unfused MFMA path
size_t packed_ws_bytes(const lococo_config* c) {
  return align_up(packed_filter_bytes(c->M, c->conv_width, c->conv_in, filter_banks(c)), 256);
}
size_t logits_bytes(const lococo_config* c, int32_t B) {     // rows of up to M + B logits, padded to a multiple of 4
  return align_up((size_t)c->batch * c->n_kv_heads * c->M * (((size_t)c->M + B + 3) / 4 * 4) * sizeof(float), 256);
}
// results of the parts of a split step (see compress_mfma.hip), 0 where the shape is not split
size_t partials_ws_bytes(const lococo_config* c) {
  return align_up(compress_partials_bytes(c->batch, c->n_kv_heads, c->M, c->conv_width, c->conv_in, cu_count()), 256);
}
// key-side logits between the two walks of a step over [K | V] filters (see compress_mfma.hip), 0 for filters over the keys
size_t prelogits_ws_bytes(const lococo_config* c, int32_t B) {
  return align_up(compress_prelogits_bytes(c->batch, c->n_kv_heads, c->M, B, c->conv_in, cu_count()), 256);
}
// MFMA path: [repacked filters][chain sync counters + status word][row statistics of one block][results of
// the parts of a split step][key-side logits of a step over [K | V] filters]; unfused MFMA path: [filters packed per tap][row statistics of one block][logits];
// generic path: the logits.
size_t step_ws_bytes(const lococo_config* c, Path path, int32_t B) {
  if (path == PATH_MFMA)
    return filter_ws_bytes(c) + scan_sync_bytes(c) + stats_bytes(c, B) + partials_ws_bytes(c) + prelogits_ws_bytes(c, B);
  if (path == PATH_MFMA_UNFUSED) return packed_ws_bytes(c) + stats_bytes(c, B) + logits_bytes(c, B);
  return logits_bytes(c, B);
}
void* partials_of(const lococo_config* c, void* ws, int32_t B) {
  return (char*)ws + filter_ws_bytes(c) + scan_sync_bytes(c) + stats_bytes(c, B);
}
void* prelogits_of(const lococo_config* c, void* ws, int32_t B) { return (char*)partials_of(c, ws, B) + partials_ws_bytes(c); }

// Bytes of one history slot pair member: one cache state [chains, M, d].
size_t state_bytes(const lococo_config* c) {
  return (size_t)c->batch * c->n_kv_heads * c->M * c->head_dim * esize(c->dtype);
}

// Workspace of the batched-attention schedule: the step workspace followed by
// K and V history slots for n_compress cache states.
// Layout: [step workspace][row statistics of the sequence][K history][V history].
size_t history_ws_bytes(const lococo_config* c, Path path, int32_t B, int64_t n_compress, int64_t L) {
  return step_ws_bytes(c, path, B) + stats_bytes(c, L) + 2 * (size_t)n_compress * align_up(state_bytes(c), 256);
}

// Whether the schedules that run the attention of many blocks in one launch exist for this shape.  On the shape-agnostic path
// where the compression has its one kernel too: with the separate ones, step by step is the better schedule, each block's
// attention bringing in the rows its compression reads (fp32, 8 heads of 128 on 2, ten blocks of 100 on 128 slots: 2.03 ms;
// with the states apart and the attention behind them 2.25 ms).
bool batched_attention(const lococo_config* c, Path path, int32_t B) {
  if (path != PATH_GENERIC) return true;
  return attn_rows_fits(c->M + B, c->head_dim) && small_step_fits(c->M + B, c->M, c->head_dim, c->conv_width, c->conv_in);
}

// Polls a waiting workgroup makes before it gives up on its chain (each poll sleeps ~128 cycles and
// reads the counter from the L2: roughly a microsecond, so the default bounds a wait to a few
// seconds).  The tests force the give-up path from the host with a limit of -1.
int spin_limit() {
  return g_debug.spin_limit ? (int)g_debug.spin_limit : (1 << 21);
}
// By default the slot tiles of a chain skip the L2 write-back between the steps of the one-launch
// scan when they find themselves on one XCD (see compress_mfma.hip).
bool chain_sync_through_l2() { return g_debug.chain_sync_device == 0; }

// One launch for all compression steps of a scan needs every workgroup of it resident at once: the
// grid must fit the occupancy the runtime reports for the kernel, and no other such launch of this
// process may still be running on another stream of the device (two of them could each hold part of
// the compute units and wait for workgroups that never become resident).
constexpr int kMaxDevices = 64;
struct ScanInFlight { hipEvent_t done = nullptr; hipStream_t stream = nullptr; bool valid = false; };
ScanInFlight g_scan[kMaxDevices];
std::mutex g_scan_mu;

bool stream_is_capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) { (void)hipGetLastError(); return false; }
  return st != hipStreamCaptureStatusNone;
}

// call with g_scan_mu held
bool another_scan_in_flight(hipStream_t s) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return true;
  ScanInFlight& g = g_scan[dev];
  if (!g.valid || g.stream == s) return false;        // same stream: ordered behind it
  const hipError_t e = hipEventQuery(g.done);
  if (e == hipSuccess) { g.valid = false; return false; }
  (void)hipGetLastError();
  return true;                                        // not ready (or unknown): assume it still runs
}
void note_scan_launched(hipStream_t s) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return;
  ScanInFlight& g = g_scan[dev];
  if (!g.done && hipEventCreateWithFlags(&g.done, hipEventDisableTiming) != hipSuccess) {
    (void)hipGetLastError();
    g.done = nullptr;
    return;
  }
  if (hipEventRecord(g.done, s) == hipSuccess) { g.stream = s; g.valid = true; }
  else (void)hipGetLastError();
}

// Whether the shape allows the one-launch form at all (grid rule and occupancy); the in-flight check
// is made under the lock right before the launch.
bool scan_fits_one_launch(const lococo_config* c, const StepArgs& a) {
  if (g_debug.scan_per_step) return false;
  const int groups = compress_scan_groups(c->batch, c->n_kv_heads, c->M, c->conv_width, c->conv_in,
                                          c->w_head_stride != 0 || c->b_head_stride != 0, cu_count());
  if (groups <= 0) return false;
  const int split = groups < c->batch * c->n_kv_heads
                        ? 1 : compress_position_split(c->batch, c->n_kv_heads, c->M, c->conv_width, c->conv_in, cu_count());
  const int pipe = groups < c->batch * c->n_kv_heads
                       ? 1 : compress_step_pipeline(c->batch, c->n_kv_heads, c->M, c->conv_width, c->conv_in, cu_count());
  const int64_t grid = (int64_t)groups * split * pipe *
                       (c->M / compress_tile_slots(c->batch, c->n_kv_heads, c->M, c->conv_width, c->conv_in, cu_count()));
  return grid <= compress_scan_max_resident(a, cu_count());
}

View view_at(const lococo_tensor& t, int64_t tok, size_t es) {
  return View{(const char*)t.p + (size_t)(tok * t.stride_t) * es, t.stride_b, t.stride_h, t.stride_t};
}

StepArgs make_args(const lococo_config* c, const lococo_qkvo* x, int64_t tok, int32_t Bn,
                   const lococo_cache* ca, const void* conv_w, const void* conv_b, bool with_q) {
  StepArgs a;
  std::memset(&a, 0, sizeof(a));
  const size_t es = esize(c->dtype);
  if (with_q) {
    a.q = view_at(x->q, tok, es);
    a.o = view_at(x->o, tok, es);
  }
  a.k = view_at(x->k, tok, es);
  a.v = view_at(x->v, tok, es);
  a.cache_k = ca->k[ca->cur];
  a.cache_v = ca->v[ca->cur];
  a.conv_w = conv_w;
  a.conv_b = conv_b;
  a.w_head_stride = c->w_head_stride;
  a.b_head_stride = c->b_head_stride;
  a.batch = c->batch;
  a.Hq = c->n_q_heads;
  a.Hkv = c->n_kv_heads;
  a.group = c->n_q_heads / c->n_kv_heads;
  a.d = c->head_dim;
  a.M = c->M;
  a.m = ca->len;
  a.Bn = Bn;
  a.k_width = c->conv_width;
  a.conv_in = c->conv_in;
  a.norm = c->norm;
  a.scale = c->attn_scale > 0.f ? c->attn_scale : 1.0f / std::sqrt((float)c->head_dim);
  a.eps = c->norm_eps > 0.f ? c->norm_eps : 1e-6f;
  a.protect = ca->protect;
  a.protect_stride = ca->protect_chain_stride;
  a.colsum = ca->attn_colsum;
  return a;
}

lococo_status check_step_shape(const lococo_config* c, int32_t B, int32_t len) {
  if (B <= 0) return fail(LOCOCO_EINVAL, "block length B must be positive");
  if (B > 65535) return fail(LOCOCO_EUNSUPPORTED, "block length above 65535");
  if ((int64_t)len + B > generic_attn_max_T())
    return fail(LOCOCO_EUNSUPPORTED, "cache.len + B = %lld exceeds the supported %d",
                (long long)len + B, generic_attn_max_T());
  return LOCOCO_OK;
}

// The MFMA kernels address the rows of a block with 32-bit byte offsets inside buffer resources of
// less than 2 GiB (out-of-range rows must read as zero): a block's rows have to span less than that.
lococo_status check_mfma_strides(const lococo_config* c, Path path, const lococo_qkvo* x, int32_t B, bool with_q) {
  if (path == PATH_GENERIC) return LOCOCO_OK;
  const int64_t lim = 0x7fff0000;
  const lococo_tensor* t[4] = {&x->k, &x->v, &x->q, &x->o};
  const char* names[4] = {"k", "v", "q", "o"};
  for (int i = 0; i < (with_q ? 4 : 2); ++i)
    if (((int64_t)B * t[i]->stride_t + c->head_dim) * (int64_t)esize(c->dtype) >= lim)
      return fail(LOCOCO_EUNSUPPORTED, "%s: a block of %d tokens with stride_t %lld spans 2 GiB or more; the MFMA "
                  "kernels address a block's rows with 32-bit offsets (use impl = GENERIC)", names[i], B,
                  (long long)t[i]->stride_t);
  if ((int64_t)c->M * c->head_dim * (int64_t)esize(c->dtype) >= lim)
    return fail(LOCOCO_EUNSUPPORTED, "a chain's cache spans 2 GiB or more");
  return LOCOCO_OK;
}

AttnArgs attn_args_one_block(const StepArgs& a) {
  AttnArgs t;
  std::memset(&t, 0, sizeof(t));
  t.q = a.q; t.k = a.k; t.v = a.v; t.o = a.o;
  t.cache_k = a.cache_k;
  t.cache_v = a.cache_v;
  t.L = a.Bn;
  t.B = a.Bn;
  t.M = a.M;
  t.len0 = a.m;
  t.n_fill = 0;            // block 0 sees the base cache with len0 slots
  t.hist_ring = 1;
  t.seg_first = 0;
  t.n_seg = 1;
  t.batch = a.batch; t.Hq = a.Hq; t.Hkv = a.Hkv; t.group = a.group;
  t.scale = a.scale;
  return t;
}

// Enqueue the attention of one block.  `stats`: room for the block's row statistics (see
// stats_bytes), or null; without it a block whose attention is to be accumulated per slot goes
// to the shape-agnostic kernel.
lococo_status enqueue_attn(const lococo_config* c, Path path, const StepArgs& a, float* stats, hipStream_t s) {
  if (path != PATH_GENERIC && attn_decode_supports(c->dtype, c->head_dim, a.Bn, c->M, a.colsum != nullptr)) {
    KTimer t(K_ATTN_DECODE, s);          // one query row per head: a matrix-vector product
    HIP_TRY(launch_attn_decode(a, s), "attention launch");
    return LOCOCO_OK;
  }
  if (path != PATH_GENERIC && (!a.colsum || stats)) {
    AttnArgs t = attn_args_one_block(a);
    t.stats = a.colsum ? stats : nullptr;
    {
      KTimer kt(K_ATTN_MFMA, s);
      HIP_TRY(launch_attn_mfma(t, s), "attention launch");
    }
    if (a.colsum && a.m > 0) {
      KTimer kt(K_ATTN_COLSUM, s);
      HIP_TRY(launch_attn_colsum_mfma(t, a.colsum, s), "attention column-sum launch");
    }
    return LOCOCO_OK;
  }
  KTimer t(K_ATTN_GENERIC, s);
  if (attn_rows_fits(a.m + a.Bn, a.d)) HIP_TRY(launch_attn_rows(c->dtype, attn_args_one_block(a), c->head_dim, a.colsum, s), "attention launch");
  else HIP_TRY(launch_attn_generic(c->dtype, a, s), "attention launch");
  return LOCOCO_OK;
}

// The statistics area of a step workspace, if the caller passed one that holds it.
float* step_stats(const lococo_config* c, Path path, int32_t B, void* workspace, size_t ws_bytes) {
  if (path == PATH_GENERIC || !workspace || ((uintptr_t)workspace & 255) || ws_bytes < step_ws_bytes(c, path, B))
    return nullptr;
  return (float*)((char*)workspace + (path == PATH_MFMA ? filter_ws_bytes(c) + scan_sync_bytes(c) : packed_ws_bytes(c)));
}

// Repack the filter bank into the workspace (MFMA path; once per call unless the caller says
// the workspace already holds it).
// sync_ws, fill: see launch_repack_filters (fused MFMA path, filters not prepared).
lococo_status enqueue_repack(const lococo_config* c, Path path, const StepArgs& a, void* ws, hipStream_t s, void* sync_ws = nullptr,
                             const StepArgs* fill = nullptr) {
  if (c->flags & LOCOCO_FLAG_FILTERS_PREPARED) return LOCOCO_OK;
  KTimer t(K_REPACK, s);
  if (path == PATH_MFMA) HIP_TRY(launch_repack_filters(a, ws, filter_banks(c), sync_ws, s, fill), "filter repack launch");
  else HIP_TRY(launch_pack_filters_per_tap(a, filter_banks(c), ws, s), "filter packing launch");
  return LOCOCO_OK;
}

// Enqueue Eq. 5, Eq. 6 and Eq. 4 of one block: from a.cache_k / a.cache_v (a.m live slots) and the block
// into a.new_k / a.new_v.  `B`: the block length the workspace was laid out for (a.Bn may be a shorter
// last block).
lococo_status enqueue_compress(const lococo_config* c, Path path, StepArgs a, void* ws, int32_t B, hipStream_t s) {
  if (path == PATH_MFMA) {
    KTimer t(K_COMPRESS_MFMA, s);
    HIP_TRY(launch_compress_mfma(a, ws, filter_banks(c), cu_count(), (char*)ws + filter_ws_bytes(c), partials_of(c, ws, B),
                                 prelogits_of(c, ws, B), B, s),
            "compress launch");
    return LOCOCO_OK;
  }
  if (path == PATH_GENERIC && small_step_fits(a.M + B, a.M, a.d, a.k_width, a.conv_in)) {
    KTimer t(K_COMPRESS_SMALL, s);
    HIP_TRY(launch_compress_small(c->dtype, a, a.M + B, 1, B, a.Bn, a.new_k, a.new_v, 0, 0, 1, s), "compress launch");
    return LOCOCO_OK;
  }
  const bool unfused = path == PATH_MFMA_UNFUSED;
  float* logits = unfused ? (float*)((char*)ws + packed_ws_bytes(c) + stats_bytes(c, B)) : (float*)ws;
  if (unfused) a.ldw = (a.m + a.Bn + 3) / 4 * 4;      // whole groups of four for the MFMA form of Eq. 4
  if (unfused) {
    KTimer t(K_CONV_MFMA, s);
    HIP_TRY(launch_conv_logits_mfma(a, ws, logits, s), "conv launch");
  } else {
    KTimer t(K_CONV_GENERIC, s);
    HIP_TRY(launch_conv_logits_generic(c->dtype, a, logits, s), "conv launch");
  }
  if (a.protect) HIP_TRY(launch_protect_logits_generic(a, logits, s), "protect launch");
  if (unfused && mixnorm_mfma_fits(a, logits)) {       // Eq. 6 inside the mixing kernel: the logits are read once
    {
      KTimer t(K_MIX_MFMA, s);
      HIP_TRY(launch_mixnorm_mfma(a, logits, s), "mix launch");
    }
    if (a.protect) HIP_TRY(launch_protect_rows_generic(c->dtype, a, s), "protect launch");
    return LOCOCO_OK;
  }
  {
    KTimer t(K_NORM_GENERIC, s);
    HIP_TRY(launch_normalise_generic(a, logits, s), "normalise launch");
  }
  if (unfused && mix_mfma_fits(a, logits)) {
    KTimer t(K_MIX_MFMA, s);
    HIP_TRY(launch_mix_mfma(a, logits, s), "mix launch");
  } else {
    KTimer t(K_MIX_GENERIC, s);
    HIP_TRY(launch_mix_generic(c->dtype, a, logits, 0, s), "mix launch");
  }
  if (a.protect) HIP_TRY(launch_protect_rows_generic(c->dtype, a, s), "protect launch");
  return LOCOCO_OK;
}

// Enqueue fill or compress of one block and update the host-side state.
lococo_status enqueue_update(const lococo_config* c, Path path, StepArgs a, lococo_cache* ca,
                             void* ws, int32_t B, hipStream_t s) {
  if (a.m + a.Bn <= a.M) {
    a.new_k = ca->k[ca->cur];
    a.new_v = ca->v[ca->cur];
    KTimer t(K_FILL, s);
    HIP_TRY(launch_fill_generic(c->dtype, a, s), "fill launch");
    ca->len = a.m + a.Bn;
    return LOCOCO_OK;
  }
  a.new_k = ca->k[ca->cur ^ 1];
  a.new_v = ca->v[ca->cur ^ 1];
  lococo_status st = enqueue_compress(c, path, a, ws, B, s);
  if (st) return st;
  ca->cur ^= 1;
  ca->len = a.M;
  return LOCOCO_OK;
}

// `n_steps` compress steps in one launch, the slot tiles of a chain handing the new cache to each other through the ring
// of states at out_k / out_v (see ScanArgs); *taken = false, and nothing launched, while another persistent scan holds
// compute units.  `clear`: the counters have been used since they were zeroed (the status word is kept).
lococo_status enqueue_scan(const lococo_config* c, const StepArgs& a, int64_t n_steps, int32_t B, int64_t tokens_left, void* out_k,
                           void* out_v, int64_t out_stride, int64_t slot0, int64_t ring, void* ws, bool clear, hipStream_t s,
                           bool* taken, float* logits = nullptr, int64_t logits_stride = 0, int32_t logits_ld = 0, void* last_k = nullptr,
                           void* last_v = nullptr) {
  const bool capturing = stream_is_capturing(s);
  std::unique_lock<std::mutex> lk(g_scan_mu);
  *taken = capturing || !another_scan_in_flight(s);
  if (!*taken) return LOCOCO_OK;
  char* sync_ws = (char*)ws + filter_ws_bytes(c);
  if (clear)
    HIP_TRY(launch_scan_sync_clear(sync_ws, c->batch, c->n_kv_heads, c->M, true, s), "clearing the scan counters");
  ScanArgs sa;
  sa.st = a;
  sa.n_steps = (int32_t)n_steps;
  sa.B = B;
  sa.tokens_left = tokens_left;
  sa.out_k = out_k;
  sa.out_v = out_v;
  sa.out_stride = out_stride;
  sa.slot0 = (int32_t)slot0;
  sa.ring = (int32_t)ring;
  sa.sync = nullptr;
  sa.status = nullptr;
  sa.logits = logits;
  sa.logits_stride = logits_stride;
  sa.logits_ld = logits_ld;
  sa.last_k = n_steps > 1 ? last_k : nullptr;
  sa.last_v = n_steps > 1 ? last_v : nullptr;
  if (last_k && n_steps == 1) {
    sa.out_k = last_k;
    sa.out_v = last_v;
    sa.slot0 = 0;
  }
  sa.spin_limit = spin_limit();
  sa.same_l2_allowed = chain_sync_through_l2() ? 1 : 0;
  {
    KTimer t(K_COMPRESS_MFMA, s);
    HIP_TRY(launch_compress_scan(sa, ws, filter_banks(c), cu_count(), sync_ws, partials_of(c, ws, B), prelogits_of(c, ws, B), s),
            "compress scan launch");
  }
  if (!capturing) note_scan_launched(s);
  return LOCOCO_OK;
}

// Steps hi, hi - 1, .. hi - n + 1 of the backward walk through a window in one launch, on the counters the scan that recomputed its
// states has finished with (the status word is kept); *taken = false, and nothing launched, where its workgroups could not all be
// resident.  `cleared`: whether the counters are at zero.
lococo_status enqueue_bwd_walk(const lococo_config* c, const BwdConvArgs& g, int hi, int n, void* ws, hipStream_t s, bool* cleared,
                               bool* taken) {
  *taken = false;
  if (g_debug.scan_per_step == 1) return LOCOCO_OK;
  const bool capturing = stream_is_capturing(s);
  std::unique_lock<std::mutex> lk(g_scan_mu);
  if (!capturing && another_scan_in_flight(s)) return LOCOCO_OK;
  char* sync_ws = (char*)ws + filter_ws_bytes(c);
  if (!*cleared)
    HIP_TRY(launch_scan_sync_clear(sync_ws, c->batch, c->n_kv_heads, c->M, true, s), "clearing the scan counters");
  {
    KTimer t(K_BWD_WALK, s);
    const hipError_t e = launch_bwd_conv_walk(g, hi, n, sync_ws, spin_limit(), chain_sync_through_l2(), taken, s);
    if (e != hipSuccess || !*taken) t.drop();
    HIP_TRY(e, "backward walk launch");
  }
  *cleared = !*taken;
  if (*taken && !capturing) note_scan_launched(s);
  return LOCOCO_OK;
}

lococo_status segment_step_impl(const lococo_config* cfg, const lococo_qkvo* blk, int32_t B,
                                const void* conv_w, const void* conv_b, lococo_cache* cache,
                                void* workspace, size_t ws_bytes, void* stream) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if ((st = check_cache(cfg, cache))) return st;
  if ((st = check_step_shape(cfg, B, cache->len))) return st;
  if ((st = check_qkvo(cfg, blk, B, true))) return st;
  Path path;
  if ((st = resolve_path(cfg, B, &path))) return st;
  if ((st = check_mfma_strides(cfg, path, blk, B, true))) return st;
  const bool compress = cache->len + B > cfg->M;
  if (compress) {
    if (!conv_w) return fail(LOCOCO_EINVAL, "conv_w is NULL but this step compresses");
    const size_t need = step_ws_bytes(cfg, path, B);
    if (need && (!workspace || ws_bytes < need || ((uintptr_t)workspace & 255)))
      return fail(LOCOCO_EWORKSPACE, "workspace needs %zu bytes, 256-byte aligned (got %zu)", need,
                  workspace ? ws_bytes : (size_t)0);
  }
  StepArgs a = make_args(cfg, blk, 0, B, cache, conv_w, conv_b, true);
  lococo_cache tmp = *cache;
  if (compress && path != PATH_GENERIC &&
      (st = enqueue_repack(cfg, path, a, workspace, (hipStream_t)stream)))
    return st;
  if (compress && path == PATH_MFMA && compress_step_fits(a, cu_count())) {
    // both halves side by side in one launch, counted as the compression's
    a.new_k = tmp.k[tmp.cur ^ 1];
    a.new_v = tmp.v[tmp.cur ^ 1];
    const AttnArgs t = attn_args_one_block(a);
    {
      KTimer kt(K_COMPRESS_MFMA, (hipStream_t)stream);
      HIP_TRY(launch_compress_mfma(a, workspace, filter_banks(cfg), cu_count(), (char*)workspace + filter_ws_bytes(cfg),
                                   partials_of(cfg, workspace, B), prelogits_of(cfg, workspace, B), B, (hipStream_t)stream, &t),
              "step launch");
    }
    tmp.cur ^= 1;
    tmp.len = cfg->M;
    *cache = tmp;
    return LOCOCO_OK;
  }
  if ((st = enqueue_attn(cfg, path, a, step_stats(cfg, path, B, workspace, ws_bytes), (hipStream_t)stream)))
    return st;
  if ((st = enqueue_update(cfg, path, a, &tmp, workspace, B, (hipStream_t)stream))) return st;
  *cache = tmp;
  return LOCOCO_OK;
}

// ---- device address of the library's own scratch array on the current device, looked up once per
// device (every device the library runs on holds its own copy at its own address) and used from then
// on wherever host code needs the array's memory
constexpr size_t kScratchBytes = LOCOCO_NOALLOC_SCRATCH_BYTES;
void* g_scratch_ptr[kMaxDevices] = {nullptr};
std::mutex g_scratch_mu;

lococo_status scratch_on_this_device(void** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) return fail(LOCOCO_EUNSUPPORTED, "device index %d above %d", dev, kMaxDevices - 1);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "address of the library's scratch array");
    if (!p || ((uintptr_t)p & 255)) return fail(LOCOCO_EHIP, "the library's scratch array has no usable device address");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return LOCOCO_OK;
}

}  // namespace

extern "C" {

const char* lococo_last_error(void) { return g_err; }
const char* lococo_version(void) { return "0.3.0"; }

lococo_status lococo_debug_option(int32_t option, int64_t value) {
  switch (option) {
    case LOCOCO_OPT_RESET: g_debug = DebugOptions{0, 0, 0, 0, 0, 0, 0}; return LOCOCO_OK;
    case LOCOCO_OPT_SPIN_LIMIT: g_debug.spin_limit = value; return LOCOCO_OK;
    case LOCOCO_OPT_SCAN_PER_STEP: g_debug.scan_per_step = value == 2 ? 2 : value != 0; return LOCOCO_OK;
    case LOCOCO_OPT_CHAIN_SYNC_DEVICE: g_debug.chain_sync_device = value != 0; return LOCOCO_OK;
    case LOCOCO_OPT_LOGITS_TILES:
      if (value != 0 && value != 64 && value != 128 && value != 256)
        return fail(LOCOCO_EINVAL, "LOCOCO_OPT_LOGITS_TILES takes 0, 64, 128 or 256");
      g_debug.logits_tiles = value;
      return LOCOCO_OK;
    case LOCOCO_OPT_MAX_RESIDENT:
      if (value < 0) return fail(LOCOCO_EINVAL, "LOCOCO_OPT_MAX_RESIDENT takes a count >= 0");
      g_debug.max_resident = value;
      return LOCOCO_OK;
    case LOCOCO_OPT_UNFUSED_KV:
      if (value != 0 && value != 1) return fail(LOCOCO_EINVAL, "LOCOCO_OPT_UNFUSED_KV takes 0 or 1");
      g_debug.unfused_kv = value;
      return LOCOCO_OK;
    case LOCOCO_OPT_NO_STEP_PIPELINE:
      if (value != 0 && value != 1) return fail(LOCOCO_EINVAL, "LOCOCO_OPT_NO_STEP_PIPELINE takes 0 or 1");
      g_debug.no_step_pipeline = value;
      return LOCOCO_OK;
    default: return fail(LOCOCO_EINVAL, "unknown debug option %d", option);
  }
}

lococo_status lococo_describe_path(const lococo_config* cfg, int32_t B, lococo_path_info* out) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if (!out) return fail(LOCOCO_EINVAL, "out is NULL");
  if (B <= 0) return fail(LOCOCO_EINVAL, "block length B must be positive");
  Path path;
  if ((st = resolve_path(cfg, B, &path))) return st;
  std::memset(out, 0, sizeof(*out));
  out->path = (int32_t)path;
  out->compute_units = cu_count();
  if (path == PATH_MFMA) {
    out->tile_slots = compress_tile_slots(cfg->batch, cfg->n_kv_heads, cfg->M, cfg->conv_width, cfg->conv_in, cu_count());
    out->position_split = compress_position_split(cfg->batch, cfg->n_kv_heads, cfg->M, cfg->conv_width, cfg->conv_in, cu_count());
    out->step_pipeline = compress_step_pipeline(cfg->batch, cfg->n_kv_heads, cfg->M, cfg->conv_width, cfg->conv_in, cu_count());
    StepArgs a;
    std::memset(&a, 0, sizeof(a));
    a.batch = cfg->batch; a.Hkv = cfg->n_kv_heads; a.M = cfg->M; a.k_width = cfg->conv_width; a.norm = cfg->norm;
    a.conv_in = cfg->conv_in;
    a.w_head_stride = cfg->w_head_stride; a.b_head_stride = cfg->b_head_stride;
    out->scan_resident_limit = compress_scan_max_resident(a, cu_count());
    if (scan_fits_one_launch(cfg, a))
      out->scan_groups = compress_scan_groups(cfg->batch, cfg->n_kv_heads, cfg->M, cfg->conv_width, cfg->conv_in,
                                              cfg->w_head_stride != 0 || cfg->b_head_stride != 0, cu_count());
  }
  return LOCOCO_OK;
}

lococo_status lococo_scan_status(const lococo_config* cfg, const void* workspace, int32_t* out) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if (!workspace || !out) return fail(LOCOCO_EINVAL, "workspace or out is NULL");
  Path path;
  if ((st = resolve_path(cfg, 1, &path))) return st;
  if (path != PATH_MFMA) {
    *out = 0;
    return LOCOCO_OK;
  }
  const char* word = (const char*)workspace + filter_ws_bytes(cfg) +
                     (size_t)cfg->batch * cfg->n_kv_heads * sizeof(uint32_t);
  HIP_TRY(hipMemcpy(out, word, sizeof(int32_t), hipMemcpyDeviceToHost), "reading the scan status");
  return LOCOCO_OK;
}

lococo_status lococo_measure_peaks(void* scratch, size_t bytes, void* stream, double* mfma_tflops,
                                   double* copy_gbs) {
  if (!scratch || !mfma_tflops || !copy_gbs) return fail(LOCOCO_EINVAL, "null argument");
  if ((uintptr_t)scratch & 15) return fail(LOCOCO_EINVAL, "scratch must be 16-byte aligned");
  if (bytes < ((size_t)32 << 20)) return fail(LOCOCO_EINVAL, "scratch must hold at least 32 MiB (got %zu bytes)", bytes);
  HIP_TRY(measure_peaks(scratch, bytes, cu_count(), (hipStream_t)stream, mfma_tflops, copy_gbs),
          "peak measurement");
  return LOCOCO_OK;
}

lococo_status lococo_timing_begin(void) {
  std::lock_guard<std::mutex> lk(g_timing_mu);
  for (auto& t : g_timed) {
    (void)hipEventDestroy(t.start);
    (void)hipEventDestroy(t.stop);
  }
  g_timed.clear();
  g_timing_on = true;
  return LOCOCO_OK;
}

lococo_status lococo_timing_end(lococo_kernel_time* out, int32_t* n_inout) {
  if (!n_inout) return fail(LOCOCO_EINVAL, "n_inout is NULL");
  std::lock_guard<std::mutex> lk(g_timing_mu);
  g_timing_on = false;
  int64_t launches[K_COUNT] = {0};
  double ms[K_COUNT] = {0.0};
  lococo_status st = LOCOCO_OK;
  for (auto& t : g_timed) {
    float dt = 0.f;
    hipError_t e = hipEventSynchronize(t.stop);
    if (e == hipSuccess) e = hipEventElapsedTime(&dt, t.start, t.stop);
    if (e != hipSuccess && st == LOCOCO_OK) st = hip_fail(e, "timing events");
    launches[t.id] += 1;
    ms[t.id] += dt;
    (void)hipEventDestroy(t.start);
    (void)hipEventDestroy(t.stop);
  }
  g_timed.clear();
  const int32_t cap = out ? *n_inout : 0;
  int32_t n = 0;
  for (int id = 0; id < K_COUNT; ++id) {
    if (!launches[id]) continue;
    if (n < cap) out[n] = lococo_kernel_time{kKernelNames[id], launches[id], ms[id]};
    ++n;
  }
  *n_inout = n;
  return st;
}

lococo_status lococo_plan(int64_t L, int32_t B, int32_t M, int32_t len0, int32_t cur0,
                          lococo_seg* out, int64_t* n_inout) {
  if (!n_inout) return fail(LOCOCO_EINVAL, "n_inout is NULL");
  if (L < 0 || B <= 0 || M <= 0) return fail(LOCOCO_EINVAL, "need L >= 0, B > 0, M > 0");
  if (len0 < 0 || len0 > M) return fail(LOCOCO_ESTATE, "len0 %d is outside [0, M=%d]", len0, M);
  if (cur0 != 0 && cur0 != 1) return fail(LOCOCO_ESTATE, "cur0 must be 0 or 1");
  const int64_t cap = out ? *n_inout : 0;
  if (cap < 0) return fail(LOCOCO_EINVAL, "negative capacity");
  const int64_t n = (L + B - 1) / B;
  int32_t occ = len0, buf = cur0;
  for (int64_t i = 0; i < n; ++i) {
    const int64_t start = i * B;
    const int32_t len = (int32_t)std::min<int64_t>(B, L - start);
    const bool fits = (int64_t)occ + len <= M;
    const int32_t occ_after = fits ? occ + len : M;
    if (!fits) buf = 1 - buf;
    if (i < cap) out[i] = lococo_seg{start, len, fits ? 0 : 1, occ, occ_after, buf, 0};
    occ = occ_after;
  }
  *n_inout = n;
  return LOCOCO_OK;
}

lococo_status lococo_workspace_bytes(const lococo_config* cfg, int64_t L, int32_t B,
                                     int32_t history, size_t* out) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if (!out) return fail(LOCOCO_EINVAL, "out is NULL");
  if (L < 0 || B <= 0) return fail(LOCOCO_EINVAL, "need L >= 0 and B > 0");
  Path path;
  if ((st = resolve_path(cfg, B, &path))) return st;
  const int64_t n_blocks = (L + B - 1) / B;
  if (history < 0) return fail(LOCOCO_EINVAL, "history must be >= 0");
  if (history == 0 || !batched_attention(cfg, path, B) || n_blocks == 0)
    *out = step_ws_bytes(cfg, path, B);
  else if (history == 1 || history >= n_blocks)
    *out = history_ws_bytes(cfg, path, B, n_blocks, L);             // every block may compress
  else {
    const int64_t g = std::max<int64_t>(history, 2);
    *out = history_ws_bytes(cfg, path, B, g + 1, g * (int64_t)B);   // a window of g blocks: g + 1 states
  }
  return LOCOCO_OK;
}

lococo_status lococo_attn_only(const lococo_config* cfg, const lococo_qkvo* blk, int32_t B,
                               const lococo_cache* cache, void* stream) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if ((st = check_cache(cfg, cache))) return st;
  if ((st = check_step_shape(cfg, B, cache->len))) return st;
  if ((st = check_qkvo(cfg, blk, B, true))) return st;
  Path path;
  if ((st = resolve_path(cfg, B, &path))) return st;
  if ((st = check_mfma_strides(cfg, path, blk, B, true))) return st;
  StepArgs a = make_args(cfg, blk, 0, B, cache, nullptr, nullptr, true);
  return enqueue_attn(cfg, path, a, nullptr, (hipStream_t)stream);
}

lococo_status lococo_prepare_filters(const lococo_config* cfg, const void* conv_w, void* workspace,
                                     size_t ws_bytes, void* stream) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if (!conv_w) return fail(LOCOCO_EINVAL, "conv_w is NULL");
  Path path;
  if ((st = resolve_path(cfg, 1, &path))) return st;
  if (path == PATH_GENERIC) return LOCOCO_OK;    // the shape-agnostic kernels read [M, C, k] as given
  const size_t need = path == PATH_MFMA ? filter_ws_bytes(cfg) : packed_ws_bytes(cfg);
  if (!workspace || ws_bytes < need || ((uintptr_t)workspace & 255))
    return fail(LOCOCO_EWORKSPACE, "workspace needs %zu bytes, 256-byte aligned (got %zu)", need,
                workspace ? ws_bytes : (size_t)0);
  StepArgs a{};
  a.conv_w = conv_w;
  a.w_head_stride = cfg->w_head_stride;
  a.M = cfg->M;
  a.k_width = cfg->conv_width;
  a.conv_in = cfg->conv_in;
  lococo_config once = *cfg;
  once.flags &= ~LOCOCO_FLAG_FILTERS_PREPARED;
  return enqueue_repack(&once, path, a, workspace, (hipStream_t)stream);
}

lococo_status lococo_segment_step(const lococo_config* cfg, const lococo_qkvo* blk, int32_t B,
                                  const void* conv_w, const void* conv_b, lococo_cache* cache,
                                  void* workspace, size_t ws_bytes, void* stream) {
  return segment_step_impl(cfg, blk, B, conv_w, conv_b, cache, workspace, ws_bytes, stream);
}

lococo_status lococo_segment_step_noalloc(const lococo_config* cfg, const lococo_qkvo* blk, int32_t B,
                                          const void* conv_w, const void* conv_b, lococo_cache* cache,
                                          void* stream) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if (cfg->flags & LOCOCO_FLAG_FILTERS_PREPARED)
    return fail(LOCOCO_EINVAL, "LOCOCO_FLAG_FILTERS_PREPARED cannot be used with the library's own scratch "
                "array: every caller on the device shares it, so nothing prepared can be assumed to be there");
  if (B <= 0) return fail(LOCOCO_EINVAL, "block length B must be positive");
  Path path;
  if ((st = resolve_path(cfg, B, &path))) return st;
  const size_t need = step_ws_bytes(cfg, path, B);
  if (need > kScratchBytes)
    return fail(LOCOCO_EWORKSPACE, "this step needs %zu bytes of scratch, the library's own array holds %zu: "
                "use lococo_segment_step with a workspace of the caller's", need, kScratchBytes);
  void* ws = nullptr;
  if ((st = scratch_on_this_device(&ws))) return st;
  return segment_step_impl(cfg, blk, B, conv_w, conv_b, cache, ws, kScratchBytes, stream);
}

lococo_status lococo_sequence_forward(const lococo_config* cfg, const lococo_qkvo* seq, int64_t L,
                                      int32_t B, const void* conv_w, const void* conv_b,
                                      lococo_cache* cache, void* workspace, size_t ws_bytes,
                                      void* stream) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if ((st = check_cache(cfg, cache))) return st;
  if (L < 0) return fail(LOCOCO_EINVAL, "L must be >= 0");
  if (B <= 0) return fail(LOCOCO_EINVAL, "block length B must be positive");
  if (L == 0) return LOCOCO_OK;  // nothing to do; tensors may be empty
  if ((st = check_step_shape(cfg, B, std::min<int64_t>(cfg->M, (int64_t)cache->len + L))))
    return st;
  if ((st = check_qkvo(cfg, seq, L, true))) return st;
  Path path;
  if ((st = resolve_path(cfg, B, &path))) return st;
  int64_t n = 0;
  if ((st = lococo_plan(L, B, cfg->M, cache->len, cache->cur, nullptr, &n))) return st;
  std::vector<lococo_seg> plan((size_t)n);
  if (n && (st = lococo_plan(L, B, cfg->M, cache->len, cache->cur, plan.data(), &n))) return st;
  bool any_compress = false;
  for (const auto& sg : plan) any_compress |= sg.branch == 1;
  if (any_compress) {
    if (!conv_w) return fail(LOCOCO_EINVAL, "conv_w is NULL but the scan compresses");
    const size_t need = step_ws_bytes(cfg, path, B);
    if (need && (!workspace || ws_bytes < need || ((uintptr_t)workspace & 255)))
      return fail(LOCOCO_EWORKSPACE, "workspace needs %zu bytes, 256-byte aligned (got %zu)", need,
                  workspace ? ws_bytes : (size_t)0);
  }
  int64_t n_compress = 0;
  for (const auto& sg : plan) n_compress += sg.branch;
  // Batched-attention schedules: run the fill / compress recurrence of a window of blocks first,
  // keeping the cache state after each of them in a ring of history slots, then one attention
  // launch over the window's blocks.  The window is the whole sequence when the workspace holds
  // every state, otherwise as many blocks as it holds (at least two: a ring of G + 1 slots serves a
  // window of G blocks, the extra one being the state the window starts from); memory then stays
  // independent of the sequence length, as in the step-by-step schedule.
  int64_t window = 0, ring = 0;
  if (batched_attention(cfg, path, B) && any_compress && workspace) {
    if (ws_bytes >= history_ws_bytes(cfg, path, B, n_compress, L)) {
      window = n;
      ring = n_compress;
    } else {
      for (int64_t g = std::min<int64_t>(n, 4096); g >= 2; --g)
        if (ws_bytes >= history_ws_bytes(cfg, path, B, g + 1, g * (int64_t)B)) { window = g; ring = g + 1; break; }
    }
  }
  lococo_cache tmp = *cache;
  // the scan status of this call starts at "no wait gave up", whichever schedule runs
  const bool clear = path == PATH_MFMA && workspace && ws_bytes >= step_ws_bytes(cfg, path, B);
  const bool repack = any_compress && path != PATH_GENERIC && !(cfg->flags & LOCOCO_FLAG_FILTERS_PREPARED);
  // the blocks from lo to before hi, all fills, as one
  auto fill_args = [&](int64_t lo, int64_t hi) {
    const lococo_seg& sg = plan[(size_t)lo];
    const int64_t tokens = plan[(size_t)(hi - 1)].start + plan[(size_t)(hi - 1)].len - sg.start;
    StepArgs a = make_args(cfg, seq, sg.start, (int32_t)tokens, &tmp, conv_w, conv_b, true);
    a.m = sg.len_before;
    a.new_k = tmp.k[tmp.cur];
    a.new_v = tmp.v[tmp.cur];
    return a;
  };
  int64_t filled = 0;                         // leading fill blocks that are behind us
  if (repack) {
    StepArgs a0 = make_args(cfg, seq, 0, B, &tmp, conv_w, conv_b, true), f;
    if (path == PATH_MFMA)
      while (filled < std::min(n, window) && plan[(size_t)filled].branch == 0) ++filled;
    if (filled) f = fill_args(0, filled);
    if ((st = enqueue_repack(cfg, path, a0, workspace, (hipStream_t)stream,
                             clear ? (char*)workspace + filter_ws_bytes(cfg) : nullptr, filled ? &f : nullptr)))
      return st;
  }
  if (clear && !repack) {
    HIP_TRY(launch_scan_sync_clear((char*)workspace + filter_ws_bytes(cfg), cfg->batch, cfg->n_kv_heads, cfg->M, false,
                                   (hipStream_t)stream), "clearing the scan counters");
  }
  if (window > 0) {
    hipStream_t s = (hipStream_t)stream;
    const size_t slot = align_up(state_bytes(cfg), 256);
    const int64_t window_rows = std::min<int64_t>(L, window * (int64_t)B);
    float* win_stats = (float*)((char*)workspace + step_ws_bytes(cfg, path, B));
    char* hist_k = (char*)win_stats + stats_bytes(cfg, window_rows);
    char* hist_v = hist_k + (size_t)ring * slot;
    const int64_t hist_stride = (int64_t)(slot / esize(cfg->dtype));
    auto slot_k = [&](int64_t c) { return hist_k + (size_t)(c % ring) * slot; };
    auto slot_v = [&](int64_t c) { return hist_v + (size_t)(c % ring) * slot; };
    bool one_launch = false;
    if (path == PATH_MFMA) {
      StepArgs probe = make_args(cfg, seq, 0, B, &tmp, conv_w, conv_b, true);
      one_launch = scan_fits_one_launch(cfg, probe);
    }
    const bool small_scan = path == PATH_GENERIC &&
                            small_scan_one_launch(cfg->dtype, cfg->M + B, cfg->M, cfg->head_dim, cfg->conv_width, cfg->conv_in);
    int64_t c_done = 0;                       // compress steps enqueued so far: state c_done - 1 is the newest
    const bool direct = n_compress > 0 && plan.back().buf_after != tmp.cur &&
                        (path != PATH_MFMA || n_compress == 1 ||
                         compress_scan_last_to_caller(make_args(cfg, seq, 0, B, &tmp, conv_w, conv_b, true), B, n_compress, cu_count()));
    for (int64_t w0 = 0; w0 < n; w0 += window) {
      const int64_t w1 = std::min<int64_t>(n, w0 + window);
      // the state the window starts from: the caller's live buffer until the first compression
      const int64_t c0 = c_done;
      const void* base_k = c0 == 0 ? tmp.k[tmp.cur] : slot_k(c0 - 1);
      const void* base_v = c0 == 0 ? tmp.v[tmp.cur] : slot_v(c0 - 1);
      int64_t fills = 0;                      // fill blocks at the head of the window
      while (w0 + fills < w1 && plan[(size_t)(w0 + fills)].branch == 0) ++fills;
      for (int64_t bi = w0; bi < w1; ++bi) {
        const lococo_seg& sg = plan[(size_t)bi];
        StepArgs a = make_args(cfg, seq, sg.start, sg.len, &tmp, conv_w, conv_b, true);
        a.m = sg.len_before;
        if (sg.branch == 0) {                 // the fill blocks at the head of the window in one launch
          bi = w0 + fills - 1;
          if (bi < filled) continue;
          KTimer t(K_FILL, s);
          HIP_TRY(launch_fill_generic(cfg->dtype, fill_args(w0, w0 + fills), s), "fill launch");
          continue;
        }
        // The last state of all is nobody's but the caller's, and goes there at once where the attention that follows does not
        // read the buffer (where that is not the one the call found the cache in) and the scan's kernel can tell its last step.
        void* const last_k = direct ? tmp.k[plan.back().buf_after] : nullptr;
        void* const last_v = direct ? tmp.v[plan.back().buf_after] : nullptr;
        a.cache_k = c_done == 0 ? tmp.k[tmp.cur] : slot_k(c_done - 1);
        a.cache_v = c_done == 0 ? tmp.v[tmp.cur] : slot_v(c_done - 1);
        if (one_launch) {
          // every later block of the window compresses too (the cache stays full): one launch runs
          // them all, the slot tiles of a chain handing the new cache to each other through the ring
          // (the counters start every launch at zero)
          if ((st = enqueue_scan(cfg, a, w1 - bi, B, L - sg.start, hist_k, hist_v, hist_stride, c_done % ring, ring, workspace,
                                 c_done > 0, s, &one_launch, nullptr, 0, 0, w1 == n ? last_k : nullptr, w1 == n ? last_v : nullptr)))
            return st;
          if (one_launch) {
            c_done += w1 - bi;
            break;
          }                              // another persistent scan holds compute units: one launch per step
        }
        if (small_scan) {                // one workgroup per chain walks the rest of the window
          KTimer t(K_COMPRESS_SMALL, s);
          HIP_TRY(launch_compress_small(cfg->dtype, a, cfg->M + B, (int)(w1 - bi), B, L - sg.start, hist_k, hist_v, hist_stride,
                                        (int)(c_done % ring), (int)ring, s, w1 == n ? last_k : nullptr, w1 == n ? last_v : nullptr),
                  "compress scan launch");
          c_done += w1 - bi;
          break;
        }
        const bool to_caller = direct && c_done + 1 == n_compress;
        a.new_k = to_caller ? last_k : slot_k(c_done);
        a.new_v = to_caller ? last_v : slot_v(c_done);
        if ((st = enqueue_compress(cfg, path, a, workspace, B, s))) return st;
        ++c_done;
      }
      // A block of one token (every block when B = 1, else a ragged last block) goes to the kernel of the
      // generation stage here as in the step-by-step schedule: which kernel a block's attention runs on depends on
      // the block, never on the schedule, so the bits do not either.  Such blocks can only end a window, and they
      // come after the window's other blocks, as they do in time (the order matters to sums kept per slot).
      int64_t w_batched = w1;
      while (w_batched > w0 && path != PATH_GENERIC &&
             attn_decode_supports(cfg->dtype, cfg->head_dim, plan[(size_t)(w_batched - 1)].len, cfg->M,
                                  cache->attn_colsum != nullptr))
        --w_batched;
      if (w_batched > w0) {
        const lococo_seg& first = plan[(size_t)w0];
        StepArgs a0 = make_args(cfg, seq, first.start, B, &tmp, conv_w, conv_b, true);
        AttnArgs t = attn_args_one_block(a0);
        t.cache_k = base_k;
        t.cache_v = base_v;
        t.hist_k = hist_k;
        t.hist_v = hist_v;
        t.hist_stride = hist_stride;
        t.hist_first = (int32_t)(c0 % ring);
        t.hist_ring = (int32_t)ring;
        t.L = std::min<int64_t>(L - first.start, (w_batched - w0) * (int64_t)B);
        t.B = B;
        t.len0 = first.len_before;
        t.n_fill = (int32_t)std::min<int64_t>(fills, w_batched - w0);
        t.n_seg = (int32_t)(w_batched - w0);
        t.stats = cache->attn_colsum ? win_stats : nullptr;
        if (path == PATH_GENERIC) {
          KTimer kt(K_ATTN_GENERIC, s);
          HIP_TRY(launch_attn_rows(cfg->dtype, t, cfg->head_dim, cache->attn_colsum, s), "attention launch");
        } else {
          KTimer kt(K_ATTN_MFMA, s);
          HIP_TRY(launch_attn_mfma(t, s), "attention launch");
        }
        if (cache->attn_colsum && path != PATH_GENERIC) {   // sums over blocks commute: one launch for all of the window's
          KTimer kt(K_ATTN_COLSUM, s);
          HIP_TRY(launch_attn_colsum_mfma(t, cache->attn_colsum, s), "attention column-sum launch");
        }
      }
      if (w_batched < w1) {
        int64_t c_before = c0;                  // compress steps ahead of block bi
        for (int64_t bi = w0; bi < w1; ++bi) {
          const lococo_seg& sg = plan[(size_t)bi];
          if (bi >= w_batched) {
            StepArgs a = make_args(cfg, seq, sg.start, sg.len, &tmp, conv_w, conv_b, true);
            a.m = sg.len_before;
            a.cache_k = c_before == 0 ? tmp.k[tmp.cur] : slot_k(c_before - 1);
            a.cache_v = c_before == 0 ? tmp.v[tmp.cur] : slot_v(c_before - 1);
            KTimer kt(K_ATTN_DECODE, s);
            HIP_TRY(launch_attn_decode(a, s), "attention launch");
          }
          if (sg.branch != 0) ++c_before;
        }
      }
    }
    const lococo_seg& last = plan.back();
    if (c_done > 0 && !direct) {
      HIP_TRY(launch_copy_pair(tmp.k[last.buf_after], slot_k(c_done - 1), tmp.v[last.buf_after], slot_v(c_done - 1),
                               state_bytes(cfg), s),
              "publishing the final cache");
    }
    tmp.cur = last.buf_after;
    tmp.len = last.len_after;
    *cache = tmp;
    return LOCOCO_OK;
  }
  for (const auto& sg : plan) {
    StepArgs a = make_args(cfg, seq, sg.start, sg.len, &tmp, conv_w, conv_b, true);
    if ((st = enqueue_attn(cfg, path, a, step_stats(cfg, path, B, workspace, ws_bytes), (hipStream_t)stream)))
      return st;
    if ((st = enqueue_update(cfg, path, a, &tmp, workspace, B, (hipStream_t)stream))) return st;
  }
  *cache = tmp;
  return LOCOCO_OK;
}

namespace {
// Eq. 4 - 6 of the backward pass run on MFMA (bwd_conv_mfma.hip) unless the shape-agnostic kernels are asked for
bool bwd_on_mfma(const lococo_config* c) {
  return c->impl != LOCOCO_IMPL_GENERIC && bwd_mfma_supports(c->dtype, c->head_dim, c->conv_in, c->conv_width);
}
bool bwd_attn_has_mfma(const lococo_config* c) {
  const char* why;
  return c->impl != LOCOCO_IMPL_GENERIC && attn_mfma_supports(c->dtype, c->head_dim, &why);
}
// the attention of the backward pass runs on its own MFMA kernels (bwd_attn_mfma.hip) where a block's rows can be
// addressed with 32-bit offsets
bool bwd_attn_on_mfma(const lococo_config* c, const lococo_qkvo* x, int32_t B) {
  if (!bwd_attn_has_mfma(c)) return false;
  const int64_t lim = 0x7fff0000;
  for (const lococo_tensor* t : {&x->q, &x->k, &x->v})
    if (((int64_t)B * t->stride_t + c->head_dim) * 2 >= lim) return false;
  return (int64_t)c->M * c->head_dim * 2 < lim && (int64_t)B * c->head_dim * 4 < lim;
}
// scratch of those kernels for `rows` query rows per head: dO as up to three bf16 parts, three floats of row statistics
size_t bwd_attn_hl_bytes(const lococo_config* c, int64_t rows) {
  return align_up((size_t)c->batch * c->n_q_heads * (size_t)rows * c->head_dim * 6, 256);
}
size_t bwd_attn_stat_bytes(const lococo_config* c, int64_t rows) {
  return align_up((size_t)c->batch * c->n_q_heads * (size_t)rows * 3 * sizeof(float), 256);
}
struct BwdLayout { size_t p, ds, w, n, dw, conv, total; bool one_filters; };
BwdConvLayout conv_layout(const lococo_config* c, int32_t T, int64_t n_blk, bool one_filters, bool with_logits = true) {
  return bwd_conv_layout(c->batch, c->n_kv_heads, c->M, T, c->conv_width, c->conv_in, filter_banks(c), n_blk, with_logits, one_filters);
}
// one_filters: the least memory a step can do with.  The filters are packed in two orders, for Eq. 5 and for its input gradient;
// with one place for both a step packs them in a launch more.
BwdLayout bwd_layout(const lococo_config* c, int32_t B, int32_t len, bool one_filters) {
  const size_t T = (size_t)len + B;
  const size_t rows = (size_t)c->batch * c->n_q_heads * B * T * sizeof(float);
  const bool compress = len + B > c->M, conv = compress && bwd_on_mfma(c);
  const size_t mat = compress && !conv ? align_up((size_t)c->batch * c->n_kv_heads * c->M * T * sizeof(float), 256) : 0;
  BwdLayout l;
  l.p = 0;                                     // attention rows, or dO as two halves; then their gradient, or the statistics
  l.ds = std::max(align_up(rows, 256), bwd_attn_hl_bytes(c, B));
  l.w = l.ds + std::max(align_up(rows, 256), bwd_attn_stat_bytes(c, B));
  l.n = l.w + mat;
  l.dw = l.n + mat;
  l.conv = 0;                                  // Eq. 4 - 6 on MFMA come when the attention is done with its arrays
  l.total = std::max(l.dw + mat, conv ? conv_layout(c, (int32_t)T, 1, one_filters).total : (size_t)0);
  l.one_filters = one_filters;
  return l;
}
// The attention of the blocks of `t` (see BwdAttnArgs; the gradient arrays hold `rows` query / block rows per head from
// the first token of the window on)
lococo_status enqueue_bwd_attn(const lococo_config* c, BwdAttnArgs t, int64_t rows, char* hl, char* stats, hipStream_t s) {
  t.q_sh = t.k_sh = rows * c->head_dim;
  t.q_sb = t.q_sh * c->n_q_heads;
  t.k_sb = t.k_sh * c->n_kv_heads;
  t.do_hl = (uint16_t*)hl;
  t.stats = (float*)stats;
  HIP_TRY(launch_bwd_attn_mfma(t, s), "attention backward launches");
  return LOCOCO_OK;
}

// Everything of a step's backward pass but (where g.attn_done) its attention.  `g`: all but the workspace filled in.
lococo_status enqueue_step_backward(const lococo_config* cfg, BwdArgs g, bool compress, const BwdLayout& l, char* ws, hipStream_t s) {
  g.ws_p = (float*)(ws + l.p);
  g.ws_ds = (float*)(ws + l.ds);
  g.ws_w = (float*)(ws + l.w);
  g.ws_n = (float*)(ws + l.n);
  g.ws_dw = (float*)(ws + l.dw);
  g.conv_elsewhere = compress && bwd_on_mfma(cfg) ? 1 : 0;
  g.gemms_mfma = cfg->impl != LOCOCO_IMPL_GENERIC && cfg->dtype == LOCOCO_BF16 ? 1 : 0;
  if (compress && !g.conv_elsewhere) {
    // recompute Eq. 5 and Eq. 6 of the forward step: raw logits and normalised rows
    HIP_TRY(launch_conv_logits_generic(cfg->dtype, g.st, g.ws_w, s), "conv launch");
    if (g.st.protect) HIP_TRY(launch_protect_logits_generic(g.st, g.ws_w, s), "protect launch");
    const size_t mat = (size_t)cfg->batch * cfg->n_kv_heads * cfg->M * ((size_t)g.st.m + g.st.Bn) * sizeof(float);
    HIP_TRY(hipMemcpyAsync(g.ws_n, g.ws_w, mat, hipMemcpyDeviceToDevice, s), "copying the logits");
    HIP_TRY(launch_normalise_generic(g.st, g.ws_n, s), "normalise launch");
  }
  HIP_TRY(launch_step_backward_generic(cfg->dtype, g, compress, s), "backward launches");
  if (!g.conv_elsewhere) return LOCOCO_OK;
  const int32_t T = g.st.m + g.st.Bn;
  BwdConvArgs c{};
  c.st = g.st;
  c.n_blk = 1;
  c.B = g.st.Bn;
  c.banks = filter_banks(cfg);
  c.three_parts = g.three_parts;
  c.tokens = g.st.Bn;
  c.d_cache_k = g.d_cache_k;
  c.d_cache_v = g.d_cache_v;
  c.d_new_k = g.d_new_k;
  c.d_new_v = g.d_new_v;
  c.d_k = g.d_k;
  c.d_v = g.d_v;
  c.kv_chain = g.kv_chain;
  c.d_conv_w = g.d_conv_w;
  c.d_conv_b = g.d_conv_b;
  bwd_conv_place(&c, conv_layout(cfg, T, 1, l.one_filters), ws + l.conv);
  HIP_TRY(launch_bwd_conv_begin(c, true, nullptr, s), "filter packing launches");
  HIP_TRY(launch_bwd_conv_logits(c, s), "conv launch");
  HIP_TRY(launch_bwd_conv_rows(c, 0, T, s), "row gradient launch");
  HIP_TRY(launch_bwd_conv_dx(c, 0, 1, 2, T, s), "input gradient launch");
  HIP_TRY(launch_bwd_conv_dw(c, s), "filter gradient launch");
  HIP_TRY(launch_bwd_conv_end(c, s), "filter gradient launch");
  return LOCOCO_OK;
}
}  // namespace

lococo_status lococo_backward_workspace_bytes(const lococo_config* cfg, int32_t B, int32_t len, size_t* out) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if (!out) return fail(LOCOCO_EINVAL, "out is NULL");
  if (B <= 0 || len < 0 || len > cfg->M) return fail(LOCOCO_EINVAL, "B must be positive and len in [0, M]");
  *out = bwd_layout(cfg, B, len, false).total;
  return LOCOCO_OK;
}

lococo_status lococo_segment_step_backward(const lococo_config* cfg, const lococo_qkvo* blk, int32_t B,
                                           const void* conv_w, const void* conv_b,
                                           const lococo_cache* cache_before, const float* d_o,
                                           const float* d_new_k, const float* d_new_v, float* d_q,
                                           float* d_k, float* d_v, float* d_cache_k, float* d_cache_v,
                                           float* d_conv_w, float* d_conv_b, void* workspace,
                                           size_t ws_bytes, void* stream) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if ((st = check_cache(cfg, cache_before))) return st;
  if ((st = check_step_shape(cfg, B, cache_before->len))) return st;
  if (!blk) return fail(LOCOCO_EINVAL, "qkvo is NULL");
  if ((st = check_tensor(cfg, blk->q, "q", B)) || (st = check_tensor(cfg, blk->k, "k", B)) ||
      (st = check_tensor(cfg, blk->v, "v", B)))
    return st;
  if (!d_o || !d_new_k || !d_new_v || !d_q || !d_k || !d_v || !d_cache_k || !d_cache_v)
    return fail(LOCOCO_EINVAL, "a gradient pointer is NULL");
  if (cfg->norm == 2) return fail(LOCOCO_EUNSUPPORTED, "norm = 2 (rectifier on the convolution input) is forward only");
  const bool compress = cache_before->len + B > cfg->M;
  if (compress && (!conv_w || !d_conv_w))
    return fail(LOCOCO_EINVAL, "conv_w or d_conv_w is NULL but the step compresses");
  BwdLayout l = bwd_layout(cfg, B, cache_before->len, false);
  if (ws_bytes < l.total) l = bwd_layout(cfg, B, cache_before->len, true);
  if (!workspace || ws_bytes < l.total || ((uintptr_t)workspace & 255))
    return fail(LOCOCO_EWORKSPACE, "workspace needs %zu bytes, 256-byte aligned (got %zu)", l.total,
                workspace ? ws_bytes : (size_t)0);
  hipStream_t s = (hipStream_t)stream;
  lococo_qkvo x = *blk;
  x.o = x.q;                                  // not read; keeps make_args' view arithmetic defined
  BwdArgs g{};
  g.st = make_args(cfg, &x, 0, B, cache_before, conv_w, conv_b, true);
  g.d_o = d_o;
  g.d_new_k = d_new_k;
  g.d_new_v = d_new_v;
  g.d_q = d_q;
  g.d_k = d_k;
  g.d_v = d_v;
  g.d_cache_k = d_cache_k;
  g.d_cache_v = d_cache_v;
  g.d_conv_w = d_conv_w;
  g.d_conv_b = d_conv_b;
  g.o_chain = g.q_chain = g.kv_chain = (int64_t)B * cfg->head_dim;
  // (with such arrays the plain contractions of a step do not take two halves: see bwd_gemms_mfma_fit)
  g.three_parts = (((uintptr_t)d_o | (uintptr_t)d_new_k | (uintptr_t)d_new_v) & 15) != 0;
  if (bwd_attn_on_mfma(cfg, blk, B)) {
    BwdAttnArgs t{};
    t.a = attn_args_one_block(g.st);
    t.d_o = d_o;
    t.d_q = d_q;
    t.d_k = d_k;
    t.d_v = d_v;
    t.d_ck = d_cache_k;
    t.d_cv = d_cache_v;
    t.three_parts = g.three_parts;
    if ((st = enqueue_bwd_attn(cfg, t, B, (char*)workspace + l.p, (char*)workspace + l.ds, s))) return st;
    g.attn_done = 1;
  }
  return enqueue_step_backward(cfg, g, compress, l, (char*)workspace, s);
}

lococo_status lococo_mix_from_logits(const lococo_config* cfg, const lococo_qkvo* blk, int32_t B,
                                     const float* logits, lococo_cache* cache, void* stream) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if ((st = check_cache(cfg, cache))) return st;
  if ((st = check_step_shape(cfg, B, cache->len))) return st;
  if ((st = check_qkvo(cfg, blk, B, false))) return st;
  if (!logits) return fail(LOCOCO_EINVAL, "logits is NULL");
  if (cache->protect)
    return fail(LOCOCO_EUNSUPPORTED, "lococo_mix_from_logits does not take protected slots");
  Path path;
  if ((st = resolve_path(cfg, B, &path))) return st;
  if ((st = check_mfma_strides(cfg, path, blk, B, false))) return st;
  StepArgs a = make_args(cfg, blk, 0, B, cache, nullptr, nullptr, false);
  a.new_k = cache->k[cache->cur ^ 1];
  a.new_v = cache->v[cache->cur ^ 1];
  // bf16 / head_dim 128 unless the shape-agnostic kernels are asked for: Eq. 6 and Eq. 4 on the matrix
  // cores (the kernel of the unfused MFMA path), which needs rows of logits that start 16-byte aligned
  if (path != PATH_GENERIC && mixnorm_mfma_fits(a, logits)) {
    KTimer t(K_MIX_MFMA, (hipStream_t)stream);
    HIP_TRY(launch_mixnorm_mfma(a, logits, (hipStream_t)stream), "mix launch");
  } else {
    KTimer t(K_MIX_GENERIC, (hipStream_t)stream);
    HIP_TRY(launch_mix_generic(cfg->dtype, a, logits, 1, (hipStream_t)stream), "mix launch");
  }
  cache->cur ^= 1;
  cache->len = cfg->M;
  return LOCOCO_OK;
}

}  // extern "C"

// ---- backward of a whole scan: the forward recurrence is run once more to keep the state every block
// started from, then the blocks are walked in reverse
namespace {
struct SeqBwdLayout {
  size_t fwd_ws, fwd_ws_bytes;        // step workspace of the recomputed forward (first: see lococo_scan_status)
  size_t states_k, states_v, state;   // the state BEFORE every block: n_blocks slots of `state` bytes each
  int64_t window;         // blocks whose attention, logits and filter gradient run in one launch (see lococo_sequence_backward)
  size_t d_ck, d_cv, slot;            // gradients w.r.t. the state before each of them, fp32, `slot` bytes each
  size_t hl, stats;       // scratch of the attention launches
  BwdConvLayout conv;     // of Eq. 4 - 6 (inside step_ws)
  bool one_filters;       // see bwd_layout
  bool keep_logits;       // the logits of all blocks have a place, `logits`: the recomputed scan leaves them there
  size_t logits;
  size_t d_o;             // a block's upstream gradient where the walk needs a copy of it (no windows)
  size_t g[2][2];         // gradient w.r.t. the cache state, ping-pong: [which][k, v], fp32 [chains, M, d]
  size_t step_ws;         // the window's Eq. 4 - 6, or the workspace of one backward step where there are no windows
  size_t total;
};
// What a window may take: enough blocks to fill the device many times over at any shape, whatever the length of the
// sequence.
constexpr size_t kBwdWindowBytes = (size_t)3 << 30;
// The logits of Eq. 5 of every block may take this much (64 blocks of 32 chains, 512 slots and 1024 positions: 4.3 GB of the
// 7.4 GiB a call on that sequence asks for, 3.2 without); what is longer computes them window by window.  Keeping them takes Eq. 5
// out of the pass once, 34.2 -> 30.8 ms on that sequence, 16 K tokens of twice the chains 33.0 -> 29.9, 3.5 K tokens on 128 slots
// 1.78 -> 1.67.  The limit bounds what a call asks for, it is not where keeping stops to pay; it is all blocks or none, and 64
// blocks of 64 such chains miss it by 0.1 %.
constexpr size_t kBwdLogitsBytes = (size_t)8 << 30;

// largest_window: blocks a window may have at most; keep: whether the logits of all blocks may have a place; one_filters: see
// bwd_layout
lococo_status seq_bwd_layout(const lococo_config* c, int64_t L, int32_t B, int64_t largest_window, bool keep, bool one_filters,
                             SeqBwdLayout* out) {
  SeqBwdLayout l{};
  l.one_filters = one_filters;
  size_t at = 0;
  auto take = [&](size_t bytes) { const size_t here = at; at += align_up(bytes, 256); return here; };
  const size_t chains = (size_t)c->batch * c->n_kv_heads, es = esize(c->dtype);
  l.state = align_up(chains * c->M * c->head_dim * es, 256);
  const int64_t n = (L + B - 1) / B;
  Path path;
  lococo_status st = resolve_path(c, B, &path);
  if (st) return st;
  l.fwd_ws_bytes = step_ws_bytes(c, path, B);
  l.fwd_ws = take(l.fwd_ws_bytes);
  if (path == PATH_MFMA && bwd_on_mfma(c) && bwd_attn_has_mfma(c) && n > 1) {
    const int split = compress_position_split(c->batch, c->n_kv_heads, c->M, c->conv_width, c->conv_in, cu_count());
    l.keep_logits = keep && compress_scan_leaves_logits(false, c->conv_in, split > 1) &&
                    conv_layout(c, c->M + B, 1, one_filters).logits_stride * 4 <= kBwdLogitsBytes / (size_t)n;
  }
  const size_t n_states = (size_t)n + (l.keep_logits ? 1 : 0);   // (then the last block's own update is made as well)
  l.states_k = take(n_states * l.state);
  l.states_v = take(n_states * l.state);
  l.slot = align_up(chains * c->M * c->head_dim * sizeof(float), 256);
  size_t step = bwd_layout(c, B, c->M, one_filters).total;   // (grows with the occupancy: the full cache bounds all)
  if (bwd_attn_has_mfma(c)) {
    size_t per_block = 2 * l.slot + bwd_attn_hl_bytes(c, B) + bwd_attn_stat_bytes(c, B);
    if (bwd_on_mfma(c)) {
      const BwdConvLayout one = conv_layout(c, c->M + B, 1, one_filters, !l.keep_logits);
      per_block += one.total - one.per_call;
    }
    // (blocks x chains and 4 x blocks are grid dimensions)
    const int64_t most = std::min<int64_t>((int64_t)(kBwdWindowBytes / per_block), (int64_t)(8192 / chains));
    l.window = std::max<int64_t>(1, std::min<int64_t>({n, most, largest_window}));
    l.d_ck = take((size_t)l.window * l.slot);
    l.d_cv = take((size_t)l.window * l.slot);
    l.hl = take(bwd_attn_hl_bytes(c, l.window * (int64_t)B));
    l.stats = take(bwd_attn_stat_bytes(c, l.window * (int64_t)B));
    if (bwd_on_mfma(c)) {
      l.conv = conv_layout(c, c->M + B, l.window, one_filters, !l.keep_logits);
      if (l.keep_logits) l.logits = take((size_t)n * l.conv.logits_stride * 4);
      step = std::max(step, l.conv.total);
    }
  }
  // (where the windows are not run after all, their scratch is idle)
  l.d_o = l.window ? l.hl : take((size_t)c->batch * c->n_q_heads * B * c->head_dim * sizeof(float));
  for (int w = 0; w < 2; ++w)
    for (int kv = 0; kv < 2; ++kv) l.g[w][kv] = take(l.slot);
  l.step_ws = take(step);
  l.total = at;
  *out = l;
  return LOCOCO_OK;
}
}  // namespace

extern "C" {

lococo_status lococo_sequence_backward_workspace_bytes(const lococo_config* cfg, int64_t L, int32_t B, size_t* out) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if (!out) return fail(LOCOCO_EINVAL, "out is NULL");
  if (L < 0 || B <= 0) return fail(LOCOCO_EINVAL, "need L >= 0 and B > 0");
  SeqBwdLayout l;
  if ((st = seq_bwd_layout(cfg, L, B, INT64_MAX, true, false, &l))) return st;
  *out = l.total;
  return LOCOCO_OK;
}

lococo_status lococo_sequence_backward(const lococo_config* cfg, const lococo_qkvo* seq, int64_t L, int32_t B,
                                       const void* conv_w, const void* conv_b, const lococo_cache* cache0,
                                       const float* d_o, const float* d_final_k, const float* d_final_v,
                                       float* d_q, float* d_k, float* d_v, float* d_cache0_k, float* d_cache0_v,
                                       float* d_conv_w, float* d_conv_b, void* workspace, size_t ws_bytes,
                                       void* stream) {
  lococo_status st;
  if ((st = check_config(cfg))) return st;
  if ((st = check_cache(cfg, cache0))) return st;
  if (L <= 0) return fail(LOCOCO_EINVAL, "L must be positive");
  if (B <= 0) return fail(LOCOCO_EINVAL, "block length B must be positive");
  if (cfg->norm == 2) return fail(LOCOCO_EUNSUPPORTED, "norm = 2 (rectifier on the convolution input) is forward only");
  if (!seq) return fail(LOCOCO_EINVAL, "qkvo is NULL");
  if ((st = check_tensor(cfg, seq->q, "q", L)) || (st = check_tensor(cfg, seq->k, "k", L)) ||
      (st = check_tensor(cfg, seq->v, "v", L)))
    return st;
  if ((st = check_step_shape(cfg, B, std::min<int64_t>(cfg->M, (int64_t)cache0->len + L)))) return st;
  if (!d_o || !d_q || !d_k || !d_v || !d_cache0_k || !d_cache0_v) return fail(LOCOCO_EINVAL, "a gradient pointer is NULL");
  if (cfg->flags & LOCOCO_FLAG_FILTERS_PREPARED)
    return fail(LOCOCO_EINVAL, "LOCOCO_FLAG_FILTERS_PREPARED has no meaning here: the call uses workspaces of its own");
  int64_t n = 0;
  if ((st = lococo_plan(L, B, cfg->M, cache0->len, 0, nullptr, &n))) return st;
  std::vector<lococo_seg> plan((size_t)n);
  if ((st = lococo_plan(L, B, cfg->M, cache0->len, 0, plan.data(), &n))) return st;
  bool any_compress = false;
  for (const auto& sg : plan) any_compress |= sg.branch == 1;
  if (any_compress && (!conv_w || !d_conv_w)) return fail(LOCOCO_EINVAL, "conv_w or d_conv_w is NULL but the scan compresses");
  SeqBwdLayout l;
  if ((st = seq_bwd_layout(cfg, L, B, INT64_MAX, true, false, &l))) return st;
  if (ws_bytes < l.total && l.keep_logits && (st = seq_bwd_layout(cfg, L, B, INT64_MAX, false, false, &l))) return st;
  if (ws_bytes < l.total && l.window > 1) {    // the largest window that fits (a layout's size grows with its window)
    int64_t fits = 1, not_fits = l.window;
    while (not_fits - fits > 1) {
      const int64_t mid = (fits + not_fits) / 2;
      if ((st = seq_bwd_layout(cfg, L, B, mid, false, false, &l))) return st;
      (l.total <= ws_bytes ? fits : not_fits) = mid;
    }
    if ((st = seq_bwd_layout(cfg, L, B, fits, false, false, &l))) return st;
  }
  if (ws_bytes < l.total && (st = seq_bwd_layout(cfg, L, B, 1, false, true, &l))) return st;
  if (!workspace || ws_bytes < l.total || ((uintptr_t)workspace & 255))
    return fail(LOCOCO_EWORKSPACE, "workspace needs %zu bytes, 256-byte aligned (got %zu)", l.total,
                workspace ? ws_bytes : (size_t)0);
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)workspace;
  const size_t es = esize(cfg->dtype), d = (size_t)cfg->head_dim;
  const size_t chains = (size_t)cfg->batch * cfg->n_kv_heads, state = chains * cfg->M * d * es;

  // ---- the recurrence once more, keeping the state every block starts from: the fill branch or steps 4-5 only (the
  // same kernels as in the forward schedules, so the same states); nobody reads the attention outputs of step 3 here.
  // A fill appends in place: the states before the fill blocks are prefixes of one array, the slot of the first block
  // that compresses (of the last block, if none before it does).
  Path path;
  if ((st = resolve_path(cfg, B, &path))) return st;
  if ((st = check_mfma_strides(cfg, path, seq, B, false))) return st;
  int64_t n_fill = 0;
  while (n_fill < n - 1 && plan[(size_t)n_fill].branch == 0) ++n_fill;
  auto state_k = [&](int64_t i) { return ws + l.states_k + (size_t)std::max(i, n_fill) * l.state; };
  auto state_v = [&](int64_t i) { return ws + l.states_v + (size_t)std::max(i, n_fill) * l.state; };
  lococo_cache fc = *cache0;
  fc.cur = 0;
  fc.attn_colsum = nullptr;
  if (cache0->len > 0)
    HIP_TRY(launch_copy_pair(state_k(0), cache0->k[cache0->cur], state_v(0), cache0->v[cache0->cur], state, s),
            "copying the first state");
  // (on the fused path the filters' launch clears the counters and appends the leading fill blocks, where there is one)
  const bool folds = path == PATH_MFMA && n_fill + 1 < n;
  if (path == PATH_MFMA && !folds)
    HIP_TRY(launch_scan_sync_clear(ws + l.fwd_ws + filter_ws_bytes(cfg), cfg->batch, cfg->n_kv_heads, cfg->M, false, s),
            "clearing the scan counters");
  bool have_logits = false;                                  // the scan leaves them
  for (int64_t i = folds ? n_fill : 0; i + 1 < n; ++i) {                      // (the last block's own update is not needed)
    const lococo_seg& sg = plan[(size_t)i];
    fc.k[0] = state_k(i); fc.k[1] = state_k(i + 1);
    fc.v[0] = state_v(i); fc.v[1] = state_v(i + 1);
    fc.cur = 0;
    if (folds && i == n_fill) fc.len = sg.len_before;
    lococo_qkvo blk = *seq;
    blk.o = blk.q;                                           // (never written)
    const StepArgs a = make_args(cfg, &blk, sg.start, sg.len, &fc, conv_w, conv_b, true);
    if (i == n_fill && path != PATH_GENERIC) {               // the first block that compresses
      StepArgs f = make_args(cfg, &blk, 0, (int32_t)sg.start, &fc, conv_w, conv_b, true);
      f.m = cache0->len;
      f.new_k = state_k(0);
      f.new_v = state_v(0);
      if ((st = enqueue_repack(cfg, path, a, ws + l.fwd_ws, s, folds ? ws + l.fwd_ws + filter_ws_bytes(cfg) : nullptr,
                               folds && i ? &f : nullptr)))
        return st;
      bool taken = path == PATH_MFMA && scan_fits_one_launch(cfg, a);
      const bool keep = l.keep_logits && compress_scan_leaves_logits(a.protect != nullptr, cfg->conv_in, false);
      if (taken && (st = enqueue_scan(cfg, a, n - i - (keep ? 0 : 1), B, L - sg.start, ws + l.states_k, ws + l.states_v,
                                      (int64_t)(l.state / es), i + 1, n + 1, ws + l.fwd_ws, false, s, &taken,
                                      keep ? (float*)(ws + l.logits) + i * (int64_t)l.conv.logits_stride : nullptr,
                                      (int64_t)l.conv.logits_stride, l.conv.ld)))
        return st;
      if (taken) { have_logits = keep; break; }
    }
    lococo_cache next = fc;
    if ((st = enqueue_update(cfg, path, a, &next, ws + l.fwd_ws, B, s))) return st;
    fc.len = next.len;
  }

  // ---- reverse walk.  (gk, gv) = gradient w.r.t. the state AFTER the block at hand.  Step 3 of a block needs nothing
  // of the walk, only the states: on the MFMA kernels the attention of a window of blocks runs in one launch ahead of
  // the walk through it and leaves its share of the gradient w.r.t. each block's starting state in a slot of its own,
  // to which the step then adds.  The same goes for the logits of Eq. 5; and what nobody in the walk waits for, the
  // gradients w.r.t. the blocks' own rows and the filters, follows it for the whole window.
  const size_t gbytes = chains * cfg->M * d * sizeof(float);
  const float* gk = d_final_k;
  const float* gv = d_final_v;
  if (!gk) { gk = (const float*)(ws + l.g[0][0]); HIP_TRY(launch_zero_fill(ws + l.g[0][0], gbytes, s), "clearing the final gradient"); }
  if (!gv) { gv = (const float*)(ws + l.g[0][1]); HIP_TRY(launch_zero_fill(ws + l.g[0][1], gbytes, s), "clearing the final gradient"); }
  const bool batched = l.window > 0 && bwd_attn_on_mfma(cfg, seq, B);
  // The step's kernels write d_q, d_k and d_v before the last of them has read d_o, and d_cache0 before d_final: where these
  // share memory, what comes in is read from a copy.  So is what the plain contractions on the matrix cores could not read
  // where it is (see bwd_gemms_mfma_fit).
  const size_t q_bytes = (size_t)cfg->batch * cfg->n_q_heads * (size_t)L * d * sizeof(float), kv_bytes = chains * (size_t)L * d * sizeof(float);
  auto shared = [](const void* a, size_t na, const void* b, size_t nb) {
    return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
  };
  auto unaligned = [&](const void* p) { return cfg->dtype == LOCOCO_BF16 && ((uintptr_t)p & 15); };
  const bool copy_d_o = !batched && (unaligned(d_o) || shared(d_o, q_bytes, d_q, q_bytes) || shared(d_o, q_bytes, d_k, kv_bytes) ||
                                     shared(d_o, q_bytes, d_v, kv_bytes));
  if (!batched) {
    const float** from[2] = {&gk, &gv};
    for (int x = 0; x < 2; ++x) {
      const float* p = *from[x];
      float* own = (float*)(ws + l.g[0][x]);
      if (p == own || !(unaligned(p) || shared(p, gbytes, d_cache0_k, gbytes) || shared(p, gbytes, d_cache0_v, gbytes))) continue;
      HIP_TRY(hipMemcpyAsync(own, p, gbytes, hipMemcpyDeviceToDevice, s), "copying the final gradient");
      *from[x] = own;
    }
  }
  const int64_t G = batched ? l.window : n;
  bool conv_begun = false, walk_clear = false;       // the walk's counters are at zero
  int w = 1;
  for (int64_t w1 = n; w1 > 0;) {
    const int64_t w0 = std::max<int64_t>(0, w1 - G);
    if (batched) {
      const lococo_seg& first = plan[(size_t)w0];
      int64_t fills = 0;                       // fill blocks at the head of the window: their states are prefixes of the last one's
      while (w0 + fills < w1 - 1 && plan[(size_t)(w0 + fills)].branch == 0) ++fills;
      lococo_cache at = fc;
      at.k[0] = state_k(w0 + fills);
      at.v[0] = state_v(w0 + fills);
      at.cur = 0;
      at.len = first.len_before;
      lococo_qkvo blk = *seq;
      blk.o = blk.q;
      BwdAttnArgs t{};
      t.a = attn_args_one_block(make_args(cfg, &blk, first.start, B, &at, conv_w, conv_b, true));
      t.a.L = std::min<int64_t>(L - first.start, (w1 - w0) * (int64_t)B);
      t.a.n_seg = (int32_t)(w1 - w0);
      t.a.n_fill = (int32_t)fills;
      t.a.hist_k = ws + l.states_k + (size_t)(w0 + fills + 1) * l.state;
      t.a.hist_v = ws + l.states_v + (size_t)(w0 + fills + 1) * l.state;
      t.a.hist_stride = (int64_t)(l.state / es);
      t.a.hist_ring = (int32_t)(w1 - w0);      // (slots in order, never wrapped)
      t.d_o = d_o + first.start * (int64_t)d;
      t.d_q = d_q + first.start * (int64_t)d;
      t.d_k = d_k + first.start * (int64_t)d;
      t.d_v = d_v + first.start * (int64_t)d;
      t.d_ck = (float*)(ws + l.d_ck);
      t.d_cv = (float*)(ws + l.d_cv);
      if ((st = enqueue_bwd_attn(cfg, t, L, ws + l.hl, ws + l.stats, s))) return st;
    }
    int64_t w_steps = w1;                      // blocks w0 .. w_steps - 1 are left to the walk step by step
    if (batched && bwd_on_mfma(cfg)) {
      while (w_steps > w0 && plan[(size_t)(w_steps - 1)].branch == 1) --w_steps;   // (fills come first)
      if (w_steps < w1) {
        const lococo_seg& first = plan[(size_t)w_steps];
        lococo_cache at = fc;
        at.k[0] = state_k(w_steps);
        at.v[0] = state_v(w_steps);
        at.cur = 0;
        at.len = first.len_before;
        lococo_qkvo blk = *seq;
        blk.o = blk.q;
        BwdConvArgs c{};
        c.st = make_args(cfg, &blk, first.start, first.len, &at, conv_w, conv_b, true);
        c.n_blk = (int32_t)(w1 - w_steps);
        c.B = B;
        c.banks = filter_banks(cfg);
        c.tokens = std::min<int64_t>(L - first.start, c.n_blk * (int64_t)B);
        c.state_stride = (int64_t)(l.state / es);
        c.d_cache_k = (float*)(ws + l.d_ck + (size_t)(w_steps - w0) * l.slot);
        c.d_cache_v = (float*)(ws + l.d_cv + (size_t)(w_steps - w0) * l.slot);
        c.d_stride = (int64_t)(l.slot / sizeof(float));
        c.d_new_k = gk;
        c.d_new_v = gv;
        c.d_k = d_k + first.start * (int64_t)d;
        c.d_v = d_v + first.start * (int64_t)d;
        c.kv_chain = L * (int64_t)d;
        c.d_conv_w = d_conv_w;
        c.d_conv_b = d_conv_b;
        bwd_conv_place(&c, l.conv, ws + l.step_ws);
        if (l.keep_logits) c.logits = (float*)(ws + l.logits) + w_steps * c.logits_stride;
        if (!conv_begun) {
          walk_clear = path == PATH_MFMA && bwd_conv_walk_takes(c);
          HIP_TRY(launch_bwd_conv_begin(c, !have_logits, walk_clear ? ws + l.fwd_ws + filter_ws_bytes(cfg) : nullptr, s),
                  "filter packing launches");
        }
        conv_begun = true;
        if (first.len_before < cfg->M) {       // the rows no entry was live in: zero
          BwdArgs g{};
          g.st = c.st;
          g.d_cache_k = c.d_cache_k;
          g.d_cache_v = c.d_cache_v;
          g.attn_done = g.conv_elsewhere = 1;
          HIP_TRY(launch_step_backward_generic(cfg->dtype, g, true, s), "clearing the rows of empty slots");
        }
        if (!have_logits) HIP_TRY(launch_bwd_conv_logits(c, s), "conv launch");
        const bool defer = bwd_conv_defers_blocks(c);
        for (int i = c.n_blk - 1; i >= 0; --i) {
          int run = 0;                         // blocks from here down whose steps one launch can take
          if (path == PATH_MFMA && bwd_conv_walk_takes(c))
            while (run <= i && bwd_conv_three_parts(c, i - run) == bwd_conv_three_parts(c, i)) ++run;
          bool taken = false;
          if (run >= bwd_conv_walk_least(c, i) && (st = enqueue_bwd_walk(cfg, c, i, run, ws + l.fwd_ws, s, &walk_clear, &taken))) return st;
          if (taken) {
            i -= run - 1;
            continue;
          }
          const lococo_seg& sg = plan[(size_t)(w_steps + i)];
          HIP_TRY(launch_bwd_conv_rows(c, i, sg.len_before + sg.len, s), "row gradient launch");
          HIP_TRY(launch_bwd_conv_dx(c, i, 1, defer ? 0 : 2, sg.len_before + (defer ? 0 : sg.len), s), "input gradient launch");
        }
        if (defer) HIP_TRY(launch_bwd_conv_dx(c, 0, c.n_blk, 1, B, s), "input gradient launch");
        HIP_TRY(launch_bwd_conv_dw(c, s), "filter gradient launch");
        if (w_steps == 0 || plan[(size_t)(w_steps - 1)].branch == 0) HIP_TRY(launch_bwd_conv_end(c, s), "filter gradient launch");
        gk = c.d_cache_k;
        gv = c.d_cache_v;
      }
    }
    for (int64_t i = w_steps - 1; i >= w0; --i) {
      const lococo_seg& sg = plan[(size_t)i];
      lococo_cache before = fc;
      before.k[0] = state_k(i);
      before.v[0] = state_v(i);
      before.cur = 0;
      before.len = sg.len_before;
      lococo_qkvo blk = *seq;
      blk.o = blk.q;
      BwdArgs g{};
      g.st = make_args(cfg, &blk, sg.start, sg.len, &before, conv_w, conv_b, true);
      g.d_o = d_o + sg.start * (int64_t)d;
      g.o_chain = L * (int64_t)d;
      if (copy_d_o) {
        const size_t row = (size_t)sg.len * d * sizeof(float);
        HIP_TRY(hipMemcpy2DAsync(ws + l.d_o, row, g.d_o, (size_t)L * d * sizeof(float), row, (size_t)cfg->batch * cfg->n_q_heads,
                                 hipMemcpyDeviceToDevice, s), "copying a block's upstream gradient");
        g.d_o = (const float*)(ws + l.d_o);
        g.o_chain = sg.len * (int64_t)d;
      }
      g.d_new_k = gk;
      g.d_new_v = gv;
      g.d_q = d_q + sg.start * (int64_t)d;
      g.d_k = d_k + sg.start * (int64_t)d;
      g.d_v = d_v + sg.start * (int64_t)d;
      g.q_chain = g.kv_chain = L * (int64_t)d;
      if (batched) {
        g.d_cache_k = (float*)(ws + l.d_ck + (size_t)(i - w0) * l.slot);
        g.d_cache_v = (float*)(ws + l.d_cv + (size_t)(i - w0) * l.slot);
        g.attn_done = 1;
      } else {
        g.d_cache_k = i == 0 ? d_cache0_k : (float*)(ws + l.g[w][0]);
        g.d_cache_v = i == 0 ? d_cache0_v : (float*)(ws + l.g[w][1]);
        w ^= 1;
      }
      g.d_conv_w = d_conv_w;
      g.d_conv_b = d_conv_b;
      if ((st = enqueue_step_backward(cfg, g, sg.branch == 1, bwd_layout(cfg, sg.len, sg.len_before, l.one_filters), ws + l.step_ws, s))) return st;
      gk = g.d_cache_k;
      gv = g.d_cache_v;
    }
    if (batched) {                             // the slots are written again by the next window
      float* ok = w0 == 0 ? d_cache0_k : (float*)(ws + l.g[w][0]);
      float* ov = w0 == 0 ? d_cache0_v : (float*)(ws + l.g[w][1]);
      HIP_TRY(launch_copy_pair(ok, gk, ov, gv, gbytes, s), "handing on the gradient of a state");
      gk = ok;
      gv = ov;
      w ^= 1;
    }
    w1 = w0;
  }
  return LOCOCO_OK;
}

}  // extern "C"
