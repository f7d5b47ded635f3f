// Launches of the fused compression kernels (the work of a workgroup is in compress_tile.inl, or in compress_roles.h): which
// build a shape runs on, how its workgroups are dealt out, and the repacking of the filters.
#include "compress_roles.h"
#include "compress_tile.h"

namespace lococo {
namespace {

using namespace compress_detail;

template <int BM, int KW, int NORM, int PROT, int MULTI, int SPLIT, int LOG>
__global__ __launch_bounds__(kThreads, 1) void compress_mfma_k(ScanArgs sa, const uint16_t* wp, int64_t wp_head_stride) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t wg_id = blockIdx.x, wg_count = gridDim.x;
#include "compress_tile.inl"
}
template <int KW, int NORM, int PROT, int MULTI, int SPLIT, int CIN>
__global__ __launch_bounds__(kRoleThreads, 2) void compress_roles_k(ScanArgs sa, const uint16_t* wp, int64_t wp_head_stride) {
  extern __shared__ __align__(16) unsigned char smem[];
  compress_roles<KW, NORM, PROT, MULTI, SPLIT, CIN>(sa, wp, wp_head_stride, smem, blockIdx.x, gridDim.x);
}
// The kernel of an instantiation, its workgroups' threads and LDS.  ROLES: waves of two roles (compress_roles.h), which every
// [K | V] bank runs on, and a single step on the builds with two workgroups per pair; both kernels of a shape give the same bits.
template <int BM, int KW, int NORM, int PROT, int MULTI, int SPLIT, int CIN, int LOG, int ROLES>
struct Build {
  static constexpr int kWgThreads = ROLES ? kRoleThreads : kThreads;
  static constexpr int kLds = ROLES ? Roles<KW>::LDS : Geo<BM, KW>::LDS;
  static constexpr auto kernel() {
    if constexpr (ROLES != 0) return &compress_roles_k<KW, NORM, PROT, MULTI, SPLIT, CIN>;
    else return &compress_mfma_k<BM, KW, NORM, PROT, MULTI, SPLIT, LOG>;
  }
};

// [M][C][k] per bank -> register order (see compress_mfma_k); one thread per 16-byte chunk.  C = 128,
// or 256 ([K | V] filters): then a bank is its key half (channels 0..127 of every slot) in that
// order followed by its value half.
// Also zeroes what a scan starts with, and appends the blocks the cache has room for (workgroups from `fill_from` on, whole 16
// bytes at a time), where the call wants these: nothing of the three waits for the others, and a launch that does costs 3 - 4 us.
__global__ void repack_filters_k(const uint16_t* w, uint16_t* wp, int M, int C, int KW, int banks,
                                 int64_t w_head_stride, uint32_t* zero, int n_zero, uint32_t* zero2, int n_zero2, StepArgs f, int fill_from) {
  if ((int)blockIdx.x >= fill_from) {
    const int64_t per = (int64_t)f.Bn * 16, n = per * f.batch * f.Hkv, step = (int64_t)(gridDim.x - fill_from) * blockDim.x;
    for (int64_t e = (int64_t)(blockIdx.x - fill_from) * blockDim.x + threadIdx.x; e < n; e += step) {
      const int ch = (int)(e / per), r = (int)(e % per), t = r >> 4, c = (r & 15) * 8, b = ch / f.Hkv, h = ch % f.Hkv;
      const int64_t to = ((int64_t)ch * f.M + f.m + t) * kD + c;
      const u32x4 k = *(const u32x4*)((const uint16_t*)f.k.p + b * f.k.sb + h * f.k.sh + t * f.k.st + c);
      const u32x4 v = *(const u32x4*)((const uint16_t*)f.v.p + b * f.v.sb + h * f.v.sh + t * f.v.st + c);
      *(u32x4*)((uint16_t*)f.new_k + to) = k;
      *(u32x4*)((uint16_t*)f.new_v + to) = v;
    }
    return;
  }
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_zero; i += fill_from * blockDim.x) zero[i] = 0u;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_zero2; i += fill_from * blockDim.x) zero2[i] = 0u;
  const int64_t chunks_per_bank = (int64_t)M * KW * (C / 8);
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < chunks_per_bank * banks;
       e += (int64_t)fill_from * blockDim.x) {
    const int bank = (int)(e / chunks_per_bank);
    int64_t r = e % chunks_per_bank;
    const int lane = (int)(r % 64); r /= 64;
    const int h = (int)(r % 2); r /= 2;
    const int t = (int)(r % KW); r /= KW;
    const int wv = (int)(r % 4); r /= 4;
    const int tile = (int)(r % (M / 32)); r /= M / 32;      // r: which half of a [K | V] bank
    const int slot = tile * 32 + (lane & 31);
    const int c0 = (int)r * kD + 32 * wv + 16 * h + (lane >> 5) * 8;
    const uint16_t* src = w + bank * w_head_stride + ((int64_t)slot * C + c0) * KW + t;
#pragma unroll
    for (int q = 0; q < 8; ++q) wp[e * 8 + q] = src[(int64_t)q * KW];
  }
}

__global__ void zero_words_k(uint32_t* p, int n, uint32_t* p2, int n2) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += gridDim.x * blockDim.x) p2[i] = 0u;
}

// The instantiation a shape runs on, handed to `f` as compile-time constants (BM, KW, NORM, PROT, MULTI).
// 64-slot tiles when they still give every compute unit a workgroup, else 32-slot tiles; the filter
// slice of a 64-slot tile fits the registers for width 15 only.
bool use_big_tiles(int batch, int Hkv, int M, int k_width, int conv_in, int n_cu) {
  return k_width == 15 && !conv_in && (M % 64 == 0) && (int64_t)batch * Hkv * (M / 64) >= n_cu;
}
template <int V> using ic = std::integral_constant<int, V>;
// Parts the positions of a step are shared out between (1: no split).  Only with 32-slot tiles and
// one chain per workgroup, as long as the grid still fits the compute units and the cache part of
// a step alone gives every part four position tiles (with fewer, handing the partial results over
// costs more than the shorter walk saves: measured on the 3.5 K-token shape, M = 128).  A function of the shape and the device only:
// every schedule and every block of a scan use the same number, so results do not depend on them.
// Two workgroups per (chain, 32-slot tile) that take the steps of a scan in turn (SPLIT = 2 builds): whenever
// that still fits the compute units.  A function of the shape and the device only, like the position split
// (which it replaces where both would apply: a scan gains more from it).
bool step_pipeline(int batch, int Hkv, int M, int k_width, int conv_in, int n_cu) {
  if (debug_options().no_step_pipeline) return false;
  if (use_big_tiles(batch, Hkv, M, k_width, conv_in, n_cu)) return false;
  return (int64_t)batch * Hkv * (M / 32) * 2 <= n_cu;
}
int position_split(int batch, int Hkv, int M, int k_width, int conv_in, int n_cu) {
  if (use_big_tiles(batch, Hkv, M, k_width, conv_in, n_cu)) return 1;
  if (step_pipeline(batch, Hkv, M, k_width, conv_in, n_cu)) return 1;
  const int64_t grid = (int64_t)batch * Hkv * (M / 32);
  int p = 1;
  while (p < 4 && grid * (2 * p) <= n_cu && M / 32 >= 4 * (2 * p)) p *= 2;
  return p;
}
// builds whose last step can write to the caller beside those that always can (last_to_caller)
template <int BM, int KW, int PROT, int SPLIT>
constexpr bool kLastBuild = BM == 32 && KW == 15 && PROT == 0 && SPLIT == 2;
template <class F>
hipError_t with_instantiation(const StepArgs& t, bool multi, int split, int log, bool one_step, int n_cu, F&& f) {   // split: 0, 1 positions, 2 steps
  const bool big = use_big_tiles(t.batch, t.Hkv, t.M, t.k_width, t.conv_in, n_cu);
  auto pick_cin = [&](auto bm, auto kw, auto norm, auto prot, auto mu, auto spl) {
    if constexpr (decltype(bm)::value == 32) {
      if (t.conv_in) return f(bm, kw, norm, prot, mu, spl, ic<1>{}, ic<0>{}, ic<1>{});
      if constexpr (decltype(spl)::value == 2) {
        if (one_step) return f(bm, kw, norm, prot, mu, spl, ic<0>{}, ic<0>{}, ic<1>{});
      }
    }
    if constexpr (decltype(prot)::value == 0 && decltype(spl)::value != 1) {
      if (log == 1) return f(bm, kw, norm, prot, mu, spl, ic<0>{}, ic<1>{}, ic<0>{});
    }
    if constexpr (kLastBuild<decltype(bm)::value, decltype(kw)::value, decltype(prot)::value, decltype(spl)::value>) {
      if (log == 2) return f(bm, kw, norm, prot, mu, spl, ic<0>{}, ic<2>{}, ic<0>{});
    }
    return f(bm, kw, norm, prot, mu, spl, ic<0>{}, ic<0>{}, ic<0>{});
  };
  auto pick_multi = [&](auto bm, auto kw, auto norm, auto prot) {
    if constexpr (decltype(bm)::value == 32) {
      if (split == 1 && !multi) return pick_cin(bm, kw, norm, prot, ic<0>{}, ic<1>{});
      if (split == 2 && !multi) return pick_cin(bm, kw, norm, prot, ic<0>{}, ic<2>{});
    }
    return multi ? pick_cin(bm, kw, norm, prot, ic<1>{}, ic<0>{}) : pick_cin(bm, kw, norm, prot, ic<0>{}, ic<0>{});
  };
  auto pick_prot = [&](auto bm, auto kw, auto norm) {
    return t.protect ? pick_multi(bm, kw, norm, ic<1>{}) : pick_multi(bm, kw, norm, ic<0>{});
  };
  auto pick_norm = [&](auto bm, auto kw) {
    return t.norm == 1 ? pick_prot(bm, kw, ic<1>{}) : pick_prot(bm, kw, ic<0>{});
  };
  if (t.k_width == 15) return big ? pick_norm(ic<64>{}, ic<15>{}) : pick_norm(ic<32>{}, ic<15>{});
  if (t.k_width == 21) return pick_norm(ic<32>{}, ic<21>{});
  return hipErrorInvalidValue;   // compress_mfma_supports() keeps other shapes away
}

template <class B>
hipError_t prepare_kernel() {
  static bool attr_set = false;   // benign race: setting it twice is harmless
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)B::kernel(), hipFuncAttributeMaxDynamicSharedMemorySize, B::kLds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  return hipSuccess;
}

hipError_t dispatch(const ScanArgs& a, const uint16_t* wp, int64_t wp_head_stride, int n_cu, hipStream_t s) {
  const bool multi = a.groups < a.st.batch * a.st.Hkv;
  return with_instantiation(a.st, multi, a.pipe ? 2 : (a.psplit > 1 ? 1 : 0), a.logits ? 1 : !a.st.conv_in && a.last_k ? 2 : 0, a.n_steps == 1 && !a.logits, n_cu, [&](auto bm, auto kw, auto norm, auto prot, auto mu, auto sp, auto ci, auto lo, auto ro) {
    constexpr int BM = decltype(bm)::value, KW = decltype(kw)::value, NORM = decltype(norm)::value;
    constexpr int PROT = decltype(prot)::value, MULTI = decltype(mu)::value, SPLIT = decltype(sp)::value;
    constexpr int CIN = decltype(ci)::value, LOG = decltype(lo)::value, ROLES = decltype(ro)::value;
    using B = Build<BM, KW, NORM, PROT, MULTI, SPLIT, CIN, LOG, ROLES>;
    hipError_t e = prepare_kernel<B>();
    if (e != hipSuccess) return e;
    dim3 grid((a.st.M / BM) * a.groups * (SPLIT ? a.psplit : 1));
    hipLaunchKernelGGL(B::kernel(), grid, dim3(B::kWgThreads), B::kLds, s, a, wp, wp_head_stride);
    return hipGetLastError();
  });
}

}  // namespace

bool compress_mfma_supports(int dtype, int d, int M, int conv_width, int conv_in, int norm,
                            const char** why) {
  if (dtype != LOCOCO_BF16) { *why = "the MFMA kernels take bf16 storage only"; return false; }
  if (d != kD) { *why = "the MFMA kernels take head_dim = 128 only"; return false; }
  (void)conv_in;                     // filters over the keys or over [K | V]
  if (norm != 0 && norm != 1) { *why = "unknown normalisation"; return false; }
  if (conv_width != 15 && conv_width != 21) {
    *why = "the MFMA compression kernel is built for conv_width = 15 and 21";
    return false;
  }
  if (M % 32) { *why = "the MFMA compression kernel needs M to be a multiple of 32"; return false; }
  return true;
}

size_t compress_mfma_filter_bytes(int M, int conv_width, int conv_in, int banks) {
  return (size_t)banks * M * conv_width * kD * (conv_in ? 2 : 1) * 2;
}

// key-side logits of the first walk of a [K | V] bank: per (chain, 32-slot tile), one 32 x 32 fp32 tile per
// position tile of the longest step
static int64_t prelogits_stride(int M, int B) { return (int64_t)((M + B + BN - 1) / BN) * 32 * BN; }
size_t compress_prelogits_bytes(int batch, int Hkv, int M, int B, int conv_in, int n_cu) {
  const int64_t pairs = (int64_t)batch * Hkv * (M / 32);
  const int areas = pairs * 2 <= n_cu ? 2 : 1;     // one per workgroup of a pair that takes the steps in turn
  return conv_in ? (size_t)pairs * areas * prelogits_stride(M, B) * sizeof(float) : 0;
}

static uint32_t* psync_of(void* sync_ws, int batch, int Hkv) { return (uint32_t*)sync_ws + 2 * batch * Hkv + 1; }

hipError_t launch_repack_filters(const StepArgs& a, void* wp, int banks, void* sync_ws, hipStream_t s, const StepArgs* fill) {
  const int C = a.conv_in ? 2 * kD : kD;
  const int64_t n = (int64_t)banks * a.M * (C / 8) * a.k_width;   // 16-byte chunks
  int blocks = (int)((n + 255) / 256);
  if (blocks > 2048) blocks = 2048;
  const int64_t rows16 = fill ? (int64_t)fill->Bn * 16 * fill->batch * fill->Hkv : 0;
  const int fills = (int)(rows16 < 256 * 4096 ? (rows16 + 255) / 256 : 4096);
  hipLaunchKernelGGL(repack_filters_k, dim3(blocks + fills), dim3(256), 0, s, (const uint16_t*)a.conv_w,
                     (uint16_t*)wp, a.M, C, a.k_width, banks, a.w_head_stride, (uint32_t*)sync_ws,
                     sync_ws ? 2 * a.batch * a.Hkv + 1 : 0, sync_ws ? psync_of(sync_ws, a.batch, a.Hkv) : nullptr,
                     sync_ws ? 2 * a.batch * a.Hkv * (a.M / 32) : 0, fill ? *fill : a, blocks);
  return hipGetLastError();
}

// [chain counters][status word][per chain: bit mask of the XCDs its workgroups run on][per (chain,
// 32-slot tile): count of the parts of a split step that have handed in their result, census of the
// XCDs the parts run on (3 bits per XCD)]
size_t compress_scan_sync_bytes(int batch, int Hkv, int M) {
  return ((size_t)batch * Hkv * (2 + 2 * (M / 32)) + 1) * sizeof(uint32_t);
}

int compress_position_split(int batch, int Hkv, int M, int k_width, int conv_in, int n_cu) {
  return position_split(batch, Hkv, M, k_width, conv_in, n_cu);
}
int compress_step_pipeline(int batch, int Hkv, int M, int k_width, int conv_in, int n_cu) {
  return step_pipeline(batch, Hkv, M, k_width, conv_in, n_cu) ? 2 : 1;
}
// room for every part's result of one step: [chain][tile][part] x (32 x 2 d accumulators + 32 references + 32 sums)
size_t compress_partials_bytes(int batch, int Hkv, int M, int k_width, int conv_in, int n_cu) {
  const int p = position_split(batch, Hkv, M, k_width, conv_in, n_cu);
  return p > 1 ? (size_t)batch * Hkv * (M / 32) * p * Geo<32, 15>::PART_FLOATS * sizeof(float) : 0;
}

hipError_t launch_scan_sync_clear(void* sync_ws, int batch, int Hkv, int M, bool keep_status, hipStream_t s) {
  const int chains = batch * Hkv;
  // everything, or the chain counters and the part counters only
  hipLaunchKernelGGL(zero_words_k, dim3(1), dim3(256), 0, s, (uint32_t*)sync_ws, keep_status ? chains : 2 * chains + 1,
                     psync_of(sync_ws, batch, Hkv), 2 * chains * (M / 32));
  return hipGetLastError();
}

hipError_t launch_compress_mfma(const StepArgs& a, const void* wp, int banks, int n_cu, void* sync_ws,
                                void* partials, void* prelogits, int B, hipStream_t s, const AttnArgs* attn) {
  ScanArgs sa;
  sa.st = a;
  sa.n_steps = 1;
  sa.B = a.Bn;
  sa.tokens_left = a.Bn;
  sa.out_k = a.new_k;
  sa.out_v = a.new_v;
  sa.out_stride = 0;
  sa.slot0 = 0;
  sa.ring = 1;
  sa.sync = nullptr;
  sa.status = nullptr;
  sa.logits = nullptr;
  sa.logits_stride = sa.logits_ld = 0;
  sa.spin_limit = 0;
  sa.same_l2_allowed = debug_options().chain_sync_device ? 0 : 1;   // (only the hand-off of a split step looks at it here)
  // more (chain, tile) pairs than compute units: one resident workgroup per compute unit, each
  // taking several chains on one load of its filter slice (nothing to wait for within one step)
  sa.groups = compress_scan_groups(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, a.w_head_stride != 0 || a.b_head_stride != 0, n_cu);
  if (sa.groups <= 0) sa.groups = a.batch * a.Hkv;
  if (a.conv_in) {
    sa.prelogits = (float*)prelogits;
    sa.pre_stride = prelogits_stride(a.M, B > a.Bn ? B : a.Bn);
  } else {
    sa.last_k = sa.last_v = nullptr;
  }
  // fewer than half as many: the positions of the step are shared out between several workgroups,
  // whose count per (chain, tile) starts at zero
  sa.psplit = sa.groups < a.batch * a.Hkv ? 1 : position_split(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, n_cu);
  sa.pipe = sa.groups == a.batch * a.Hkv && step_pipeline(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, n_cu) ? 1 : 0;
  sa.partials = (float*)partials;
  sa.psync = psync_of(sync_ws, a.batch, a.Hkv);
  if (sa.pipe) sa.psplit = 2;            // (workgroups per pair; nothing is handed over)
  if (sa.psplit > 1 && !sa.pipe) {
    hipLaunchKernelGGL(zero_words_k, dim3(1), dim3(256), 0, s, sa.psync, 2 * a.batch * a.Hkv * (a.M / 32), sa.psync, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int64_t wp_head_stride = banks > 1 ? (int64_t)a.M * a.k_width * kD * (a.conv_in ? 2 : 1) : 0;
  if (attn) return launch_compress_step(sa, *attn, wp, wp_head_stride, s);
  return dispatch(sa, (const uint16_t*)wp, wp_head_stride, n_cu, s);
}

bool compress_scan_last_to_caller(const StepArgs& a, int B, int64_t n_steps, int n_cu) {
  // (scans over [K | V] run on the kernel of two roles, which single steps of 17 us share: with the choice in it these took 0.4 us
  // longer)
  if (a.conv_in) return false;
  const bool per_head = a.w_head_stride != 0 || a.b_head_stride != 0;
  const bool multi = compress_scan_groups(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, per_head, n_cu) < a.batch * a.Hkv;
  if (last_to_caller(use_big_tiles(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, n_cu) ? 64 : 32, a.k_width, multi)) return true;
  // The build of pairs that can tell its last step costs as much more a step as its walk is long, the copy 2 - 3 us a call.  With it
  // against without, us: 96 slots of 192 positions, 32 chains, 3 steps 57.6 and 60.2, 127 steps 1147 and 1163; 512 of 798, 8 chains, 3
  // steps 114.3 and 116.1, 9 steps 258.1 and 256.2, 127 steps 3139 and 3096; 256 of 512, 9 steps 161.4 and 162.2, 63 steps 896 and 891.
  const int T = a.M + B;
  return !a.protect && (T <= 256 || n_steps * T <= 5000) && step_pipeline(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, n_cu);
}

bool compress_scan_leaves_logits(bool protect, int conv_in, bool position_split) { return !protect && !conv_in && !position_split; }

int compress_tile_slots(int batch, int Hkv, int M, int k_width, int conv_in, int n_cu) {
  return use_big_tiles(batch, Hkv, M, k_width, conv_in, n_cu) ? 64 : 32;
}

int compress_scan_max_resident(const StepArgs& a, int n_cu) {
  if (debug_options().max_resident > 0) return (int)debug_options().max_resident;
  const int groups = compress_scan_groups(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, a.w_head_stride != 0 || a.b_head_stride != 0, n_cu);
  const bool multi = groups < a.batch * a.Hkv;
  const int split = multi ? 0 : step_pipeline(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, n_cu) ? 2
                    : position_split(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, n_cu) > 1 ? 1 : 0;
  int per_cu = 0;
  hipError_t e = with_instantiation(a, multi, split, 0, false, n_cu, [&](auto bm, auto kw, auto norm, auto prot, auto mu, auto sp, auto ci, auto lo, auto ro) {
    constexpr int BM = decltype(bm)::value, KW = decltype(kw)::value, NORM = decltype(norm)::value;
    constexpr int PROT = decltype(prot)::value, MULTI = decltype(mu)::value, SPLIT = decltype(sp)::value;
    constexpr int CIN = decltype(ci)::value, LOG = decltype(lo)::value, ROLES = decltype(ro)::value;
    using B = Build<BM, KW, NORM, PROT, MULTI, SPLIT, CIN, LOG, ROLES>;
    hipError_t e2 = prepare_kernel<B>();
    if (e2 != hipSuccess) return e2;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)B::kernel(), B::kWgThreads, B::kLds);
  });
  if (e != hipSuccess) { (void)hipGetLastError(); return 0; }
  return per_cu * n_cu;
}

int compress_scan_groups(int batch, int Hkv, int M, int k_width, int conv_in, bool per_head, int n_cu) {
  const int bm = use_big_tiles(batch, Hkv, M, k_width, conv_in, n_cu) ? 64 : 32;
  const int tiles = M / bm, chains = batch * Hkv;
  // one workgroup per compute unit (LDS): every workgroup of the launch must be resident at once
  int g = n_cu / tiles;
  if (g >= chains) return chains;
  // Fewer workgroups than (chain, tile) pairs: each takes several chains.  They must share its
  // resident filter slice, and the tiles of a group should share an XCD (ids are dealt round-robin
  // over 8 XCDs: a multiple of 8 groups does that).
  const int unit = per_head ? (Hkv % 8 == 0 ? Hkv : (8 % Hkv == 0 ? 8 : 8 * Hkv)) : 8;
  if (g >= unit) g -= g % unit;
  else if (per_head) g -= g % Hkv;
  return g;
}

hipError_t launch_compress_scan(const ScanArgs& a_in, const void* wp, int banks, int n_cu,
                                void* sync_ws, void* partials, void* prelogits, hipStream_t s) {
  ScanArgs a = a_in;
  const int chains = a.st.batch * a.st.Hkv;
  a.sync = (uint32_t*)sync_ws;
  a.status = (int32_t*)sync_ws + chains;
  a.groups = compress_scan_groups(a.st.batch, a.st.Hkv, a.st.M, a.st.k_width, a.st.conv_in,
                                  a.st.w_head_stride != 0 || a.st.b_head_stride != 0, n_cu);
  if (a.st.conv_in) {
    a.prelogits = (float*)prelogits;
    a.pre_stride = prelogits_stride(a.st.M, a.B > a.st.Bn ? a.B : a.st.Bn);
  }
  if (a.groups <= 0) return hipErrorInvalidValue;   // the caller keeps such shapes away
  if (!a.st.conv_in && a.last_k && !compress_scan_last_to_caller(a.st, a.B, a.n_steps, n_cu)) return hipErrorInvalidValue;   // (and these)
  a.psplit = a.groups < chains ? 1 : position_split(a.st.batch, a.st.Hkv, a.st.M, a.st.k_width, a.st.conv_in, n_cu);
  a.pipe = a.groups == chains && step_pipeline(a.st.batch, a.st.Hkv, a.st.M, a.st.k_width, a.st.conv_in, n_cu) ? 1 : 0;
  if (a.pipe) a.psplit = 2;
  a.partials = (float*)partials;
  a.psync = psync_of(sync_ws, a.st.batch, a.st.Hkv);
  const int64_t wp_head_stride = banks > 1 ? (int64_t)a.st.M * a.st.k_width * kD * (a.st.conv_in ? 2 : 1) : 0;
  return dispatch(a, (const uint16_t*)wp, wp_head_stride, n_cu, s);
}

}  // namespace lococo
