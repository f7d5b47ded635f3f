// One block step in one launch: the attention of the block and its compression need only the state before the step, not
// each other.  Where the compression of a single step leaves compute units without a workgroup (each workgroup of it fills
// one: LDS and registers), the attention's workgroups take those.  The bodies are those of the separate launches, so are
// the bits.  Bound by the compression (filter slice, walk, epilogue in series); measured, one token of 32 heads on 128
// slots: 16.2 us as two launches (11.1 + 5), 11.9 us as one, 10.9 with the compression on waves of two roles; 77 tokens of 32
// heads on 8 kv heads, 256 slots: 29.2 us (18.5 + 10.5), 18.9, 16.7 us (on inputs not in any cache 43.6 -> 41.3 us: there the first
// reads of the filters and of the cache, one after the other, are most of it).
#include "attn_decode_row.h"
#include "attn_tile.h"
#include "compress_roles.h"

namespace lococo {
namespace {

using namespace compress_detail;

template <int KW, int NORM, int CIN>
__global__ __launch_bounds__(kRoleThreads, 2) void compress_step_k(ScanArgs sa, const uint16_t* wp, int64_t wp_head_stride,
                                                               int n_compress, AttnArgs at) {
  extern __shared__ __align__(16) unsigned char smem[];
  if ((int)blockIdx.x >= n_compress) {
    const int id = blockIdx.x - n_compress;
    if (sa.st.Bn == 1)
      attn_decode_detail::attn_decode_row<kRoleThreads / 64, false>(sa.st, *(attn_decode_detail::Parts*)smem, nullptr, id);
    else if (threadIdx.x < 256)              // (its work is cut for four waves)
      attn_tile_detail::attn_tile(at, smem, id);
    return;
  }
  // The build that has two workgroups per pair in a scan, of which the first has the one step: item 2 k of twice n_compress,
  // numbered so that the slot tiles of a chain are on one XCD here too
  const uint32_t wg_count = 2 * n_compress, per = wg_count / 8;
  uint32_t k = blockIdx.x;
  if (k < n_compress / 8u * 8u) k = (k % 8) * (n_compress / 8u) + k / 8;
  const uint32_t wg_id = 2 * k < per * 8 ? 2 * k % per * 8 + 2 * k / per : 2 * k;
  compress_roles<KW, NORM, 0, 0, 2, CIN>(sa, wp, wp_head_stride, smem, wg_id, wg_count);
}

template <int KW, int NORM, int CIN>
hipError_t launch(const ScanArgs& sa, const uint16_t* wp, int64_t wp_head_stride, const AttnArgs& at, int n_attn, hipStream_t s) {
  constexpr int lds = Roles<KW>::LDS;
  static_assert(lds >= attn_tile_detail::LDS_BYTES && lds >= (int)sizeof(attn_decode_detail::Parts), "one LDS area for all");
  static bool attr_set = false;   // benign race: setting it twice is harmless
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)compress_step_k<KW, NORM, CIN>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int n = sa.st.batch * sa.st.Hkv * (sa.st.M / 32);
  hipLaunchKernelGGL((compress_step_k<KW, NORM, CIN>), dim3(n + n_attn), dim3(kRoleThreads), lds, s, sa, wp, wp_head_stride, n, at);
  return hipGetLastError();
}

int attn_workgroups(const StepArgs& a) { return a.batch * a.Hq * (a.Bn == 1 ? 1 : (a.Bn + 127) / 128); }

}  // namespace

// Whether the step's two halves fit the device side by side: a compression that runs on pairs of workgroups in a scan (so
// that at most half of the compute units have work in a single step), every workgroup of both on a compute unit of its own.
// With more, the attention's would queue behind the compression's and nothing overlaps.
bool compress_step_fits(const StepArgs& a, int n_cu) {
  if (a.protect || a.colsum || a.Bn < 1) return false;
  if (compress_step_pipeline(a.batch, a.Hkv, a.M, a.k_width, a.conv_in, n_cu) != 2) return false;
  return (int64_t)a.batch * a.Hkv * (a.M / 32) + attn_workgroups(a) <= n_cu;
}

hipError_t launch_compress_step(const ScanArgs& sa, const AttnArgs& at_in, const void* wp, int64_t wp_head_stride, hipStream_t s) {
  const StepArgs& a = sa.st;
  AttnArgs at = at_in;
  at.qtiles = (a.Bn + 127) / 128;
  const int n_attn = attn_workgroups(a);
  const uint16_t* w = (const uint16_t*)wp;
  auto with_cin = [&](auto kw, auto norm) {
    constexpr int KW = decltype(kw)::value, NORM = decltype(norm)::value;
    return a.conv_in ? launch<KW, NORM, 1>(sa, w, wp_head_stride, at, n_attn, s) : launch<KW, NORM, 0>(sa, w, wp_head_stride, at, n_attn, s);
  };
  auto with_norm = [&](auto kw) {
    return a.norm == 1 ? with_cin(kw, std::integral_constant<int, 1>{}) : with_cin(kw, std::integral_constant<int, 0>{});
  };
  if (a.k_width == 15) return with_norm(std::integral_constant<int, 15>{});
  if (a.k_width == 21) return with_norm(std::integral_constant<int, 21>{});
  return hipErrorInvalidValue;
}

}  // namespace lococo
