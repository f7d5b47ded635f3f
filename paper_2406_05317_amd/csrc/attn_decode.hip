// Attention of one new token per sequence as a launch of its own (the work of a workgroup is in attn_decode_row.h); a
// step whose compression leaves compute units idle has it in one launch with that (compress_step.hip).
#include "attn_decode_row.h"

namespace lococo {
namespace {

using namespace attn_decode_detail;

constexpr int kThreads = 1024;           // a wave per share: enough loads in flight to hide HBM latency on few workgroups

template <bool COLSUM>
__global__ __launch_bounds__(kThreads) void attn_decode_k(StepArgs a) {
  extern __shared__ float sc[];            // COLSUM: a.m raw scores (log2 units)
  __shared__ Parts part;
  attn_decode_row<kThreads / 64, COLSUM>(a, part, sc, blockIdx.x);
}

// LDS the kernel holds besides the scores
constexpr size_t kStaticLds = sizeof(Parts);

}  // namespace

bool attn_decode_supports(int dtype, int d, int Bn, int M, bool colsum) {
  if (colsum && kStaticLds + sizeof(float) * (size_t)M > 64 * 1024) return false;   // scores must fit LDS
  return dtype == LOCOCO_BF16 && d == kD && Bn == 1;
}

hipError_t launch_attn_decode(const StepArgs& a, hipStream_t s) {
  if (a.colsum)
    hipLaunchKernelGGL(attn_decode_k<true>, dim3(a.batch * a.Hq), dim3(kThreads), sizeof(float) * (size_t)a.M, s, a);
  else
    hipLaunchKernelGGL(attn_decode_k<false>, dim3(a.batch * a.Hq), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace lococo
