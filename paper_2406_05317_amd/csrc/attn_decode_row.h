// Attention of Alg. 2 step 3 for the generation stage (one new token per
// sequence, B = 1): softmax(q [K_cache ; k_new]^T / sqrt(d)) [V_cache ; v_new]
// for one query row per head.  bf16 storage, fp32 arithmetic, head_dim 128.
//
// One query row against m + 1 keys is a matrix-vector product, not a matrix
// product: 4(m+1)d flops per head against 4(m+1)d bytes of keys and values, so
// the roofline that bounds it is HBM (or, with 32 heads, the launch itself).
// The MFMA attention kernel would spend a 128-query tile on this one row.
//
// One workgroup per (batch, query head).  A key row is 256 bytes =
// 16 lanes x 16 bytes, so one wave-wide load brings 4 consecutive keys; sixteen
// shares of the keys take groups of 4 keys round-robin.  Each 16-lane group of a
// share keeps its own online softmax state (reference, row sum, 8 output columns
// per lane); the 64 states of a workgroup are merged through LDS at the end.
//
// With accumulated attention scores asked for (StepArgs::colsum), the raw
// scores of the cache slots are also kept in LDS, and once the row's reference
// and sum are known every slot's probability is added to its accumulator.
#pragma once

#include "lococo_internal.h"

namespace lococo {
namespace attn_decode_detail {

constexpr int kD = 128;
constexpr int kWaves = 16, kParts = kWaves * 4;      // shares of the keys, whatever the number of real waves
constexpr float kLog2e = 1.4426950408889634f;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// sum over the 16 lanes of a row, result in every lane: quad xor 1, quad xor 2, mirror inside
// 8 lanes, mirror inside 16 lanes
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  v += dpp<0x140>(v);
  return v;
}
__device__ __forceinline__ void unpack8(const u32x4& r, float* f) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(r[i] << 16);
    f[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u);
  }
}

// The row of one (batch entry, query head) by a workgroup of WAVES waves: every wave takes kWaves / WAVES of the sixteen
// shares of the keys, so that the sums, and the bits, do not depend on the number of waves.
struct Parts {
  float o[kParts][kD + 4];
  float m[kParts], l[kParts];
  float fin[2];
};
template <int WAVES, bool COLSUM>
__device__ __forceinline__ void attn_decode_row(const StepArgs& a, Parts& part, float* sc, int row) {
  constexpr int V = kWaves / WAVES, kThreads = WAVES * 64;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, grp = l >> 4, c16 = l & 15;
  const int hq = row % a.Hq, b = row / a.Hq, hkv = hq / a.group;
  const int ch = b * a.Hkv + hkv;
  const int T = a.m + 1;

  float q[8];
  unpack8(*(const u32x4*)((const uint16_t*)a.q.p + b * a.q.sb + hq * a.q.sh + c16 * 8), q);
  const float c = a.scale * kLog2e;               // exp(x * scale) = exp2(x * c)
#pragma unroll
  for (int i = 0; i < 8; ++i) q[i] *= c;

  const uint16_t* ck = (const uint16_t*)a.cache_k + (int64_t)ch * a.M * kD + c16 * 8;
  const uint16_t* cv = (const uint16_t*)a.cache_v + (int64_t)ch * a.M * kD + c16 * 8;
  const uint16_t* nk = (const uint16_t*)a.k.p + b * a.k.sb + hkv * a.k.sh + c16 * 8;
  const uint16_t* nv = (const uint16_t*)a.v.p + b * a.v.sb + hkv * a.v.sh + c16 * 8;

  float m_run[V], l_run[V], o[V][8];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    m_run[v] = -INFINITY;
    l_run[v] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[v][i] = 0.f;
  }
  // share s = w * V + v has the keys 8 * kWaves * it + 4 * s + grp (+ 4 * kWaves); two groups of loads in flight per
  // iteration and share
  for (int jb = 0; jb < T; jb += 8 * kWaves) {
    u32x4 k0[V], v0[V], k1[V], v1[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int j0 = jb + 4 * (w * V + v) + grp, j1 = j0 + 4 * kWaves;
      k0[v] = v0[v] = k1[v] = v1[v] = u32x4{0, 0, 0, 0};
      if (j0 < T) {
        k0[v] = *(const u32x4*)(j0 < a.m ? ck + (int64_t)j0 * kD : nk);
        v0[v] = *(const u32x4*)(j0 < a.m ? cv + (int64_t)j0 * kD : nv);
      }
      if (j1 < T) {
        k1[v] = *(const u32x4*)(j1 < a.m ? ck + (int64_t)j1 * kD : nk);
        v1[v] = *(const u32x4*)(j1 < a.m ? cv + (int64_t)j1 * kD : nv);
      }
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int j0 = jb + 4 * (w * V + v) + grp, j1 = j0 + 4 * kWaves;
      if (j0 >= T) continue;
      const bool has1 = j1 < T;
      float kf[8], s0 = 0.f, s1 = 0.f;
      unpack8(k0[v], kf);
#pragma unroll
      for (int i = 0; i < 8; ++i) s0 = fmaf(q[i], kf[i], s0);
      unpack8(k1[v], kf);
#pragma unroll
      for (int i = 0; i < 8; ++i) s1 = fmaf(q[i], kf[i], s1);
      s0 = row16_sum(s0);                            // scores in log2 units
      s1 = has1 ? row16_sum(s1) : -INFINITY;
      if (COLSUM && c16 == 0) {
        if (j0 < a.m) sc[j0] = s0;
        if (j1 < a.m) sc[j1] = s1;
      }
      const float m_new = fmaxf(m_run[v], fmaxf(s0, s1));
      const float alpha = __builtin_amdgcn_exp2f(m_run[v] - m_new);
      const float p0 = __builtin_amdgcn_exp2f(s0 - m_new), p1 = __builtin_amdgcn_exp2f(s1 - m_new);
      l_run[v] = l_run[v] * alpha + p0 + p1;
      m_run[v] = m_new;
      float vf[8];
      unpack8(v0[v], vf);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[v][i] = fmaf(p0, vf[i], o[v][i] * alpha);
      unpack8(v1[v], vf);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[v][i] = fmaf(p1, vf[i], o[v][i]);
    }
  }

  // merge the partial states (one per share and lane group); a group that saw no key has
  // m = -inf, l = 0 and weighs nothing
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int pi = (w * V + v) * 4 + grp;
#pragma unroll
    for (int i = 0; i < 8; ++i) part.o[pi][c16 * 8 + i] = o[v][i];
    if (c16 == 0) {
      part.m[pi] = m_run[v];
      part.l[pi] = l_run[v];
    }
  }
  __syncthreads();
  if (tid < kD) {
    float mx = part.m[0];
#pragma unroll
    for (int p = 1; p < kParts; ++p) mx = fmaxf(mx, part.m[p]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
      const float wgt = __builtin_amdgcn_exp2f(part.m[p] - mx);   // exp2(-inf) = 0 for empty groups
      num = fmaf(wgt, part.o[p][tid], num);
      den = fmaf(wgt, part.l[p], den);
    }
    if (COLSUM && tid == 0) {
      part.fin[0] = mx;
      part.fin[1] = den;
    }
    const float r = num / den;
    // round to nearest even bf16
    uint32_t u = __float_as_uint(r);
    u += 0x7fffu + ((u >> 16) & 1u);
    ((uint16_t*)a.o.p)[b * a.o.sb + hq * a.o.sh + tid] = (uint16_t)(u >> 16);
  }
  if (COLSUM) {
    __syncthreads();
    const float mx = part.fin[0], inv = 1.f / part.fin[1];
    float* cs = a.colsum + (int64_t)ch * a.M;
    for (int j = tid; j < a.m; j += kThreads) atomicAdd(cs + j, __builtin_amdgcn_exp2f(sc[j] - mx) * inv);
  }
}

}  // namespace attn_decode_detail
}  // namespace lococo
