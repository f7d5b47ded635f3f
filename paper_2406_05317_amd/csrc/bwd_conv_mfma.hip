// Backward of Eq. 5, 6 and 4 of the compress steps of a window of blocks, bf16 storage, head_dim 128, filters over the
// keys or over [K | V], any odd width up to 31.  With X = [cache ; block], g = the gradient w.r.t. the new cache:
//
//   G[i, j]      = g_k[i] . Xk[j] + g_v[i] . Xv[j]                                  (Eq. 4 w.r.t. the weights)
//   dl[i, j]     = n[i, j] (G[i, j] - sum_j n G)                                    (Eq. 6; n: the normalised row i)
//   dX[j, :]    += sum_i n[i, j] g[i, :] + sum_t sum_i dl[i, j - t + p] W[i, :, t]  (Eq. 4 and Eq. 5 w.r.t. the entries)
//   dW[i, c, t] += sum_j dl[i, j] X[j + t - p, c]                                   (Eq. 5 w.r.t. the filters)
//
// Only g has to wait for the walk, and of dX only the rows of the cache are what the walk hands on.  So the logits of all
// blocks come from the recomputed scan, or from one launch ahead of the walk (tiled_mfma.hip), the walk is one launch for all blocks
// (bwd_walk_k) or two for each (bwd_rows_k, bwd_dx_k over the cache rows), and the rows of the blocks and the filter gradient follow
// in one launch each for the whole window.
//
// g, n and dl enter the matrix products as two bf16 halves (16 bits kept): n g in three products, the others in two.  In a
// block whose number of positions is no multiple of 4, and in a step whose gradients are not 16-byte aligned, n and g enter as
// three parts (G 3 products, n g 6): Eq. 4 of those has always been computed in fp32, and its error stays at that level.  dl
// and n are kept as "planes" [chain][32 slots][position][32 high halves | 32 low halves]: 128 bytes per position, read row
// by row where the slots are contracted (bwd_dx_k) and down the rows where the positions are (bwd_dw_k).
#include <algorithm>
#include <type_traits>

#include "lococo_internal.h"
#include "mfma_util.h"

namespace lococo {
namespace {

constexpr int kD = 128;

// 64 lanes x 16 bytes, lane l from its own address p into cell l of the 1 KB of LDS at lds_addr (see load_to_lds)
__device__ __forceinline__ void gather_to_lds(const unsigned char* p, uint32_t lds_addr) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "{m0}"(lds_addr), "v"(p) : "memory");
}
// the same from a uniform address and a 32-bit offset per lane
__device__ __forceinline__ void gather_to_lds(const unsigned char* base, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "{m0}"(lds_addr), "v"(voff), "s"(base) : "memory");
}
// and from a buffer: offset `voff` per lane and `soff` for all
__device__ __forceinline__ void load_to_lds_at(const u32x4& rsrc, uint32_t lds_addr, uint32_t voff, uint32_t soff) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" :: "{m0}"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
// every wave has finished reading and its awaited loads have landed (waited for by hand)
__device__ __forceinline__ void barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Rows of 128 bytes in LDS (8 cells): chunk c of row r sits in cell c ^ pswz(r).  Sixteen consecutive rows put one chunk on
// sixteen different cells of 256 bytes; four rows from a multiple of four put four consecutive chunks there.
__device__ __forceinline__ int pswz(int r) { return (((r >> 1) & 1) << 2) | ((r >> 2) & 3); }

struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

struct Block { int m, Bn, T; const uint16_t* ck; const uint16_t* cv; const uint16_t* k; const uint16_t* v; };
__device__ __forceinline__ Block block_of(const BwdConvArgs& g, int blk) {
  const StepArgs& a = g.st;
  Block b;
  const int64_t left = g.tokens - (int64_t)blk * g.B;
  b.m = blk ? a.M : a.m;
  b.Bn = (int)(left < g.B ? left : g.B);
  b.T = b.m + b.Bn;
  b.ck = (const uint16_t*)a.cache_k + blk * g.state_stride;
  b.cv = (const uint16_t*)a.cache_v + blk * g.state_stride;
  b.k = (const uint16_t*)a.k.p + (int64_t)blk * g.B * a.k.st;
  b.v = (const uint16_t*)a.v.p + (int64_t)blk * g.B * a.v.st;
  return b;
}
// gradient w.r.t. the state after a block: that of the next block's state
__device__ __forceinline__ const float* grad_new(const BwdConvArgs& g, int blk, bool val) {
  if (blk + 1 < g.n_blk) return (val ? g.d_cache_v : g.d_cache_k) + (blk + 1) * g.d_stride;
  return val ? g.d_new_v : g.d_new_k;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// v[i] (i < 16) reduced over the 32 lanes of each half of a wave: every step halves the values a lane still carries, so
// that lane l31 ends with the result of i = l31 / 2.
template <bool MAX>
__device__ __forceinline__ float over32(const f32x16& v, int l31) {
  auto op = [](float x, float y) { return MAX ? fmaxf(x, y) : x + y; };
  float a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {            // lanes 16 .. 31 keep i + 8
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 8]), false, false);
    a[i] = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  const bool b3 = l31 & 8, b2 = l31 & 4, b1 = l31 & 2;
  float b[4], c[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {            // row_ror:8, the lane 8 away
    const float keep = b3 ? a[i + 4] : a[i], give = b3 ? a[i] : a[i + 4];
    b[i] = op(keep, dpp<0x128>(give));
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {            // row_half_mirror: the other four of eight lanes
    const float keep = b2 ? b[i + 2] : b[i], give = b2 ? b[i] : b[i + 2];
    c[i] = op(keep, dpp<0x141>(give));
  }
  const float keep = b1 ? c[1] : c[0], give = b1 ? c[0] : c[1];
  const float d = op(keep, dpp<0x4E>(give));   // quad_perm [2,3,0,1]
  return op(d, dpp<0xB1>(d));                  // quad_perm [1,0,3,2]
}
// exp(x), x <= 0: the product with log2 e carried to twice the working precision (v_exp_f32 is exact to one unit)
__device__ __forceinline__ float exp_neg(float x) {
  constexpr float lo2e = 1.9259629911e-8f;                 // log2(e) - (float)log2(e)
  const float t = x * kLog2e, r = fmaf(x, lo2e, fmaf(x, kLog2e, -t));
  const float e = __builtin_amdgcn_exp2f(t);
  return x < -104.f ? 0.f : fmaf(e, r * 0.69314718f, e);   // (below: zero, and -inf has no remainder)
}

// ---- G, Eq. 6 and its gradient: a workgroup per (chain, 32 slots), all positions, eight waves of NT 32-position tiles
// each; the rows of a step stay in registers from the logits to dl.  Bound by memory in turns, one workgroup filling a compute
// unit from 257 positions on: the logits in (64 MB a step of 32 chains, 512 slots, 1024 positions), the entries from the L2 (512 KB a
// workgroup), the planes out (134 MB): 66 us a step; as five kernels with fp32 arrays in memory between them 250 us.  Up to 256
// positions two share it (128 slots on 256: 13.0 us for 128 workgroups, 22.8 for 512; 96 on 177, three parts, 384 workgroups: 20.7,
// one to a compute unit 26.1).  Entries and planes go through LDS, 4 KB of a wave's own, so that an instruction covers whole lines: with
// fragments straight from memory and 16 bytes a lane straight to it, 32 lines an instruction in quarters, 83 and 14.8 us.
// MULTI: more positions than that: they are walked twice in chunks, first for the row sums alone.
template <int NT, bool MULTI, int NORM, int PARTS>
__global__ __launch_bounds__(512, 2) void bwd_rows_k(BwdConvArgs g, int blk) {
  const StepArgs& a = g.st;
  // [part][keys, values]: tiles of 32 rows of g (see swz)
  __shared__ __align__(16) unsigned char Gs[PARTS * 2 + (MULTI ? 1 : 0)][32 * 256];
  __shared__ __align__(16) unsigned char Xs[8][32 * 128];        // a wave's own: 32 rows of 128 bytes (see pswz)
  // Results of a row in what is idle then: a wave's own in its rows, between the products and the planes; those of all waves
  // (reference, 1 / sum, sum n G) in place of g, behind the barrier after the products, or behind g where more products come.
  // (Three parts, 80 KB: two workgroups to a compute unit with one tile a wave.)
  float* const row_s = (float*)Gs[MULTI ? PARTS * 2 : 0];
  const Block x = block_of(g, blk);
  const int tiles = (a.M + 31) / 32, item = xcd_item(blockIdx.x, gridDim.x);
  const int sb = item % tiles, ch = item / tiles, s0 = sb * 32, hkv = ch % a.Hkv;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l31 = l & 31, lh = l >> 5;
  const float* gk = grad_new(g, blk, false) + (int64_t)ch * a.M * kD;
  const float* gv = grad_new(g, blk, true) + (int64_t)ch * a.M * kD;
  const uint32_t* prot = a.protect ? a.protect + (int64_t)ch * a.protect_stride : nullptr;
  uint16_t* gsp = g.gsplit + (int64_t)blk * g.gsplit_stride;
  // the logits (row i of the tile: slot s0 + 8 (i / 4) + 4 lh + i % 4; this lane: a position) of a chunk; a position that
  // does not count has the logit -inf.  (Rows of a slot past M hold whatever follows: they end as zeros below.)
  const float* lg = g.logits + blk * g.logits_stride + ((int64_t)ch * a.M + s0) * g.ld;
  f32x16 acc[NT], xl[NT];
  auto fetch = [&](int pc, int n) {
    const int p0 = pc + (w + 8 * n) * 32;
    if (p0 < x.T) {
      const float* p = lg + (int64_t)(lh * 4) * g.ld + p0 + l31;           // (rows are padded to whole tiles)
#pragma unroll
      for (int i = 0; i < 16; ++i) xl[n][i] = p[(int64_t)((i >> 2) * 8 + (i & 3)) * g.ld];
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) xl[n][i] = -INFINITY;
    }
  };
  auto mask = [&](int pc) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int pos = pc + (w + 8 * n) * 32 + l31;
      bool out = pos >= x.T;
      if (prot && pos < x.m) out = (prot[pos >> 5] >> (pos & 31)) & 1u;
#pragma unroll
      for (int i = 0; i < 16; ++i) xl[n][i] = out ? -INFINITY : xl[n][i];
    }
  };
  // slots that mix: all live ones but the protected
  uint32_t mixing = a.M - s0 >= 32 ? 0xffffffffu : (1u << (a.M - s0)) - 1u;
  if (prot && s0 < x.m) {
    uint32_t p = prot[sb];
    if (x.m - s0 < 32) p &= (1u << (x.m - s0)) - 1u;
    if (p) {                                // a protected slot hands its gradient to the old row
      float* dk = g.d_cache_k + blk * g.d_stride + (int64_t)ch * a.M * kD;
      float* dv = g.d_cache_v + blk * g.d_stride + (int64_t)ch * a.M * kD;
      for (int e = tid; e < 32 * kD; e += 512) {
        const int64_t o = (int64_t)s0 * kD + e;
        if ((p >> (e >> 7)) & 1u & (mixing >> (e >> 7))) { dk[o] += gk[o]; dv[o] += gv[o]; }
      }
    }
    mixing &= ~p;
  }
  mixing = __builtin_amdgcn_readfirstlane(mixing);
  // Rows of [g_k | g_v] first, then the entries' rows and the logits of the first tile: loads come back in the order they are
  // asked for, and g is what the workgroup meets over.
  f32x4 gr[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {             // eight columns of a row of [g_k | g_v] per item
    const int it = tid + i * 512, r = it >> 5, c8 = it & 31;
    const float* p = (c8 >> 4 ? gv : gk) + (int64_t)min(s0 + r, a.M - 1) * kD + (c8 & 15) * 8;
    gr[i][0] = *(const f32x4_any*)p;
    gr[i][1] = *(const f32x4_any*)(p + 4);
  }
  auto entry = [&](int j, int val) {
    j = j < x.T ? j : x.T - 1;
    const uint16_t* c = (val ? x.cv : x.ck) + ((int64_t)ch * a.M + j) * kD;
    const View& st = val ? a.v : a.k;
    const uint16_t* q = (val ? x.v : x.k) + (ch / a.Hkv) * st.sb + hkv * st.sh + (int64_t)(j - x.m) * st.st;
    return j < x.m ? c : q;
  };
  // A tile's keys and values, whole rows of 128 bytes at a time (half h of row 8 i + l / 8: register 4 h + i), become operand
  // fragments on the way through the wave's own LDS; each is requested again for the next tile when it is there.
  bf16x8 fx[2][8];
  auto request_entries = [&](int p0, int val) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint16_t* row = entry(p0 + 8 * i + (l >> 3), val) + (l & 7) * 8;
      fx[val][i] = *(const bf16x8*)row;
      fx[val][4 + i] = *(const bf16x8*)(row + 64);
    }
  };
  auto request_tile0 = [&](int pc) {
    request_entries(pc + w * 32, 0);
    request_entries(pc + w * 32, 1);
    fetch(pc, 0);
  };
  unsigned char* const xs = Xs[w];
  const int by_row = (l >> 3) * 128 + (((l & 7) ^ pswz(l >> 3)) << 4);      // rows 8 i + l / 8: + 1024 i, ^ 32 where i is odd
  const int by_pos = l31 * 128 + ((lh ^ pswz(l31)) << 4);                   // chunk 2 k + l / 32 of row l % 32: ^ 32 k
  auto wave_sync = [&]() {                  // (LDS serves a wave in order: nothing to wait for)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  request_tile0(0);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int it = tid + i * 512, r = it >> 5, c8 = it & 31, val = c8 >> 4;
    float v[8] = {gr[i][0][0], gr[i][0][1], gr[i][0][2], gr[i][0][3], gr[i][1][0], gr[i][1][1], gr[i][1][2], gr[i][1][3]};
    if (s0 + r >= a.M)
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = 0.f;
    bf16x8 part[PARTS];
    split_parts<PARTS>(v, part);
    const int at = r * 256 + (((c8 & 15) ^ swz(r)) << 4);
#pragma unroll
    for (int u = 0; u < PARTS; ++u) *(bf16x8*)(Gs[u * 2 + val] + at) = part[u];
  }
  int ga[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) ga[ks] = l31 * 256 + (((2 * ks + lh) ^ swz(l31)) << 4);
  __syncthreads();
  {                                         // g for bwd_dx_k, as operand fragments: wave w the columns 32 w .. of [K | V]
    const int s16 = l & 15, g2 = (l >> 4) & 1, chunk = (w & 3) * 4 + 2 * g2 + ((s16 & 3) >> 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = h * 16 + lh * 8 + (s16 >> 2), r4 = r + 4;
      const int at = r * 256 + ((chunk ^ swz(r)) << 4) + (s16 & 1) * 8, at4 = r4 * 256 + ((chunk ^ swz(r4)) << 4) + (s16 & 1) * 8;
#pragma unroll
      for (int u = 0; u < PARTS; ++u)
        *(bf16x8*)(gsp + ((((int64_t)u * a.batch * a.Hkv + ch) * tiles * 2 + sb * 2 + h) * 8 + w) * 512 + l * 8) =
            frag_tr(Gs[u * 2 + (w >> 2)] + at, Gs[u * 2 + (w >> 2)] + at4);
    }
  }

  auto contract = [&](int pc) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int p0 = pc + (w + 8 * n) * 32;
      acc[n] = zero16();
      if (p0 >= x.T) {
        if (n + 1 < NT) fetch(pc, n + 1);
        continue;
      }
#pragma unroll
      for (int val = 0; val < 2; ++val) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int i = 0; i < 4; ++i) *(bf16x8*)(xs + i * 1024 + (by_row ^ (i & 1) << 5)) = fx[val][4 * h + i];
          if (h && n + 1 < NT) request_entries(p0 + 256, val);   // (rows past the end: the last one again)
          wave_sync();
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const bf16x8 f = *(const bf16x8*)(xs + (by_pos ^ k << 5));
#pragma unroll
            for (int u = 0; u < PARTS; ++u) acc[n] = mfma32(*(const bf16x8*)(Gs[u * 2 + val] + ga[4 * h + k]), f, acc[n]);
          }
          wave_sync();
        }
      }
      if (n + 1 < NT) fetch(pc, n + 1);
    }
  };
  // the 16 rows' values of a lane, combined over the lanes and the waves; the result of row r lands with thread r
  auto over_waves = [&](const f32x16& v, int which, auto mx) {
    const float t = over32<decltype(mx)::value>(v, l31);
    const int i = l31 >> 1;
    ((float*)xs)[which * 32 + (i >> 2) * 8 + lh * 4 + (i & 3)] = t;          // (two lanes hold the same)
  };
  auto collect = [&](int which, bool mx) {
    float t = ((const float*)Xs[0])[which * 32 + tid];
    for (int k = 1; k < 8; ++k) {
      const float o = ((const float*)Xs[k])[which * 32 + tid];
      t = mx ? fmaxf(t, o) : t + o;
    }
    return t;
  };
  f32x16 rv;
  auto rows = [&](int which) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 t = *(const f32x4*)(row_s + which * 32 + q * 8 + lh * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) rv[q * 4 + e] = t[e];
    }
  };
  // logits -> unnormalised weights, and the sums of a chunk on top of (sum, dot) of thread r < 32
  float ref = -INFINITY, sum = 0.f, dot = 0.f;
  auto weigh = [&]() {
    if (NORM == 0) {
      f32x16 mx = xl[0];
#pragma unroll
      for (int n = 1; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx[i] = fmaxf(mx[i], xl[n][i]);
      over_waves(mx, 0, Yes{});
      __syncthreads();
      if (tid < 32) {
        const float t = fmaxf(ref, collect(0, true));
        if (MULTI && ref > -INFINITY) {
          const float f = exp_neg(ref - t);
          sum *= f;
          dot *= f;
        }
        ref = t;
        // (a chunk whose positions are all protected: nothing to refer to yet, and -inf - -inf is no number)
        row_s[tid] = MULTI && t == -INFINITY ? 0.f : t;
      }
      __syncthreads();
      rows(0);
    }
    f32x16 ps = zero16(), pd = zero16();
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float e = NORM == 0 ? exp_neg(xl[n][i] - rv[i]) : fmaxf(xl[n][i], 0.f);
        xl[n][i] = e;
        ps[i] += e;
        pd[i] = fmaf(e, acc[n][i], pd[i]);
      }
    over_waves(ps, 0, No{});
    over_waves(pd, 1, No{});
    __syncthreads();
    if (tid < 32) {
      sum += collect(0, false);
      dot += collect(1, false);
    }
  };
  auto publish = [&]() {
    if (tid < 32) {
      const float inv = 1.0f / (NORM == 0 ? sum : sum + a.eps);
      row_s[32 + tid] = inv;
      row_s[64 + tid] = dot * inv;
    }
    __syncthreads();
  };
  f32x16 bsum = zero16();
  auto finish = [&](int pc) {               // xl: unnormalised weights
    f32x16 inv, r;
    rows(1); inv = rv;
    rows(2); r = rv;
    uint16_t* pn = g.wn + blk * g.plane_stride;
    uint16_t* pl = g.dl + blk * g.plane_stride;
    uint16_t* pw = g.wn_low + blk * g.plane_stride;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int p0 = pc + (w + 8 * n) * 32;
      if (p0 >= x.T) continue;
      u32x4 out[3][2][2];                   // [plane][high, low halves][slots 16 qp + 8 lh ..]
#pragma unroll
      for (int qp = 0; qp < 2; ++qp) {      // slots 16 qp .. + 15: two groups of four of this lane
        uint32_t nh[2][2], nl[2][2], n3[2][2], dh[2][2], dlo[2][2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          float vn[4], vd[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = (qp * 2 + q) * 4 + e, slot = (qp * 2 + q) * 8 + lh * 4 + e;
            const bool on = (mixing >> slot) & 1u;
            const float nn = xl[n][i] * inv[i], dG = acc[n][i] - r[i];
            const float d = NORM == 0 ? nn * dG : (xl[n][i] > 0.f ? dG * inv[i] : 0.f);
            vn[e] = on ? nn : 0.f;
            vd[e] = on ? d : 0.f;
            bsum[i] += vd[e];                // (zero where the position does not count)
          }
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            split2(vn[2 * e], vn[2 * e + 1], nh[q][e], nl[q][e]);
            if (PARTS == 3) {
              const f32x2 left = {vn[2 * e] - __uint_as_float(nh[q][e] << 16) - __uint_as_float(nl[q][e] << 16),
                                  vn[2 * e + 1] - __uint_as_float(nh[q][e] & 0xffff0000u) - __uint_as_float(nl[q][e] & 0xffff0000u)};
              n3[q][e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(left, bf16x2));
            }
          }
          split2(vd[0], vd[1], dh[q][0], dlo[q][0]);
          split2(vd[2], vd[3], dh[q][1], dlo[q][1]);
        }
        // the halves of the wave trade groups, so that a lane has eight consecutive slots: 16 qp + 8 lh ..
        auto trade = [&](const uint32_t (&v)[2][2]) {
          const auto t0 = __builtin_amdgcn_permlane32_swap(v[0][0], v[1][0], false, false);
          const auto t1 = __builtin_amdgcn_permlane32_swap(v[0][1], v[1][1], false, false);
          return u32x4{t0[0], t1[0], t0[1], t1[1]};
        };
        out[0][0][qp] = trade(nh);
        out[0][1][qp] = trade(nl);
        if (PARTS == 3) {
          out[2][0][qp] = trade(n3);
          out[2][1][qp] = out[0][0][qp];
        }
        out[1][0][qp] = trade(dh);
        out[1][1][qp] = trade(dlo);
      }
      // a plane's 32 positions through the wave's LDS, so that every store covers whole lines: eight positions, 1 KB
      // (positions T .. of the last tile: zeros, which bwd_dw_k reads)
      const int64_t o = (((int64_t)ch * tiles + sb) * g.P + p0) * 64 + l * 8;
      auto put = [&](uint16_t* at, const u32x4 (&v)[2][2]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) *(u32x4*)(xs + (by_pos ^ k << 5)) = v[k >> 1][k & 1];
        wave_sync();
        u32x4 t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = *(const u32x4*)(xs + i * 1024 + (by_row ^ (i & 1) << 5));
        wave_sync();
#pragma unroll
        for (int i = 0; i < 4; ++i) *(u32x4*)(at + o + i * 512) = t[i];
      };
      put(pn, out[0]);
      put(pl, out[1]);
      if (PARTS == 3) put(pw, out[2]);
    }
  };
  if (!MULTI) {
    contract(0);
    mask(0);
    weigh();
    publish();
    finish(0);
  } else {
    for (int pc = 0; pc < x.T; pc += 256 * NT) {
      if (pc) request_tile0(pc);
      contract(pc);
      mask(pc);
      weigh();
      __syncthreads();
    }
    publish();
    for (int pc = 0; pc < x.T; pc += 256 * NT) {
      request_tile0(pc);
      contract(pc);
      mask(pc);
      if (NORM == 0) rows(0);
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) xl[n][i] = NORM == 0 ? exp_neg(xl[n][i] - rv[i]) : fmaxf(xl[n][i], 0.f);
      finish(pc);
    }
  }
  if (g.d_conv_b) {
    __syncthreads();
    over_waves(bsum, 0, No{});
    __syncthreads();
    if (tid < 32 && ((mixing >> tid) & 1u)) atomicAdd(g.d_conv_b + hkv * a.b_head_stride + s0 + tid, collect(0, false));
  }
}

// ---- dX: a workgroup per (PT positions, NC key or value columns) of a chain and block, contraction over the slots in
// chunks of 16 KS.  A chunk is a phase with dl (one product per tap: its rows, shifted, times that tap's filters) and one
// with n (times the parts of g).  Eight waves split a chunk KS ways (16 slots each) and the columns 8 / KS ways; the partial
// sums meet in LDS at the end.  No two waves want the same filters, so these come from memory straight into the registers,
// packed in fragment order, D taps ahead: within a phase there is nothing to meet for, and only the plane rows (which the
// taps read at shifted rows) pass through LDS, by loads that write it directly, a phase or more ahead.  Rows outside the
// sequence read as zero (buffer bounds).  139 us a step of 32 chains, 512 slots and 1024 positions (155 GFLOP), 10.9 us for the
// cache rows at 128 slots (161 and 16.4 with the filters through LDS, two taps a barrier: requests, fragment reads and products
// were a chain that the two waves of a SIMD overlapped in part).  Of 145 us, before a chain's tiles shared an XCD, 131 were left
// without the filter loads and 133 without the LDS reads; the value columns' workgroups, which follow the key columns', took 20 of
// it and the sums 6.
// part 0: the cache rows of block blk0; 1: the rows of blocks blk0, blk0 + 1, .. themselves (grid.z); 2: both, of blk0.
// FINE: the blocks whose n and g enter in three parts.
template <int PT, int NC, int KS, bool FINE>
struct Dx {
  static constexpr int CW = 8 / KS, PB = PT / 32, CB = NC / 32 / CW;     // column groups; 32 x 32 output blocks of a wave
  static constexpr int PL = KS / 2, DR = PT + 32;                        // 32-slot planes of a chunk; rows with the halo
  static constexpr int DB = PL * DR * 128, NB = PL * PT * 128;           // bytes of a chunk's rows of dl, of n
  static constexpr int ND = DB / 8192, NN = NB / 8192;                   // requests of a wave for them
  // two workgroups on a compute unit, 128 registers a wave: no room for g of the next chunk, whose wait the other one fills
  static constexpr bool SHARED = PT == 64;
  static constexpr int D = 3;                                            // taps of filters in flight (a divisor of 15 and 21)
  static constexpr int RR = PB * CB >= 8 ? 64 : PB * CB >= 2 ? 32 : 16;  // registers of a wave summed up at a time
  static constexpr int rings = 2 * DB + (FINE ? 2 : 1) * NB, sums = 8 * RR * 256;
  static constexpr int lds = rings > sums ? rings : sums;
  static_assert(DB % 8192 == 0 && NB % 8192 == 0, "whole requests");
};
template <int PT, int NC, int KS, bool FINE>
__global__ __launch_bounds__(512, NC == 64 || PT == 64 ? 4 : 2) void bwd_dx_k(BwdConvArgs g, int blk0, int part) {
  extern __shared__ __align__(16) unsigned char smem[];
  using G = Dx<PT, NC, KS, FINE>;
  constexpr int PB = G::PB, CB = G::CB, D = G::D, GP = FINE ? 3 : 2;
  const StepArgs& a = g.st;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)smem);
  constexpr int ZC = 256 / NC;
  // the tiles of a chain on one XCD: they read the same g, and their halos overlap (the cache rows of a step, 32 chains of 256
  // slots, 32-row tiles, three parts: 44.1 -> 34.9 us; 128 slots, two parts: 11.6 -> 10.9; 512 slots, 128-row tiles: 141 -> 139)
  const int item = xcd_item(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int blk = blk0 + blockIdx.z / ZC, val = blockIdx.z % ZC * NC / kD, cbase = blockIdx.z % ZC * NC % kD, ch = item / gridDim.x, hkv = ch % a.Hkv;
  const Block x = block_of(g, blk);
  const int p0 = (part == 1 ? x.m : 0) + item % gridDim.x * PT, pend = part == 0 ? x.m : x.T;
  if (p0 >= pend) return;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l31 = l & 31, lh = l >> 5;
  const int kq = w % KS, wo = w / KS;
  const int KW = a.k_width, pad = (KW - 1) / 2, C = a.conv_in ? 2 * kD : kD, tiles = (a.M + 31) / 32;
  const bool taps = val == 0 || a.conv_in;
  const int n16 = (a.M + 15) / 16, nsc = (n16 + KS - 1) / KS;

  // right-hand fragments, 1 KB each: the filters [bank][32 channels][16 slots][tap], and g [part][chain][16 slots][32 columns].
  // (16 slots past M: the last ones again, their partners in the planes are zero)
  const uint32_t lane16 = l * 16;
  const unsigned char* wf = (const unsigned char*)g.wf +
      (int64_t)((a.w_head_stride ? hkv * (C / 32) : 0) + ((val ? kD : 0) + cbase) / 32 + wo * CB) * n16 * KW * 1024;
  const unsigned char* gf = (const unsigned char*)(g.gsplit + blk * g.gsplit_stride) +
      ((int64_t)ch * tiles * 16 + (val * kD + cbase) / 32 + wo * CB) * 1024;
  const int64_t gpart = (int64_t)a.batch * a.Hkv * tiles * (16 * 1024);
  bf16x8 fw[D][CB];
  auto tap0 = [&](int sc) { return wf + (int64_t)min(min(sc, nsc - 1) * KS + kq, n16 - 1) * KW * 1024; };   // of this wave's 16 slots
  auto load_tap = [&](bf16x8 (&f)[CB], const unsigned char* p) {
#pragma unroll
    for (int c = 0; c < CB; ++c) f[c] = *(const bf16x8*)(p + (int64_t)c * n16 * KW * 1024 + lane16);
  };
  const bool whole = KW % D == 0;            // the taps of a chunk end where those of the next one begin
  auto first_taps = [&](int sc) {
#pragma unroll
    for (int i = 0; i < D; ++i) load_tap(fw[i], tap0(sc) + min(i, KW - 1) * 1024);
  };

  // plane rows: offsets inside the 32-slot planes of a chunk, of dl (with the halo) and of n.  SHARED works them out again for
  // every request: its 128 registers hold no more than sums and fragments, and a reload from scratch memory waits for the request
  // before it and for the filters on their way.
  uint32_t dvo[G::ND], nvo[G::NN];
  auto plane_cell = [&](int ra, int rows, int first) -> uint32_t {
    int l = tid & 63;
    if (G::SHARED) asm volatile("" : "+v"(l));
    const int pl = ra / rows, r = ra - pl * rows + (l >> 3), q = first + r;
    return q >= 0 && q < x.T ? (uint32_t)((pl * g.P + q) * 128 + (((l & 7) ^ pswz(r)) << 4)) : 0x80000000u;
  };
  auto d_cell = [&](int i) { return plane_cell((w * G::ND + i) * 8, G::DR, p0 - (KW - 1) + pad); };
  auto n_cell = [&](int i) { return plane_cell((w * G::NN + i) * 8, PT, p0); };
  if (!G::SHARED) {
#pragma unroll
    for (int i = 0; i < G::ND; ++i) dvo[i] = d_cell(i);
#pragma unroll
    for (int i = 0; i < G::NN; ++i) nvo[i] = n_cell(i);
  }
  const int64_t chain_planes = (int64_t)ch * tiles * g.P * 128;
  const unsigned char* pl = (const unsigned char*)(g.dl + blk * g.plane_stride) + chain_planes;
  const unsigned char* pn = (const unsigned char*)(g.wn + blk * g.plane_stride) + chain_planes;
  const unsigned char* pw = (const unsigned char*)(g.wn_low + blk * g.plane_stride) + chain_planes;
  auto planes_rsrc = [&](const unsigned char* p, int sc) {
    return make_rsrc(p + (int64_t)sc * G::PL * g.P * 128, (uint32_t)(min(G::PL, tiles - sc * G::PL) * g.P * 128));
  };
  const uint32_t ddst = __builtin_amdgcn_readfirstlane(lds0 + w * G::ND * 1024), ndst = __builtin_amdgcn_readfirstlane(lds0 + w * G::NN * 1024);
  auto request_d = [&](int sc) {
    const u32x4 r = planes_rsrc(pl, sc);
#pragma unroll
    for (int i = 0; i < G::ND; ++i) load_to_lds_at(r, ddst + (sc & 1) * G::DB + i * 1024, G::SHARED ? d_cell(i) : dvo[i], 0u);
  };
  // the rows of n have one place behind the two of dl; without taps they take turns in those
  const bool turns = !taps && !FINE;
  auto n_at = [&](int sc) { return turns ? (sc & 1) * G::DB : 2 * G::DB; };
  auto request_n = [&](int sc) {
    const u32x4 r = planes_rsrc(pn, sc);
#pragma unroll
    for (int i = 0; i < G::NN; ++i) load_to_lds_at(r, ndst + n_at(sc) + i * 1024, G::SHARED ? n_cell(i) : nvo[i], 0u);
    if (FINE) {
      const u32x4 r3 = planes_rsrc(pw, sc);
#pragma unroll
      for (int i = 0; i < G::NN; ++i) load_to_lds_at(r3, ndst + n_at(sc) + G::NB + i * 1024, G::SHARED ? n_cell(i) : nvo[i], 0u);
    }
  };
  f32x16 acc[PB][CB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[pb][cb] = zero16();
  auto multiply = [&](const bf16x8 (&fd)[PB], const bf16x8 (&fr)[CB]) {
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[pb][cb] = mfma32(fd[pb], fr[cb], acc[pb][cb]);
  };
  const int dchunk = (kq & 1) * 2 + lh;
  // high or low halves of this wave's slots in 32 PB rows from row r on
  auto rows_at = [&](const unsigned char* p, int r, int low, bf16x8 (&f)[PB]) {
    p += r * 128 + (((dchunk ^ pswz(r)) << 4) ^ low * 64);
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) f[pb] = *(const bf16x8*)(p + pb * 32 * 128);
  };

  if (taps) {
    request_d(0);
    first_taps(0);
    if (nsc > 1) request_d(1);
  }
  request_n(0);
  if (turns && nsc > 1) request_n(1);
  wait_loads<0>();
  barrier();
  bf16x8 fg[GP][CB];
  auto load_part = [&](int sc, int u, bf16x8 (&f)[CB]) {
    const unsigned char* p = gf + (int64_t)min(min(sc, nsc - 1) * KS + kq, n16 - 1) * (8 * 1024) + u * gpart;
#pragma unroll
    for (int c = 0; c < CB; ++c) f[c] = *(const bf16x8*)(p + c * 1024 + lane16);
  };
  auto load_g = [&](int sc, bf16x8 (&f)[GP][CB]) {
#pragma unroll
    for (int u = 0; u < GP; ++u) load_part(sc, u, f[u]);
  };
  if (!G::SHARED) load_g(0, fg);
  for (int sc = 0; sc < nsc; ++sc) {
    if (taps) {
      const unsigned char* dp = smem + (sc & 1) * G::DB + (kq >> 1) * G::DR * 128;
      int l31 = tid & 31;
      if (G::SHARED) asm volatile("" : "+v"(l31));     // (nor are the walk's first rows kept)
      // a tap's low halves are read ahead of the products with the high ones, the next tap's high ones ahead of those with the
      // low ones; its filters are replaced by those D taps on, which at the end of a chunk are the next one's first
      bf16x8 fh[PB], fl[PB];
      auto tap = [&](int t, bf16x8 (&f)[CB]) {
        rows_at(dp, l31 + KW - 1 - t, 1, fl);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fh, f);
        __builtin_amdgcn_sched_barrier(0);
        rows_at(dp, l31 + max(KW - 2 - t, 0), 0, fh);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fl, f);
        __builtin_amdgcn_sched_barrier(0);
      };
      rows_at(dp, l31 + KW - 1, 0, fh);
      const unsigned char* here = tap0(sc);
      const unsigned char* there = whole ? tap0(sc + 1) : here;
      int t0 = 0;
      for (; t0 + D <= KW; t0 += D)
#pragma unroll
        for (int i = 0; i < D; ++i) {
          tap(t0 + i, fw[i]);
          const int t = t0 + i + D;
          load_tap(fw[i], t < KW ? here + t * 1024 : there + (t - KW) * 1024);
        }
#pragma unroll
      for (int i = 0; i < D - 1; ++i)
        if (t0 + i < KW) tap(t0 + i, fw[i]);
      wait_loads<0>();
      barrier();
      if (sc + 2 < nsc) request_d(sc + 2);
      if (!whole && sc + 1 < nsc) first_taps(sc + 1);
    }
    {
      const unsigned char* np = smem + n_at(sc) + (kq >> 1) * PT * 128;
      bf16x8 fh[PB], fl[PB], next[GP][CB];
      if (G::SHARED) {
        load_part(sc, 1, fg[1]);
        load_part(sc, 0, fg[0]);
      } else {
        load_g(sc + 1, next);
      }
      rows_at(np, l31, 0, fh);
      rows_at(np, l31, 1, fl);
      multiply(fh, fg[1]);
      // (low half x low half is below the 16 bits kept of two parts, not below the 24 of three)
      if constexpr (FINE) {
        multiply(fl, fg[1]);
        if (G::SHARED) {                       // the third part in the place of the second
          __builtin_amdgcn_sched_barrier(0);
          load_part(sc, 2, fg[2]);
        }
      }
      multiply(fh, fg[0]);
      multiply(fl, fg[0]);
      if constexpr (FINE) {
        rows_at(np + G::NB, l31, 0, fl);       // the third part, [third | first]
        multiply(fl, fg[0]);
        multiply(fh, fg[2]);
      }
      if (!G::SHARED)
#pragma unroll
        for (int u = 0; u < GP; ++u)
#pragma unroll
          for (int c = 0; c < CB; ++c) fg[u][c] = next[u][c];
    }
    if (sc + 1 == nsc) break;
    if (turns) wait_loads<0>();
    barrier();
    if (!turns) request_n(sc + 1);
    else if (sc + 2 < nsc) request_n(sc + 2);
    if (!taps && !turns) {
      wait_loads<0>();
      barrier();
    }
  }
  // ---- the KS partial sums of each output, RR registers of every wave at a time: a wave adds up RR / KS of them
  constexpr int RR = G::RR, X = RR / KS;
  float* red = (float*)smem + wo * KS * RR * 64 + l;
#pragma unroll
  for (int rd = 0; rd < PB * CB * 16 / RR; ++rd) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RR; ++q) red[(kq * RR + q) * 64] = acc[(rd * RR + q) / 16 / CB][(rd * RR + q) / 16 % CB][q % 16];
    const int b = (rd * RR + kq * X) / 16, i0 = kq * X % 16;      // what this wave adds up: registers i0 .. of block b
    float* at[X];
    float old[X];
#pragma unroll
    for (int i = 0; i < X; ++i) {          // every load before the first store
      const int p = min(p0 + b / CB * 32 + ((i0 + i) >> 2) * 8 + lh * 4 + (i & 3), pend - 1);
      float* cr = (val ? g.d_cache_v : g.d_cache_k) + blk * g.d_stride + ((int64_t)ch * a.M + p) * kD;
      float* br = (val ? g.d_v : g.d_k) + ch * g.kv_chain + ((int64_t)blk * g.B + p - x.m) * kD;
      at[i] = (p < x.m ? cr : br) + cbase + (wo * CB + b % CB) * 32 + l31;
      old[i] = *at[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < X; ++i) {
      float v = 0.f;
#pragma unroll
      for (int k = 0; k < KS; ++k) v += red[(k * RR + kq * X + i) * 64];
      if (p0 + b / CB * 32 + ((i0 + i) >> 2) * 8 + lh * 4 + (i & 3) < pend) *at[i] = old[i] + v;
    }
  }
}

// ---- The walk over a run of blocks in one launch: what bwd_rows_k and bwd_dx_k over the cache rows do block by block.  A step is
// bound by the chain of latencies from one block's g to the next one's, for 3 us of matrix work at the chip's rate on 32 chains of 128
// slots and 256 positions: two launches a block 23.6 us, some 4 of either the launch, here 20.6 (256 slots, 512 positions, 16 chains:
// 34.4 and 30).  Four workgroups to 64 slots of a chain stay for all blocks.  Each has one tile of 32 slots, whose rows it takes
// in turn with another, every second block; and 64 cache rows by 32 key and 32 value columns of dX of every block.  What does not
// wait for g is out of the way before it arrives: the normalised rows and their planes (made by the one workgroup while the other is at
// work on the block before), the entries' first rows, the first filters.  The workgroups of a chain meet twice a block, over dl (all of
// its tiles) and over the next g (the four of 64 rows), on counters and by rules that are those of the forward scan (compress_tile.inl):
// through the L2 where they share one, with device-scope release and acquire where not; waits are bounded.  Planes and fragments of g
// have places of their own in every block, so no compute unit can have read them before they were written; g itself it can, as what
// its sums were added to, so that is read past its L1.
// Clock stamps of the former (49 000 cycles a step): 4 000 from g to its halves in LDS, 2 400 G, 1 200 row sums, 3 800 dl, 4 700 until it
// is known to have arrived, 3 000 to have it back, 9 500 taps and n g (4 600 of matrix work, the rest the forty instructions around a
// tap's four products), 6 000 partial sums.  (143 to 168 scalar values of a build lie in lanes of vector registers; none of the
// vector registers is in scratch memory.)
struct WalkArgs {
  BwdConvArgs c;
  int32_t hi, n;             // blocks hi, hi - 1, .. hi - n + 1
  uint32_t* sync;            // per chain
  uint32_t* tsync;           // per (chain, tile): two words, the count of a tile's halves; the second of a chain's first: XCD mask
  int32_t* status;
  int32_t spin_limit, same_l2_allowed;
};
// loads of what other workgroups have written since this one began: from the L2, never from this compute unit's L1
__device__ __forceinline__ f32x4 load_f4_shared(const void* base, uint32_t bytes, uint32_t off) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 1 << 4));
}
// 32-slot tiles whose rows of dl and n are in LDS at once: all of them in as few rounds as there is room for
template <int PARTS>
__host__ __device__ inline int walk_round(int tiles) {
  constexpr int most = PARTS == 3 ? 5 : 8;
  const int rounds = (tiles + most - 1) / most;
  return (tiles + rounds - 1) / rounds;
}
__host__ __device__ inline int walk_rows(int KW) { return (64 + KW - 1 + 7) / 8 * 8; }
template <int PARTS>
int walk_lds(int tiles, int KW) {
  const int rows = PARTS * 2 * 8192 + 8 * 4096, dx = walk_round<PARTS>(tiles) * (walk_rows(KW) * 128 + 8192 * (PARTS - 1)), sums = 8 * 64 * 256;
  return std::max(rows, std::max(dx, sums));
}

// NT: 32-position tiles a wave holds of a row; PARTS: of n and g (see above)
template <int NT, int PARTS>
__global__ __launch_bounds__(512, 2) void bwd_walk_k(WalkArgs wa) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ __align__(16) float row_s[3 * 32];                  // of a row: reference, 1 / sum, sum n G
  __shared__ int bail, same_l2;
  const BwdConvArgs& g = wa.c;
  const StepArgs& a = g.st;
  unsigned char* const Gs = smem;                                // [part][keys, values]: tiles of 32 rows of g (see swz)
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int l = tid & 63, l31 = l & 31, lh = l >> 5;
  // addresses belong to a phase of a step: hoisted out of the walk, they spill
  auto phase = [&]() { asm volatile("" : "+v"(l), "+v"(l31), "+v"(lh)); };
  unsigned char* const Xs0 = smem + PARTS * 2 * 8192;            // a wave's own 4 KB each: 32 rows of 128 bytes (see pswz)
  unsigned char* const xs = Xs0 + w * 4096;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)smem);
  const int tiles = a.M / 32, mine = (tiles + 1) / 2 * 4, item = xcd_item(blockIdx.x, gridDim.x);
  const int ch = item / mine, r2 = item % mine >> 2, cg = item & 3, tile = r2 * 2 + (cg & 1), half = cg >> 1, s0 = tile * 32, hkv = ch % a.Hkv;
  const int KW = a.k_width, pad = (KW - 1) / 2, n16 = tiles * 2, DR = walk_rows(KW);

  // ---- meeting points
  if (tid == 0) { bail = 0; same_l2 = 0; }
  __syncthreads();
  auto signal = [&](uint32_t* c) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      if (same_l2) __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  auto await = [&](const uint32_t* c, uint32_t target) -> bool {
    if (tid == 0) {
      int polls = 0;
      while (__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        __builtin_amdgcn_s_sleep(1);
        if (++polls > wa.spin_limit) {       // bounded: never spin forever on a workgroup that is not there
          __hip_atomic_store(wa.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          bail = 1;
          break;
        }
      }
      if (!same_l2) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    return bail == 0;
  };
  uint32_t* const chain_count = wa.sync + ch;
  uint32_t* const rows_count = wa.tsync + 2 * (ch * tiles + r2);
  {                                          // the first meeting is a census of the XCDs a chain's workgroups run on
    uint32_t* const mask = wa.tsync + 2 * ch * tiles + 1;
    if (tid == 0) {
      const uint32_t xcd = __builtin_amdgcn_s_getreg(20 | ((4 - 1) << 11));   // XCC_ID, bits [3:0]
      __hip_atomic_fetch_or(mask, 1u << xcd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    signal(chain_count);
    if (!await(chain_count, (uint32_t)mine)) return;
    if (tid == 0) {
      const uint32_t seen = __hip_atomic_load(mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      same_l2 = wa.same_l2_allowed && (seen & (seen - 1)) == 0;
    }
    __syncthreads();
  }

  // ---- rows: this workgroup's 32 slots, all positions; wave w has the position tiles w, w + 8, ..  (see bwd_rows_k)
  auto wave_sync = [&]() {                   // (LDS serves a wave in order: nothing to wait for)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto by_row = [&]() { return (l >> 3) * 128 + (((l & 7) ^ pswz(l >> 3)) << 4); };   // rows 8 i + l / 8: + 1024 i, ^ 32 where i is odd
  auto by_pos = [&]() { return l31 * 128 + ((lh ^ pswz(l31)) << 4); };                // chunk 2 k + l / 32 of row l % 32: ^ 32 k
  auto over_waves = [&](const f32x16& v, auto mx) {
    const float t = over32<decltype(mx)::value>(v, l31);
    const int i = l31 >> 1;
    ((float*)xs)[(i >> 2) * 8 + lh * 4 + (i & 3)] = t;           // (two lanes hold the same)
  };
  auto collect = [&](bool mx) {
    float t = ((const float*)Xs0)[tid];
    for (int k = 1; k < 8; ++k) {
      const float o = ((const float*)(Xs0 + k * 4096))[tid];
      t = mx ? fmaxf(t, o) : t + o;
    }
    return t;
  };
  auto rows = [&](int which) {
    f32x16 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 t = *(const f32x4*)(row_s + which * 32 + q * 8 + lh * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) r[q * 4 + e] = t[e];
    }
    return r;
  };
  // 32 slots x 32 positions of a lane's values -> rows of a plane [position][32 high | 32 low halves], through the wave's LDS, whole
  // lines a store; `third`: what the two halves leave over, with the high ones beside it, into a plane of its own
  auto planes = [&](const f32x16& v, uint16_t* at, uint16_t* third) {
    u32x4 out[2][2], out3[2];
#pragma unroll
    for (int qp = 0; qp < 2; ++qp) {         // slots 16 qp .. + 15: two groups of four of this lane
      uint32_t hi[2][2], lo[2][2], th[2][2];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float x0 = v[(qp * 2 + q) * 4 + 2 * e], x1 = v[(qp * 2 + q) * 4 + 2 * e + 1];
          split2(x0, x1, hi[q][e], lo[q][e]);
          if (third) {
            const f32x2 left = {x0 - __uint_as_float(hi[q][e] << 16) - __uint_as_float(lo[q][e] << 16),
                                x1 - __uint_as_float(hi[q][e] & 0xffff0000u) - __uint_as_float(lo[q][e] & 0xffff0000u)};
            th[q][e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(left, bf16x2));
          }
        }
      // the halves of the wave trade groups, so that a lane has eight consecutive slots: 16 qp + 8 lh ..
      auto trade = [&](const uint32_t (&p)[2][2]) {
        const auto t0 = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
        const auto t1 = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
        return u32x4{t0[0], t1[0], t0[1], t1[1]};
      };
      out[0][qp] = trade(hi);
      out[1][qp] = trade(lo);
      if (third) out3[qp] = trade(th);
    }
    const int br = by_row(), bp = by_pos();
    auto put = [&](uint16_t* to, const u32x4 (&x)[2], const u32x4 (&y)[2]) {
#pragma unroll
      for (int k = 0; k < 4; ++k) *(u32x4*)(xs + (bp ^ k << 5)) = k < 2 ? x[k & 1] : y[k & 1];
      wave_sync();
      u32x4 t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = *(const u32x4*)(xs + i * 1024 + (br ^ (i & 1) << 5));
      wave_sync();
#pragma unroll
      for (int i = 0; i < 4; ++i) *(u32x4*)(to + l * 8 + i * 512) = t[i];
    };
    put(at, out[0], out[1]);
    if (third) put(third, out3, out[0]);
  };
  const int64_t plane0 = ((int64_t)ch * tiles + tile) * g.P * 64;
  f32x16 xn[NT];                             // the normalised rows of the block this workgroup's rows are next
  // What does not wait for g: the normalised rows of block blk and their planes.
  auto prepare = [&](int blk) {
    phase();
    const Block x = block_of(g, blk);
    const float* lg = g.logits + blk * g.logits_stride + ((int64_t)ch * a.M + s0) * g.ld + (int64_t)(lh * 4) * g.ld + l31;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int p0 = (w + 8 * n) * 32;
      if (p0 < x.T) {
#pragma unroll
        for (int i = 0; i < 16; ++i) xn[n][i] = lg[(int64_t)((i >> 2) * 8 + (i & 3)) * g.ld + p0];
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) xn[n][i] = -INFINITY;
      }
    }
    f32x16 mx;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const bool out = (w + 8 * n) * 32 + l31 >= x.T;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        xn[n][i] = out ? -INFINITY : xn[n][i];
        mx[i] = n ? fmaxf(mx[i], xn[n][i]) : xn[n][i];
      }
    }
    over_waves(mx, Yes{});
    barrier();
    if (tid < 32) row_s[tid] = collect(true);
    barrier();
    {
      const f32x16 ref = rows(0);
      f32x16 ps = zero16();
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          xn[n][i] = exp_neg(xn[n][i] - ref[i]);
          ps[i] += xn[n][i];
        }
      over_waves(ps, No{});
    }
    barrier();
    if (tid < 32) row_s[32 + tid] = 1.0f / collect(false);
    barrier();
    const f32x16 inv = rows(1);
    uint16_t* pn = g.wn + blk * g.plane_stride + plane0;
    uint16_t* pw = PARTS == 3 ? g.wn_low + blk * g.plane_stride + plane0 : nullptr;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
#pragma unroll
      for (int i = 0; i < 16; ++i) xn[n][i] *= inv[i];
      const int p0 = (w + 8 * n) * 32;
      if (p0 < x.T) planes(xn[n], pn + (int64_t)p0 * 64, PARTS == 3 ? pw + (int64_t)p0 * 64 : nullptr);
    }
  };

  // The entries' rows of a wave's first tile in block blk are asked for ahead, under the wait for g, the others a tile ahead.  (A row's
  // offset in the cache or in the block: 32 bits.)
  bf16x8 fx[2][8];
  auto request_entries = [&](const Block& x, int p0, int val) {
    const unsigned char* cache = (const unsigned char*)((val ? x.cv : x.ck) + (int64_t)ch * a.M * kD);
    const View& st = val ? a.v : a.k;
    const unsigned char* block = (const unsigned char*)((val ? x.v : x.k) + (ch / a.Hkv) * st.sb + hkv * st.sh);
    const uint32_t stride = (uint32_t)st.st * 2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = min(p0 + 8 * i + (l >> 3), x.T - 1);
      const unsigned char* row = (j < x.m ? cache : block) + ((j < x.m ? j * 256u : (uint32_t)(j - x.m) * stride) + (l & 7) * 16);
      fx[val][i] = *(const bf16x8*)row;
      fx[val][4 + i] = *(const bf16x8*)(row + 128);
    }
  };
  auto request_first = [&](int blk) {
    if (blk < 0) {                           // (none: nothing of them is kept from here on)
#pragma unroll
      for (int i = 0; i < 8; ++i) fx[0][i] = fx[1][i] = bf16x8{};
      return;
    }
    phase();
    const Block x = block_of(g, blk);
    request_entries(x, w * 32, 0);
    request_entries(x, w * 32, 1);
  };

  // G, its row sums and dl of block blk; target: of the count of this tile's halves (0: g is there)
  auto differentiate = [&](int blk, uint32_t target) -> bool {
    phase();
    const Block x = block_of(g, blk);
    {                                        // the first tile's entries have come: through the wave's LDS into operand order
      const int br = by_row(), bp = by_pos();
#pragma unroll
      for (int val = 0; val < 2; ++val)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int i = 0; i < 4; ++i) *(bf16x8*)(xs + i * 1024 + (br ^ (i & 1) << 5)) = fx[val][4 * h + i];
          wave_sync();
#pragma unroll
          for (int q = 0; q < 4; ++q) fx[val][4 * h + q] = *(const bf16x8*)(xs + (bp ^ q << 5));
          wave_sync();
        }
    }
    if (target && !await(rows_count, target)) return false;
    const int by_chunk = tid >> 4, c8 = tid & 15;                // eight columns of a row of g_k, and of g_v
    {
      f32x4 gr[2][2];
#pragma unroll
      for (int val = 0; val < 2; ++val)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          gr[val][h] = load_f4_shared(grad_new(g, blk, val) + (int64_t)ch * a.M * kD, (uint32_t)a.M * kD * 4,
                                      (uint32_t)((s0 + by_chunk) * kD + c8 * 8 + h * 4) * 4);
#pragma unroll
      for (int val = 0; val < 2; ++val) {
        const float v[8] = {gr[val][0][0], gr[val][0][1], gr[val][0][2], gr[val][0][3], gr[val][1][0], gr[val][1][1], gr[val][1][2], gr[val][1][3]};
        bf16x8 part[PARTS];
        split_parts<PARTS>(v, part);
#pragma unroll
        for (int u = 0; u < PARTS; ++u) *(bf16x8*)(Gs + (u * 2 + val) * 8192 + by_chunk * 256 + ((c8 ^ swz(by_chunk)) << 4)) = part[u];
      }
    }
    barrier();
    {                                        // g for cache_rows, as operand fragments: wave w the columns 32 w .. of [K | V]
      uint16_t* gsp = g.gsplit + (int64_t)blk * g.gsplit_stride;
      const int s16 = l & 15, g2 = (l >> 4) & 1, chunk = (w & 3) * 4 + 2 * g2 + ((s16 & 3) >> 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = h * 16 + lh * 8 + (s16 >> 2), r4 = r + 4;
        const int at = r * 256 + ((chunk ^ swz(r)) << 4) + (s16 & 1) * 8, at4 = r4 * 256 + ((chunk ^ swz(r4)) << 4) + (s16 & 1) * 8;
#pragma unroll
        for (int u = 0; u < PARTS; ++u) {
          const unsigned char* p = Gs + (u * 2 + (w >> 2)) * 8192;
          *(bf16x8*)(gsp + ((((int64_t)u * a.batch * a.Hkv + ch) * n16 + tile * 2 + h) * 8 + w) * 512 + l * 8) = frag_tr(p + at, p + at4);
        }
      }
    }
    f32x16 acc[NT];
    {
      const int br = by_row(), bp = by_pos();
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const int p0 = (w + 8 * n) * 32;
        acc[n] = zero16();
        if (p0 >= x.T) continue;
#pragma unroll
        for (int val = 0; val < 2; ++val)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            if (n) {
#pragma unroll
              for (int i = 0; i < 4; ++i) *(bf16x8*)(xs + i * 1024 + (br ^ (i & 1) << 5)) = fx[val][4 * h + i];
              if (h && n + 1 < NT) request_entries(x, p0 + 256, val);    // (rows past the end: the last one again)
              wave_sync();
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const bf16x8 f = n ? *(const bf16x8*)(xs + (bp ^ q << 5)) : fx[val][4 * h + q];
              const int at = l31 * 256 + (((2 * (4 * h + q) + lh) ^ swz(l31)) << 4);
#pragma unroll
              for (int u = 0; u < PARTS; ++u) acc[n] = mfma32(*(const bf16x8*)(Gs + (u * 2 + val) * 8192 + at), f, acc[n]);
            }
            if (n) wave_sync();
            else if (h && NT > 1) request_entries(x, p0 + 256, val);
          }
      }
    }
    {
      f32x16 pd = zero16();
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) pd[i] = fmaf(xn[n][i], acc[n][i], pd[i]);
      over_waves(pd, No{});
    }
    barrier();
    if (tid < 32) row_s[64 + tid] = collect(false);
    barrier();
    const f32x16 r = rows(2);
    uint16_t* pl = g.dl + blk * g.plane_stride + plane0;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int p0 = (w + 8 * n) * 32;
      if (p0 >= x.T) continue;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[n][i] = xn[n][i] * (acc[n][i] - r[i]);
      planes(acc[n], pl + (int64_t)p0 * 64, nullptr);
    }
    return true;
  };

  // ---- dX over 64 rows of the cache, 32 key and 32 value columns: the contraction over (slot, tap) shared out evenly among the
  // waves, that with n over the slots; partial sums meet in LDS.  Filters come straight into registers, a few taps ahead, rows of
  // dl and n through LDS (see bwd_dx_k).  (32 rows and 64 columns each: twice the filters for the same products.)
  constexpr int D = 6;                       // taps of filters in flight (even)
  const int ct = walk_round<PARTS>(tiles), dl_bytes = ct * DR * 128, p0 = r2 * 64, units = n16 * KW;
  const unsigned char* const f0 = (const unsigned char*)g.wf + ((int64_t)(a.w_head_stride ? hkv * 4 : 0) + cg) * units * 1024;
  bf16x8 fw[D];
  float old[2][4];
  const int prow = p0 + w * 8;               // what this lane adds up: rows prow + 4 lh .. + 3 of column 32 cg + l31
  auto load_unit = [&](int u, bf16x8& f) { f = *(const bf16x8*)(f0 + (int64_t)min(u, units - 1) * 1024 + l * 16); };
  auto sums_of = [&](int blk, int val) { return (val ? g.d_cache_v : g.d_cache_k) + blk * g.d_stride + (int64_t)ch * a.M * kD + cg * 32; };
  // what does not wait for the chain: the first filters, and what the sums are added to
  auto look_ahead = [&](int blk) {
    phase();
    const int m = max(blk ? a.M : a.m, 1);
#pragma unroll
    for (int i = 0; i < D; ++i) load_unit(ct * 2 * KW * w / 8 + i, fw[i]);
#pragma unroll
    for (int val = 0; val < 2; ++val)
#pragma unroll
      for (int i = 0; i < 4; ++i) old[val][i] = sums_of(blk, val)[min(prow + lh * 4 + i, m - 1) * kD + l31];
  };
  auto cache_rows = [&](int blk, int next, uint32_t target) -> bool {
    const Block x = block_of(g, blk);
    if (!await(chain_count, target)) return false;
    if (p0 >= x.m) {
      request_first(next);
      return true;
    }
    phase();
    f32x16 acc[2][2];                        // [keys, values][32 rows]
#pragma unroll
    for (int val = 0; val < 2; ++val) acc[val][0] = acc[val][1] = zero16();
    const int64_t chain_planes = (int64_t)ch * tiles * g.P * 128;
    for (int c = 0; c * ct < tiles; ++c) {
      const int here = min(ct, tiles - c * ct), s_first = c * ct * 2, groups = here * 2;
      const int64_t off = chain_planes + (int64_t)c * ct * g.P * 128;
      if (c) __syncthreads();                // the rows of the tiles before are read
      // rows of a plane, eight a request; those outside 0 .. T - 1 lie outside the buffer and read as zero
      const int lr = l >> 3;
      const uint32_t cell0 = (uint32_t)(lr * 128 + (((l & 7) ^ pswz(lr)) << 4));       // (rows 8 i + lr: i even; odd: ^ 32)
      auto request_rows = [&](const uint16_t* planes, int pl, int first, int i, int at) {
        const u32x4 r = make_rsrc((const unsigned char*)(planes + blk * g.plane_stride) + off + (int64_t)pl * g.P * 128, (uint32_t)x.T * 128);
        load_to_lds(r, lds0 + (uint32_t)(at + i * 1024), (cell0 ^ (uint32_t)(i & 1) << 5) + (uint32_t)((first + i * 8) * 128));
      };
      // dl first; n and g, which the products with the taps do not need, come under these
      const int per = DR / 8;
      for (int i = w, pl = 0; i < here * per; i += 8) {
        while (i >= (pl + 1) * per) ++pl;
        request_rows(g.dl, pl, p0 - (KW - 1) + pad, i - pl * per, pl * DR * 128);
      }
      wait_loads<0>();
      barrier();
      for (int pl = 0; pl < here; ++pl) {
        request_rows(g.wn, pl, p0, w, dl_bytes + pl * 8192);
        if (PARTS == 3) request_rows(g.wn_low, pl, p0, w, dl_bytes + (ct + pl) * 8192);
      }
      bf16x8 fg[PARTS][2];
      auto load_g = [&](int s) {
#pragma unroll
        for (int u = 0; u < PARTS; ++u)
#pragma unroll
          for (int val = 0; val < 2; ++val)
            fg[u][val] = *(const bf16x8*)(g.gsplit + (int64_t)blk * g.gsplit_stride +
                                          ((((int64_t)u * a.batch * a.Hkv + ch) * n16 + s) * 8 + val * 4 + cg) * 512 + l * 8);
      };
      load_g(s_first + min(w, groups - 1));
      // dl, this wave's share of the (slots, tap)
      phase();
      const int all = groups * KW, u0 = all * w / 8, u1 = all * (w + 1) / 8, base = s_first * KW;
      int s = u0 / KW, t = u0 - s * KW;
      bf16x8 fd[2][2][2];                    // [this unit, the next][high, low halves][32 rows]
      auto rows_of = [&](int s, int t, bf16x8 (&f)[2][2]) {
        const int r = l31 + KW - 1 - t, cell = (((s & 1) * 2 + lh) ^ pswz(r)) << 4;
        const unsigned char* q = smem + ((s >> 1) * DR + r) * 128;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          f[0][rb] = *(const bf16x8*)(q + rb * 4096 + cell);
          f[1][rb] = *(const bf16x8*)(q + rb * 4096 + (cell ^ 64));
        }
      };
      rows_of(s, t, fd[0]);
      auto unit = [&](int i) {
        if (++t == KW) { t = 0; ++s; }
        rows_of(min(s, groups - 1), t, fd[(i + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int rb = 0; rb < 2; ++rb) acc[0][rb] = mfma32(fd[i & 1][h][rb], fw[i], acc[0][rb]);
        __builtin_amdgcn_sched_barrier(0);
      };
      int u = u0;
      for (; u + D < u1; u += D)
#pragma unroll
        for (int i = 0; i < D; ++i) {
          unit(i);
          load_unit(base + u + i + D, fw[i]);
        }
#pragma unroll
      for (int i = 0; i < D; ++i)            // (nothing more is asked for: what is on its way keeps its registers)
        if (u + i < u1) unit(i);
      // n g of slots 16 (s_first + gi) ..
      auto mix = [&](int gi) {
        const unsigned char* np = smem + dl_bytes + (gi >> 1) * 8192 + l31 * 128;
        const int cell = (((gi & 1) * 2 + lh) ^ pswz(l31)) << 4;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb, np += 4096) {
          const bf16x8 fh = *(const bf16x8*)(np + cell), fl = *(const bf16x8*)(np + (cell ^ 64));
          auto multiply = [&](const bf16x8& f, const bf16x8 (&v)[2]) {
#pragma unroll
            for (int val = 0; val < 2; ++val) acc[val][rb] = mfma32(f, v[val], acc[val][rb]);
          };
          multiply(fh, fg[1]);
          if constexpr (PARTS == 3) multiply(fl, fg[1]);
          multiply(fh, fg[0]);
          multiply(fl, fg[0]);
          if constexpr (PARTS == 3) {
            multiply(*(const bf16x8*)(np + ct * 8192 + cell), fg[0]);          // the third part, [third | first]
            multiply(fh, fg[2]);
          }
        }
      };
      phase();
      wait_loads<0>();
      barrier();
      for (int gi = w; gi < groups; gi += 8) {
        if (gi != w) load_g(s_first + gi);
        mix(gi);
      }
      if ((c + 1) * ct < tiles) {
        const int then = base + all, n_all = min(ct, tiles - (c + 1) * ct) * 2 * KW;
#pragma unroll
        for (int i = 0; i < D; ++i) load_unit(then + n_all * w / 8 + i, fw[i]);
      }
    }
    // the eight partial sums of each output: a wave adds up four registers of each
    phase();
    f32x4* red = (f32x4*)smem + l;
    barrier();
#pragma unroll
    for (int val = 0; val < 2; ++val)
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const f32x16& v = acc[val][q / 4];
        const int e = q % 4 * 4;
        red[((w * 2 + val) * 8 + q) * 64] = f32x4{v[e], v[e + 1], v[e + 2], v[e + 3]};
      }
    request_first(next);
    barrier();
#pragma unroll
    for (int val = 0; val < 2; ++val) {
      f32x4 v = red[(val * 8 + w) * 64];
#pragma unroll
      for (int k = 1; k < 8; ++k) v += red[((k * 2 + val) * 8 + w) * 64];
      float* at = sums_of(blk, val) + (prow + lh * 4) * kD + l31;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (prow + lh * 4 + i < x.m) at[i * kD] = old[val][i] + v[i];
    }
    return true;
  };

  for (int k = -1; k < wa.n; ++k) {
    const int blk = wa.hi - k;
    const bool now = tile < tiles && (k & 1) == half, next = tile < tiles && (k & 1) != half && k + 1 < wa.n;   // whose rows are its own
    if (k >= 0 && now && !differentiate(blk, 4u * k)) return;
    if (next) prepare(blk - 1);
    if (k < 0) {
      request_first(next ? blk - 1 : -1);
      continue;
    }
    look_ahead(blk);
    if (now) signal(chain_count);
    if (!cache_rows(blk, next ? blk - 1 : -1, (uint32_t)(mine + tiles * (k + 1)))) return;
    signal(rows_count);
  }
}

// What a call starts with: the filters in the order bwd_dx_k's waves read them, zeros from `zero` on, and the walk's counters (null:
// not its business)
__global__ void bwd_begin_k(StepArgs a, uint16_t* wf, int banks, u32x4* zero, int64_t zeros, uint32_t* sync) {
  if (sync && blockIdx.x == 0) {             // (see WalkArgs: the status word and the masks of the scan in between are kept)
    const int chains = a.batch * a.Hkv, words = 2 * chains * (a.M / 32);
    for (int i = threadIdx.x; i < chains; i += blockDim.x) sync[i] = 0u;
    for (int i = threadIdx.x; i < words; i += blockDim.x) sync[2 * chains + 1 + i] = 0u;
  }
  const int C = a.conv_in ? 2 * kD : kD, KW = a.k_width, n16 = (a.M + 15) / 16;
  const int64_t step = (int64_t)gridDim.x * blockDim.x, n = (int64_t)banks * (C / 32) * n16 * KW * 64;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += step) {
    const int l = (int)(e & 63);
    int64_t r = e >> 6;
    const int t = (int)(r % KW); r /= KW;
    const int s = (int)(r % n16) * 16 + (l >> 5) * 8; r /= n16;
    const int c = (int)(r % (C / 32)) * 32 + (l & 31), bank = (int)(r / (C / 32));
    const uint16_t* w = (const uint16_t*)a.conv_w + bank * a.w_head_stride + ((int64_t)s * C + c) * KW + t;
    uint16_t v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = s + q < a.M ? w[(int64_t)q * C * KW] : (uint16_t)0;
    u32x4 out;
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = v[2 * q] | (uint32_t)v[2 * q + 1] << 16;
    *(u32x4*)(wf + e * 8) = out;
  }
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < zeros; e += step) zero[e] = u32x4{0u, 0u, 0u, 0u};
}

// ---- dW: a workgroup per (128 slots, 128 columns, two taps) and share of the contraction over (block, chain, position),
// in stages of 32 positions.  The plane rows and the entries' rows (33 of them: the two taps are one row apart) come two
// stages ahead into a ring of three; both operands are read down their rows, and the fragments of dl serve both taps.
// Sums go to dwt [bank][tap][slot][channel] with atomics, once per workgroup.  Bound by the products: 99 us a block of 32
// chains, 512 slots and 1024 positions in windows of nine, 1.3 PFLOP/s (210 us with a tap per workgroup and the atomics once
// per block).
constexpr int kDwDl = 4 * 32 * 128, kDwX = 36 * 256, kDwStage = kDwDl + kDwX;
__global__ __launch_bounds__(256, 2) void bwd_dw_k(BwdConvArgs g, int groups, int n_units, int spu) {
  extern __shared__ __align__(16) unsigned char smem[];
  const StepArgs& a = g.st;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)smem);
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l31 = l & 31, lh = l >> 5;
  const int KW = a.k_width, pad = (KW - 1) / 2, C = a.conv_in ? 2 * kD : kD, tiles = (a.M + 31) / 32;
  const int tg = (KW + 1) / 2, stiles = (a.M + 127) / 128;
  const int gi = blockIdx.x % groups, tile = blockIdx.x / groups;
  const int t0 = (tile % tg) * 2, st = (tile / tg) % stiles, val = tile / tg / stiles, sbw = st * 4 + w;
  const bool two = t0 + 1 < KW, per_head = a.w_head_stride != 0;
  const int hkv = per_head ? blockIdx.y : 0;
  // unit u: (block, chain), or (block, batch entry) of this kv head where the filters are per head
  const int per_blk = per_head ? a.batch : a.batch * a.Hkv;
  const int64_t total = (int64_t)n_units * spu;
  int64_t n = total * gi / groups;
  const int64_t n_end = total * (gi + 1) / groups;
  if (n >= n_end) return;
  const unsigned char* zero = (const unsigned char*)g.zero_page;

  // where the stage requested next stands, and its unit's rows
  int blk = (int)(n / spu) / per_blk, e = (int)(n / spu) % per_blk, stage = (int)(n % spu);
  const View& sv = val ? a.v : a.k;
  const int64_t st_bytes = sv.st * 2;
  const bool near_rows = st_bytes * 36 < 0x7fffffff;                // a stage's rows of a block have 32-bit offsets
  int m = 0, T = 0;
  const unsigned char* plane = nullptr;
  const unsigned char* crow = nullptr;
  const unsigned char* brow = nullptr;
  auto enter_unit = [&]() {
    const int ch = per_head ? e * a.Hkv + hkv : e;
    const Block x = block_of(g, blk < g.n_blk ? blk : 0);
    m = x.m;
    T = x.T;
    plane = (const unsigned char*)(g.dl + blk * g.plane_stride) + ((int64_t)ch * tiles + sbw) * g.P * 128;
    crow = (const unsigned char*)((val ? x.cv : x.ck) + (int64_t)ch * a.M * kD);
    brow = (const unsigned char*)((val ? x.v : x.k) + (ch / a.Hkv) * sv.sb + (ch % a.Hkv) * sv.sh);
  };
  uint32_t dvo[4], cvo[3], bvo[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {            // 32 rows of slot block sbw
    const int r = i * 8 + (l >> 3);
    dvo[i] = r * 128 + (((l & 7) ^ pswz(r)) << 4);
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {            // entry rows 8 w .. + 7, and 32 .. 35 (wave 0)
    const int r = (i < 2 ? w * 2 + i : 8) * 4 + (l >> 4), c = ((l & 15) ^ swz(r)) << 4;
    cvo[i] = r * 256 + c;
    bvo[i] = (uint32_t)(r * st_bytes) + c;
  }
  auto request = [&](int buf) {
    const int pc = stage * 32, q0 = pc + t0 - pad;
    const uint32_t lds = lds0 + buf * kDwStage, ldx = lds + kDwDl;
    if (pc < T && sbw < tiles) {           // (the planes are padded with zeros to whole stages)
      const unsigned char* p = plane + (int64_t)pc * 128;
#pragma unroll
      for (int i = 0; i < 4; ++i) gather_to_lds(p, dvo[i], lds + (w * 4 + i) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) gather_to_lds(zero, (uint32_t)(l & 15) * 16, lds + (w * 4 + i) * 1024);
    }
    const uint32_t at[3] = {ldx + w * 2048, ldx + w * 2048 + 1024, ldx + 8192};
    if (q0 >= 0 && q0 + 36 <= m) {         // all rows in the cache
      const unsigned char* p = crow + (int64_t)q0 * 256;
      gather_to_lds(p, cvo[0], at[0]);
      gather_to_lds(p, cvo[1], at[1]);
      if (w == 0) gather_to_lds(p, cvo[2], at[2]);
    } else if (q0 >= m && q0 + 36 <= T && near_rows) {   // all in the block
      const unsigned char* p = brow + (q0 - m) * st_bytes;
      gather_to_lds(p, bvo[0], at[0]);
      gather_to_lds(p, bvo[1], at[1]);
      if (w == 0) gather_to_lds(p, bvo[2], at[2]);
    } else {                               // across the seam or an end: row by row, zeros outside
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int r = (i < 2 ? w * 2 + i : 8) * 4 + (l >> 4), q = q0 + r, c = ((l & 15) ^ swz(r)) << 4;
        const unsigned char* p = q < m ? crow + (int64_t)q * 256 : brow + (q - m) * st_bytes;
        p = q >= 0 && q < T ? p + c : zero + (l & 15) * 16;
        if (i < 2 || w == 0) gather_to_lds(p, at[i]);
      }
    }
    if (++stage == spu) {
      stage = 0;
      if (++e == per_blk) { e = 0; ++blk; }
      enter_unit();
    }
  };
  const int wy = w >> 1, wx = w & 1, s16 = l & 15, g2 = (l >> 4) & 1;
  int da[2];                               // [4-row half] of k step 0, slot block wy * 2 (high halves; low: ^ 64)
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = lh * 8 + (s16 >> 2) + 4 * h, chunk = 2 * g2 + ((s16 & 3) >> 1);
    da[h] = wy * 2 * 32 * 128 + r * 128 + ((chunk ^ pswz(r)) << 4) + (s16 & 1) * 8;
  }
  int xa[2][2][2];                         // [tap][column block][4-row half]
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = lh * 8 + (s16 >> 2) + 4 * h + t, chunk = 8 * wx + 4 * cb + 2 * g2 + ((s16 & 3) >> 1);
        xa[t][cb][h] = kDwDl + r * 256 + ((chunk ^ swz(r)) << 4) + (s16 & 1) * 8;
      }
  f32x16 acc[2][2][2];                     // [tap][slot block][column block]
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[t][y][c] = zero16();
  enter_unit();
  request(0);
  if (n + 1 < n_end) request(1);
  wait_loads<0>();
  barrier();
  int buf = 0;
  for (; n < n_end; ++n) {
    const bool more = n + 2 < n_end;
    if (more) request(buf == 0 ? 2 : buf - 1);
    const unsigned char* base = smem + buf * kDwStage;
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {       // (16 rows on: swz and pswz repeat)
      bf16x8 fh[2], fl[2], fx[2][2];
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const unsigned char* p = base + y * 32 * 128 + kc * 16 * 128;
        fh[y] = frag_tr(p + da[0], p + da[1]);
        fl[y] = frag_tr(p + (da[0] ^ 64), p + (da[1] ^ 64));
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) fx[t][c] = frag_tr(base + kc * 16 * 256 + xa[t][c][0], base + kc * 16 * 256 + xa[t][c][1]);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (t && !two) break;
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int c = 0; c < 2; ++c) acc[t][y][c] = mfma32(fh[y], fx[t][c], acc[t][y][c]);
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int c = 0; c < 2; ++c) acc[t][y][c] = mfma32(fl[y], fx[t][c], acc[t][y][c]);
      }
    }
    if (!more) wait_loads<0>();            // the next stage has landed; this one's requests may be on their way
    else if (w == 0) wait_loads<7>();
    else wait_loads<6>();
    barrier();
    buf = buf == 2 ? 0 : buf + 1;
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (t && !two) break;
    float* o = g.dwt + (((int64_t)hkv * KW + t0 + t) * a.M) * C + val * kD;
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int s = st * 128 + wy * 64 + y * 32 + (i >> 2) * 8 + lh * 4 + (i & 3);
        if (s >= a.M) continue;
#pragma unroll
        for (int c = 0; c < 2; ++c) atomicAdd(o + (int64_t)s * C + wx * 64 + c * 32 + l31, acc[t][y][c][i]);
      }
  }
}

// d_conv_w[bank][slot][channel][tap] += dwt[bank][tap][slot][channel]
__global__ void bwd_add_dw_k(const float* dwt, float* d_conv_w, int M, int C, int KW, int banks, int64_t w_head_stride) {
  const int64_t n = (int64_t)banks * M * C * KW;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(e % KW);
    const int c = (int)((e / KW) % C);
    const int s = (int)((e / ((int64_t)KW * C)) % M);
    const int bank = (int)(e / ((int64_t)KW * C * M));
    d_conv_w[bank * w_head_stride + ((int64_t)s * C + c) * KW + t] += dwt[(((int64_t)bank * KW + t) * M + s) * C + c];
  }
}

template <typename F>
hipError_t allow_lds(F* k, int bytes, bool& done) {      // benign race: setting it twice is harmless
  if (done) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  done = e == hipSuccess;
  return e;
}

template <int NT, bool MULTI, int NORM>
void launch_rows_norm(const BwdConvArgs& g, int blk, int T, int grid, hipStream_t s) {
  if (T % 4 == 0 && !g.three_parts) hipLaunchKernelGGL((bwd_rows_k<NT, MULTI, NORM, 2>), dim3(grid), dim3(512), 0, s, g, blk);
  else hipLaunchKernelGGL((bwd_rows_k<NT, MULTI, NORM, 3>), dim3(grid), dim3(512), 0, s, g, blk);
}
template <int NT, bool MULTI>
void launch_rows(const BwdConvArgs& g, int blk, int T, int grid, hipStream_t s) {
  if (g.st.norm == 0) launch_rows_norm<NT, MULTI, 0>(g, blk, T, grid, s);
  else launch_rows_norm<NT, MULTI, 1>(g, blk, T, grid, s);
}

template <int PT, int NC, int KS, bool FINE>
hipError_t launch_dx(const BwdConvArgs& g, int blk0, int n_blk, int part, int rows, hipStream_t s) {
  constexpr int lds = Dx<PT, NC, KS, FINE>::lds;
  static bool lds_set = false;
  const hipError_t e = allow_lds(bwd_dx_k<PT, NC, KS, FINE>, lds, lds_set);
  if (e != hipSuccess) return e;
  const StepArgs& a = g.st;
  hipLaunchKernelGGL((bwd_dx_k<PT, NC, KS, FINE>), dim3((rows + PT - 1) / PT, a.batch * a.Hkv, 256 / NC * n_blk), dim3(512), lds, s, g, blk0,
                     part);
  return hipGetLastError();
}

template <int NT, int PARTS>
hipError_t walk_kernel(const WalkArgs& wa, int grid, int n_cu, bool* resident, hipStream_t s) {
  static bool lds_set = false;
  const int lds = walk_lds<PARTS>(wa.c.st.M / 32, wa.c.st.k_width);
  hipError_t e = allow_lds(bwd_walk_k<NT, PARTS>, 160 * 1024 - 1024, lds_set);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)bwd_walk_k<NT, PARTS>, 512, lds);
  if (e != hipSuccess) return e;
  const int64_t limit = debug_options().max_resident > 0 ? debug_options().max_resident : (int64_t)per_cu * n_cu;
  *resident = grid <= limit;
  if (!*resident) return hipSuccess;
  hipLaunchKernelGGL((bwd_walk_k<NT, PARTS>), dim3(grid), dim3(512), lds, s, wa);
  return hipGetLastError();
}

}  // namespace

BwdConvLayout bwd_conv_layout(int batch, int Hkv, int M, int T, int conv_width, int conv_in, int banks, int64_t n_blk, bool with_logits,
                              bool one_filters) {
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  const size_t chains = (size_t)batch * Hkv, C = conv_in ? 2 * kD : kD;
  BwdConvLayout l;
  l.ld = l.P = (T + 31) / 32 * 32;
  l.logits_stride = up((chains * M + 31) * l.ld * 4) / 4;        // (whole tiles of 32 slots are read)
  l.plane_stride = up(chains * ((M + 31) / 32) * l.P * 128) / 2;
  l.gsplit_stride = up(chains * ((M + 31) / 32 * 32) * 2 * kD * 2 * 3) / 2;
  size_t at = 0;
  auto take = [&](size_t bytes) { const size_t here = at; at += up(bytes); return here; };
  const size_t wf_bytes = (size_t)banks * conv_width * ((M + 15) / 16 * 16) * C * 2;
  l.wt = take(one_filters ? wf_bytes : (size_t)banks * conv_width * M * C * 2);
  l.wf = one_filters ? l.wt : take(wf_bytes);
  l.zero_page = take(256);
  l.dwt = take((size_t)banks * conv_width * M * C * 4);
  l.per_call = at;
  l.logits = take(with_logits ? (size_t)n_blk * l.logits_stride * 4 : 0);
  l.dl = take((size_t)n_blk * l.plane_stride * 2);
  l.wn = take((size_t)n_blk * l.plane_stride * 2);
  l.wn_low = take((size_t)n_blk * l.plane_stride * 2);
  l.gsplit = take((size_t)n_blk * l.gsplit_stride * 2);
  l.total = at;
  return l;
}

void bwd_conv_place(BwdConvArgs* g, const BwdConvLayout& l, void* ws) {
  char* p = (char*)ws;
  g->wt = (uint16_t*)(p + l.wt);
  g->wf = (uint16_t*)(p + l.wf);
  g->zero_page = p + l.zero_page;
  g->dwt = (float*)(p + l.dwt);
  g->logits = (float*)(p + l.logits);
  g->dl = (uint16_t*)(p + l.dl);
  g->wn = (uint16_t*)(p + l.wn);
  g->wn_low = (uint16_t*)(p + l.wn_low);
  g->gsplit = (uint16_t*)(p + l.gsplit);
  g->logits_stride = (int64_t)l.logits_stride;
  g->plane_stride = (int64_t)l.plane_stride;
  g->gsplit_stride = (int64_t)l.gsplit_stride;
  g->ld = l.ld;
  g->P = l.P;
}

hipError_t launch_bwd_conv_begin(const BwdConvArgs& g, bool for_logits, void* walk_sync_ws, hipStream_t s) {
  const StepArgs& a = g.st;
  const size_t n = (size_t)g.banks * a.k_width * a.M * (a.conv_in ? 2 * kD : kD);
  const bool one_filters = g.wf == g.wt;     // (then launch_bwd_conv_logits packs them)
  if (for_logits && !one_filters) {
    const hipError_t e = launch_pack_filters_per_tap(a, g.banks, g.wt, s);
    if (e != hipSuccess) return e;
  }
  // the page of zeros lies right before the sums (n is a multiple of 4)
  const int64_t zeros = ((char*)(g.dwt + n) - (char*)g.zero_page) / 16;
  hipLaunchKernelGGL(bwd_begin_k, dim3((unsigned)std::min<int64_t>((zeros + 255) / 256, 2048)), dim3(256), 0, s, a, g.wf,
                     one_filters ? 0 : g.banks, (u32x4*)g.zero_page, zeros, (uint32_t*)walk_sync_ws);
  return hipGetLastError();
}

hipError_t launch_bwd_conv_logits(const BwdConvArgs& g, hipStream_t s) {
  StepArgs a = g.st;
  a.ldw = g.ld;
  LogitsWindow win = {g.n_blk, g.B, g.tokens, g.state_stride, g.logits_stride};
  if (g.wf != g.wt) return launch_conv_logits_mfma(a, g.wt, g.logits, s, &win);
  // one place for both packings: that per tap for this kernel, then the one the kernels of the walk read
  hipError_t e = launch_pack_filters_per_tap(a, g.banks, g.wt, s);
  if (e == hipSuccess) e = launch_conv_logits_mfma(a, g.wt, g.logits, s, &win);
  if (e != hipSuccess) return e;
  const int64_t n = (int64_t)g.banks * (a.conv_in ? 2 : 1) * (kD / 32) * ((a.M + 15) / 16) * a.k_width * 64;
  hipLaunchKernelGGL(bwd_begin_k, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 2048)), dim3(256), 0, s, a, g.wf, g.banks,
                     (u32x4*)g.zero_page, 0, (uint32_t*)nullptr);
  return hipGetLastError();
}

hipError_t launch_bwd_conv_rows(const BwdConvArgs& g, int blk, int T, hipStream_t s) {
  const StepArgs& a = g.st;
  const int grid = (a.M + 31) / 32 * a.batch * a.Hkv;
  if (T <= 256) launch_rows<1, false>(g, blk, T, grid, s);
  else if (T <= 512) launch_rows<2, false>(g, blk, T, grid, s);
  else if (T <= 1024) launch_rows<4, false>(g, blk, T, grid, s);
  else launch_rows<2, true>(g, blk, T, grid, s);
  return hipGetLastError();
}

template <bool FINE>
static hipError_t launch_dx_tiles(const BwdConvArgs& g, int blk0, int n_blk, int part, int rows, hipStream_t s) {
  // The largest tile of which there is one for every compute unit.  128 rows have one to themselves, 64 share it by two (32 chains,
  // 512 slots on 1024 positions: 142 and 153 us, 128 slots, 27 blocks of 128 rows: 175 and 179), so 64 where they leave a tenth
  // less to pad: blocks of 134 rows 1000 -> 868 us, 192 rows 341 -> 273, 320 rows 256 -> 220, 303 rows (three parts) 565 -> 524.
  // 32 rows in halves, two workgroups on a compute unit, where even those are too few (128 slots: 11.9 us, whole 15.0).  The
  // slots of 32 rows go four ways, two workgroups on a compute unit: with eight, one (256 slots: 31.6 against 28.8 us; 160: 51 -
  // 39; 384: 63 - 59; three parts 71 - 66).
  const int64_t per = (int64_t)g.st.batch * g.st.Hkv * n_blk, slots = g.st.M;
  const int64_t rows128 = ((int64_t)rows + 127) / 128 * 128, rows64 = ((int64_t)rows + 63) / 64 * 64, halves = per * ((rows + 31) / 32) * 4;
  if (per * (rows128 / 128) >= cu_count() && rows128 * 10 <= rows64 * 11) return launch_dx<128, 128, 4, FINE>(g, blk0, n_blk, part, rows, s);
  if (per * (rows64 / 64) >= cu_count()) return launch_dx<64, 128, 4, FINE>(g, blk0, n_blk, part, rows, s);
  if (per * ((rows + 31) / 32) >= cu_count()) return launch_dx<32, 128, 4, FINE>(g, blk0, n_blk, part, rows, s);
  // Halves go eight ways, half as many phases in series, but four ways where that leaves an eighth less of the slots to pad and
  // there are workgroups enough to fill each other's waits.  Four against eight ways, by workgroups: 192 slots 128 1.02, 256 0.99,
  // 384 0.91 (three parts 0.99, 0.97, 0.91); 320 slots 192 1.08, 384 1.03, 576 0.96 (1.08, 1.04, 0.87); 448 slots 256 1.16, 384 1.09,
  // 512 1.02, 768 0.98 (1.12, 1.10, 0.91, 0.91); 128 slots, nothing less to pad, 1.02 - 1.26.  Up to 64 slots half of eight have none.
  const int64_t enough = slots <= 64 ? 0 : slots <= 192 ? cu_count() / 2 : 2 * cu_count();
  const bool four_ways = (slots + 63) / 64 * 64 * 9 <= (slots + 127) / 128 * 128 * 8 && halves >= enough;
  return four_ways ? launch_dx<32, 64, 4, FINE>(g, blk0, n_blk, part, rows, s) : launch_dx<32, 64, 8, FINE>(g, blk0, n_blk, part, rows, s);
}
bool bwd_conv_three_parts(const BwdConvArgs& g, int i) {
  const int64_t left = g.tokens - (int64_t)i * g.B;
  return g.three_parts || ((i ? g.st.M : g.st.m) + (int)(left < g.B ? left : g.B)) % 4 != 0;
}
hipError_t launch_bwd_conv_dx(const BwdConvArgs& g, int blk0, int n_blk, int part, int rows, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  auto fine = [&](int i) { return bwd_conv_three_parts(g, i); };
  hipError_t e = hipSuccess;
  for (int i = blk0, n = 0; i < blk0 + n_blk && e == hipSuccess; i += n) {      // runs of blocks of one form
    for (n = 1; i + n < blk0 + n_blk && fine(i + n) == fine(i);) ++n;
    e = fine(i) ? launch_dx_tiles<true>(g, i, n, part, rows, s) : launch_dx_tiles<false>(g, i, n, part, rows, s);
  }
  return e;
}

// Which blocks the walk takes in one launch: whole slot tiles, Eq. 6 as a softmax over the keys' logits, all slots mixing, its
// workgroups one to a compute unit at most.  Up to 256 slots and 512 positions: the launches it saves are less of a longer step (a
// pass over 29 blocks of 100 tokens on 128 slots, 8 chains, 1101 -> 1021 us, 19 of 101 on 160 1033 -> 958, 14 of 200 on 256, 16 chains,
// 1722 -> 1611; 9 of 256 on 288, 8 chains, 907 -> 908, 15 of 331 on 384 2173 -> 2161, 9 of 400 on 512 1658 -> 1699).
bool bwd_conv_walk_takes(const BwdConvArgs& g) {
  const StepArgs& a = g.st;
  return a.M % 32 == 0 && a.norm == 0 && !a.conv_in && !a.protect && !g.d_conv_b && a.k_width <= 25 && a.M <= 256 && a.M + g.B <= 512 &&
         (int64_t)a.batch * a.Hkv * ((a.M + 63) / 64 * 4) <= cu_count() && bwd_conv_defers_blocks(g);
}
// The fewest blocks (hi, hi - 1, ..) it is worth taking: its start, a census and a first block prepared with nothing to hide that, costs
// 10 - 20 us (and clearing the counters 3 in every window but the first), and a block saves 2 - 4 in two parts, 8 in three.  A pass over
// few blocks, from a full cache, in two launches a block and in one launch, us: 128 slots, 256 positions, 32 chains 237 / 246 (2 blocks),
// 321 / 323 (4), 409 / 404 (6); 96 slots of width 21 199 / 212, 295 / 301, 373 / 372; 256 slots, 384 positions, 8 chains 248 / 261, 337 /
// 345, 427 / 433, 517 / 515 (8); 128 slots, 229 positions, three parts 249 / 256, 342 / 339, 457 / 439; 64 slots, 8 chains 136 / 142, 187 /
// 187, 234 / 229.
int bwd_conv_walk_least(const BwdConvArgs& g, int hi) { return bwd_conv_three_parts(g, hi) || g.st.M <= 64 ? 4 : 6; }
hipError_t launch_bwd_conv_walk(const BwdConvArgs& g, int hi, int n, void* sync_ws, int spin_limit, bool through_l2, bool* taken,
                                hipStream_t s) {
  const StepArgs& a = g.st;
  const int chains = a.batch * a.Hkv, tiles = a.M / 32;
  WalkArgs wa;
  wa.c = g;
  wa.hi = hi;
  wa.n = n;
  wa.sync = (uint32_t*)sync_ws;
  wa.status = (int32_t*)sync_ws + chains;
  wa.tsync = (uint32_t*)sync_ws + 2 * chains + 1;
  wa.spin_limit = spin_limit;
  wa.same_l2_allowed = through_l2 ? 1 : 0;
  const int grid = chains * ((tiles + 1) / 2 * 4), T = a.M + g.B;
  auto go = [&](auto parts) {
    constexpr int P = decltype(parts)::value;
    if (T <= 256) return walk_kernel<1, P>(wa, grid, cu_count(), taken, s);
    return walk_kernel<2, P>(wa, grid, cu_count(), taken, s);
  };
  return bwd_conv_three_parts(g, hi) ? go(std::integral_constant<int, 3>{}) : go(std::integral_constant<int, 2>{});
}

// A step alone fills the device with 128-row tiles: nothing is gained by leaving its block's rows for later.
bool bwd_conv_defers_blocks(const BwdConvArgs& g) {
  return (int64_t)g.st.batch * g.st.Hkv * ((g.st.M + g.B + 127) / 128) < cu_count();
}

hipError_t launch_bwd_conv_dw(const BwdConvArgs& g, hipStream_t s) {
  static bool lds_set = false;
  const hipError_t e = allow_lds(bwd_dw_k, 3 * kDwStage, lds_set);
  if (e != hipSuccess) return e;
  const StepArgs& a = g.st;
  const bool per_head = a.w_head_stride != 0;
  const int units = g.n_blk * (per_head ? a.batch : a.batch * a.Hkv), spu = g.P / 32;
  const int tiles = (a.k_width + 1) / 2 * ((a.M + 127) / 128) * (a.conv_in ? 2 : 1);
  // two workgroups per compute unit, the workgroups of a share (all tiles read the same rows) on one XCD
  const int64_t want = std::max<int64_t>(1, 2 * cu_count() / ((int64_t)tiles * (per_head ? a.Hkv : 1)));
  int64_t groups = std::min<int64_t>(want >= 8 ? want / 8 * 8 : want, (int64_t)units * spu);
  hipLaunchKernelGGL(bwd_dw_k, dim3((unsigned)(tiles * groups), per_head ? a.Hkv : 1), dim3(256), 3 * kDwStage, s, g,
                     (int)groups, units, spu);
  return hipGetLastError();
}

hipError_t launch_bwd_conv_end(const BwdConvArgs& g, hipStream_t s) {
  const StepArgs& a = g.st;
  const int C = a.conv_in ? 2 * kD : kD;
  const int64_t n = (int64_t)g.banks * a.k_width * a.M * C;
  hipLaunchKernelGGL(bwd_add_dw_k, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, s, g.dwt, g.d_conv_w,
                     a.M, C, a.k_width, g.banks, a.w_head_stride);
  return hipGetLastError();
}

}  // namespace lococo
