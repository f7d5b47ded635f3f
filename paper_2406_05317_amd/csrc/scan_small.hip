// Small scans of the shape-agnostic path (single precision, or bf16 with a head_dim the MFMA kernels do not
// take): Eq. 5 + Eq. 6 + Eq. 4a / 4b of a block in one workgroup per (chain, group of 16-slot tiles), everything
// in LDS, contractions on the fp32 matrix instruction (v_mfma_f32_16x16x4: fp32 operands, fp32 sums), and the
// attention of many blocks in one launch.
//
// What bounds it: latency.  The smallest scan (one head of 64, M = B = 16, width 3, 256 tokens) is 0.2 MFLOP per
// step, so a step is a handful of dependent LDS passes; what it costs is launches and idle lanes.  Where the
// whole chain fits one workgroup (filters included) the steps of a scan therefore run in ONE launch, the cache
// rows staying in LDS from step to step; otherwise each step is one launch of a workgroup per 16 slots.
// Measured on that smallest scan (15 compressions): 1209 us with three kernels per step and one attention launch per
// block (63 us of each step in the 64 x 64-tiled Eq. 5, one workgroup), 71 us here.  Before operand reads were issued in groups
// ahead of their products, reductions left the LDS crossbar, divisions the index arithmetic and row strides became constants
// for head_dim 64 it was 104 us, 12 900 cycles a step.  Two heads of other sizes gained as well, fp32 and bf16: 576 tokens of
// 32, 96 slots, width 15: 182 -> 139 us; 144 of 56, 24 slots, width 5: 88 -> 75; 192 of 80, 32 slots: 110 -> 96; 96 of 128,
// 16 slots, width 3: 63 -> 54 (bf16 64 -> 64); 384 of 64, 64 slots, width 9: 159 -> 127.
#include <algorithm>
#include <type_traits>

#include "lococo_internal.h"

namespace lococo {
namespace {

struct bf16_t { uint16_t x; };
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

__device__ __forceinline__ float to_f(float v) { return v; }
__device__ __forceinline__ float to_f(bf16_t v) { return __uint_as_float((uint32_t)v.x << 16); }
// stores v and returns what was stored
__device__ __forceinline__ float store_f(float v, float* out) { *out = v; return v; }
__device__ __forceinline__ float store_f(float v, bf16_t* out) {
  uint32_t u = __float_as_uint(v);
  if ((u & 0x7fffffffu) > 0x7f800000u) u = (u | 0x400000u) & 0xffff0000u;   // NaN
  else u += 0x7fffu + ((u >> 16) & 1u);                                     // round to nearest, ties to even
  out->x = (uint16_t)(u >> 16);
  return __uint_as_float(u & 0xffff0000u);
}

// LDS written by one lane is read by another of the same wave
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v combined over the 32 lanes of each half of a wave, on the vector unit alone
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <typename Op>
__device__ __forceinline__ float over32(float v, Op op) {
  v = op(v, dpp<0xB1>(v));                   // quad_perm [1,0,3,2]
  v = op(v, dpp<0x4E>(v));                   // quad_perm [2,3,0,1]
  v = op(v, dpp<0x141>(v));                  // row_half_mirror
  v = op(v, dpp<0x140>(v));                  // row_mirror
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// u / n for small numbers (exact below two million): the integer division is a chain of some forty instructions
__device__ __forceinline__ int small_div(int u, int n) {       // (both uniform)
  return __builtin_amdgcn_readfirstlane((int)(((float)u + 0.5f) * __builtin_amdgcn_rcpf((float)n)));
}

constexpr int kNT = 512, kNW = kNT / 64;     // threads, waves
constexpr int kPG = 2;                       // position tiles of 16 per unit of Eq. 5
constexpr int kMaxMix = 8;                   // 16 x 16 tiles of Eq. 4 a wave holds at once
constexpr int kPF = 8;                       // values of the next block a thread fetches ahead, per array
constexpr int kLds = 160 * 1024;

// Row strides are a multiple of 4 floats that is an odd multiple of 4: the 16 rows x 4 columns one operand
// read touches then fall on 64 different banks.
__host__ __device__ constexpr int odd4(int n) {
  const int q = (n + 3) / 4;
  return 4 * (q | 1);
}

// Parts the inner dimension of Eq. 5 is shared out in where a slot tile has fewer units than there are waves.  A
// function of the positions alone, so that every form of the launch adds up in the same order.
static_assert(kNW == 8, "eight waves over the parts");
__host__ __device__ inline int log_planes_of(int pg) { return pg == 1 ? 3 : pg == 2 ? 2 : pg <= 4 ? 1 : 0; }
__host__ __device__ inline int planes_of(int pg) { return 1 << log_planes_of(pg); }

struct SmallLayout {
  int tiles;          // slot tiles of 16 per workgroup
  int sx, sv;         // row strides (floats) of X and V (0: V inside X)
  int taps;           // taps whose filters are resident at once
  int off_v, off_l, off_w, bytes;
};

// Layout for up to T positions; it fits where bytes <= kLds.
SmallLayout layout_of(int T, int d, int k, int conv_in, int tiles, int taps) {
  SmallLayout l;
  const int C = conv_in ? 2 * d : d, pg = (T + 31) / 32;
  l.tiles = tiles;
  l.taps = taps;
  l.sx = odd4(C);
  l.sv = conv_in ? 0 : odd4(d);
  int64_t at = (int64_t)(32 * pg + k + 3) * l.sx;    // the positions, the zero rows around them, whole groups of 32
  l.off_v = (int)at;
  at += (int64_t)((T + 3) / 4 * 4) * l.sv;
  l.off_l = (int)at;
  int planes = 0;
  for (int g = 1; g <= pg; ++g) planes = std::max(planes, planes_of(g) * odd4(32 * g));
  at += (int64_t)planes * tiles * 16;
  l.off_w = (int)at;
  at += (int64_t)tiles * taps * ((C + 3) / 4 * 4) * 16;
  l.bytes = (int)std::min<int64_t>(at * 4, 1 << 30);
  return l;
}

struct SmallArgs {
  StepArgs st;            // step 0: source cache, occupancy, block; k / v views at its first token
  int n_steps, B;
  int64_t tokens_left;
  void* out_k; void* out_v;
  int64_t out_stride;     // elements between states
  int slot0, ring;
  SmallLayout l;
};

// One workgroup: 16 l.tiles slots of one chain.  n_steps > 1 only where those are all slots of the chain.
// MIX: 16 x 16 tiles of Eq. 4 per wave.  D: head_dim where it is a constant (0: any), and then CIN: filters over [K | V].
template <typename T, int MIX, int D, int CIN>
__global__ __launch_bounds__(kNT) void compress_small_k(SmallArgs g) {
  extern __shared__ __align__(16) float sm[];
  const StepArgs& a = g.st;
  const SmallLayout& L = g.l;
  float* Xs = sm;
  float* Vs = sm + L.off_v;
  float* Ls = sm + L.off_l;
  float* Ws = sm + L.off_w;
  int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l15 = l & 15, lk = l >> 4;
  const int ch = blockIdx.y, b = ch / a.Hkv, hkv = ch % a.Hkv, i0 = blockIdx.x * 16 * L.tiles;
  const int d = D ? D : a.d, C = (D ? CIN : a.conv_in) ? 2 * d : d, C4 = (C + 3) / 4, k = a.k_width, pad = (k - 1) / 2, M = a.M;
  const int sx = D ? odd4(C) : L.sx, sv = D ? (CIN ? 0 : odd4(d)) : L.sv;
  const T* wbase = (const T*)a.conv_w + hkv * a.w_head_stride;
  const T* bias = a.conv_b ? (const T*)a.conv_b + hkv * a.b_head_stride : nullptr;
  const uint32_t* protect = a.protect ? a.protect + (int64_t)ch * a.protect_stride : nullptr;

  // where column c of the value row / key row of position j lives
  auto yv = [&](int j) -> float* { return sv ? Vs + j * sv : Xs + (pad + j) * sx + d; };
  auto load_filters = [&](int t0, int nt) {       // [tile][tap][channel (padded to 4)][slot]
    for (int st = 0; st < L.tiles; ++st) {
      const int i = i0 + st * 16 + (tid & 15);
      for (int f = tid >> 4; f < C4 * 4 * nt; f += kNT / 16) {
        const int c = f / nt, t = f % nt;
        Ws[((st * L.taps + t) * C4 * 4 + c) * 16 + (tid & 15)] =
            i < M && c < C ? to_f(wbase[((int64_t)i * C + c) * k + t0 + t]) : 0.f;
      }
    }
  };
  const T* kb = (const T*)a.k.p + b * a.k.sb + hkv * a.k.sh;
  const T* vb = (const T*)a.v.p + b * a.v.sb + hkv * a.v.sh;
  // rows of the first state and the first block; everything else of X and V starts at zero
  for (int e = tid; e < L.off_l; e += kNT) sm[e] = 0.f;
  __syncthreads();
  int m = a.m, Bn = a.Bn;
  {
    const T* ck = (const T*)a.cache_k + (int64_t)ch * M * d;
    const T* cv = (const T*)a.cache_v + (int64_t)ch * M * d;
    for (int e = tid; e < (m + Bn) * d; e += kNT) {
      const int j = e / d, c = e % d;
      Xs[(pad + j) * sx + c] = to_f(j < m ? ck[e] : kb[(int64_t)(j - m) * a.k.st + c]);
      yv(j)[c] = to_f(j < m ? cv[e] : vb[(int64_t)(j - m) * a.v.st + c]);
    }
  }
  const bool resident = L.taps == k;
  if (resident) load_filters(0, k);

  int slot = g.slot0 % g.ring;
  for (int step = 0;; ++step) {
    asm volatile("" : "+v"(tid), "+s"(w), "+v"(l15), "+v"(lk));   // addresses belong to the step: hoisted, they all spill
    const int Tn = m + Bn, pg = (Tn + 16 * kPG - 1) / (16 * kPG), units = L.tiles * pg;
    const int log_planes = log_planes_of(pg), planes = 1 << log_planes, sl = odd4(32 * pg), plane = L.tiles * 16 * sl;
    const int64_t next_tok = (int64_t)(step + 1) * g.B;
    const bool more = step + 1 < g.n_steps;
    const int Bnext = more ? (int)min((int64_t)g.B, g.tokens_left - next_tok) : 0;
    // the next block's first values, in flight under this step
    float pk[kPF], pv[kPF];
    {
      const T* kp = kb + next_tok * a.k.st;
      const T* vp = vb + next_tok * a.v.st;
#pragma unroll
      for (int n = 0; n < kPF; ++n) {
        if (n * kNT >= Bnext * d) break;
        const int e = tid + n * kNT;
        if (e < Bnext * d) {
          pk[n] = to_f(kp[(int64_t)(e / d) * a.k.st + e % d]);
          pv[n] = to_f(vp[(int64_t)(e / d) * a.v.st + e % d]);
        }
      }
    }
    __syncthreads();
    // ---- Eq. 5: 32 positions x 16 slots per unit (A: positions x channels at a tap's row shift, B: filters)
    for (int t0 = 0; t0 < k; t0 += L.taps) {
      const int nt = min(L.taps, k - t0);
      if (!resident) {
        __syncthreads();
        load_filters(t0, nt);
        __syncthreads();
      }
      for (int u = w; u < units * planes; u += kNW) {
        const int part = small_div(u, units), uu = u - part * units, st = small_div(uu, pg), p0 = (uu - st * pg) * 16 * kPG;
        f32x4 acc[kPG];
        float* out = Ls + part * plane + (st * 16 + l15) * sl + p0 + 4 * lk;
#pragma unroll
        for (int x = 0; x < kPG; ++x) acc[x] = t0 ? *(const f32x4*)(out + 16 * x) : f32x4{0.f, 0.f, 0.f, 0.f};
        // this part's channels, tap by tap: the order of the sum does not depend on how the taps are brought in
        const int k0 = C4 * part >> log_planes, k1 = C4 * (part + 1) >> log_planes;
        const float* wb = Ws + (st * L.taps * C4 * 4 + lk) * 16 + l15 + k0 * 64;
        const float* xb = Xs + (p0 + l15 + t0) * sx + lk + 4 * k0;
        // KN channel groups at a time, TN taps of them in flight together: a wave's operand reads are what it waits for
        auto taps = [&](auto kn, auto tn, auto rect) {
          constexpr int KN = decltype(kn)::value, TN = decltype(tn)::value;
          auto some = [&](auto n_t, int kc) {
            constexpr int N = decltype(n_t)::value;
            float fb[N][KN], fa[N][KN][kPG];
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
              for (int q = 0; q < KN; ++q) {
                fb[t][q] = wb[(t * C4 + kc + q) * 64];
#pragma unroll
                for (int x = 0; x < kPG; ++x) fa[t][q][x] = xb[(16 * x + t) * sx + 4 * (kc + q)];
              }
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
              for (int q = 0; q < KN; ++q)
#pragma unroll
                for (int x = 0; x < kPG; ++x) {
                  if (decltype(rect)::value) fa[t][q][x] = fmaxf(fa[t][q][x], 0.f);   // the rectifier in front of the convolution
                  acc[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[t][q][x], fb[t][q], acc[x], 0, 0, 0);
                }
          };
          int t = 0;
          if (TN > 1)
#pragma clang loop unroll(disable)
            for (; t + TN <= nt; t += TN, wb += TN * C4 * 64, xb += TN * sx) some(tn, 0);
#pragma clang loop unroll(disable)
          for (; t < nt; ++t, wb += C4 * 64, xb += sx)
#pragma clang loop unroll(disable)
            for (int kc = 0; kc < k1 - k0; kc += KN) some(std::integral_constant<int, 1>{}, kc);
        };
        auto widths = [&](auto rect) {
          const int kn = k1 - k0;
          if (kn == 2) taps(std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{}, rect);
          else if (kn == 4) taps(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{}, rect);
          else if (kn % 8 == 0) taps(std::integral_constant<int, 8>{}, std::integral_constant<int, 1>{}, rect);
          else taps(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, rect);
        };
        if (a.norm == 2) widths(std::true_type{});
        else widths(std::false_type{});
#pragma unroll
        for (int x = 0; x < kPG; ++x) *(f32x4*)(out + 16 * x) = acc[x];
      }
    }
    __syncthreads();
    // ---- Eq. 6: 32 lanes per slot
    for (int row = tid >> 5; row < L.tiles * 16; row += kNT / 32) {
      const int i = i0 + row, c = tid & 31;
      float* r = Ls + row * sl;
      const float bi = bias && i < M ? to_f(bias[i]) : 0.f;
      const bool soft = a.norm == 0;
      float mx = -INFINITY;
      for (int j = c; j < Tn; j += 32) {
        float x = r[j] + bi;
        if (planes == kNW) {
          float more_x[kNW - 1];
#pragma unroll
          for (int p = 1; p < kNW; ++p) more_x[p - 1] = r[p * plane + j];
#pragma unroll
          for (int p = 1; p < kNW; ++p) x += more_x[p - 1];
        } else {
          for (int p = 1; p < planes; ++p) x += r[p * plane + j];
        }
        if (protect && j < m && ((protect[j >> 5] >> (j & 31)) & 1u)) x = soft ? -INFINITY : 0.f;
        r[j] = x;
        mx = fmaxf(mx, x);
      }
      if (soft) mx = over32(mx, [](float x, float y) { return fmaxf(x, y); });
      float z = 0.f;
      for (int j = c; j < Tn; j += 32) {
        const float x = r[j], e = soft ? expf(x - mx) : a.norm == 1 ? fmaxf(x, 0.f) : (isfinite(x) ? x : 0.f);
        r[j] = e;
        z += e;
      }
      z = over32(z, [](float x, float y) { return x + y; });
      if (a.norm == 1) z += a.eps;
      if (a.norm == 2 && fabsf(z) < a.eps) z = z < 0.f ? -a.eps : a.eps;
      for (int j = c; j < Tn; j += 32) r[j] /= z;
      if (c < 4 && Tn + c < (Tn + 3) / 4 * 4) r[Tn + c] = 0.f;
    }
    __syncthreads();
    // ---- Eq. 4a / 4b: 16 slots x 16 columns of [K | V] per unit (A: weights, B: rows)
    const int ct = (d + 15) / 16, mix_units = L.tiles * 2 * ct, k4 = (Tn + 3) / 4;
    f32x4 acc[MIX];
#pragma unroll
    for (int n = 0; n < MIX; ++n) {
      const int u = w + n * kNW;
      acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (u < mix_units) {
        const int st = small_div(u, 2 * ct), cu = u - st * 2 * ct;
        const bool val = cu >= ct;
        const int c = (val ? cu - ct : cu) * 16 + l15;
        const int stride = val && sv ? sv : sx;
        const float* wr = Ls + (st * 16 + l15) * sl + lk;
        const float* yr = (val ? yv(0) : Xs + pad * sx) + lk * stride + (c < d ? c : 0);   // a column past d is dropped
        int kk = 0;
#pragma clang loop unroll(disable)
        for (; kk + 8 <= k4; kk += 8, wr += 32, yr += 32 * stride) {    // eight groups of operands in flight
          float fw[8], fy[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            fw[q] = wr[4 * q];
            fy[q] = yr[4 * q * stride];
          }
#pragma unroll
          for (int q = 0; q < 8; ++q) acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[q], fy[q], acc[n], 0, 0, 0);
        }
#pragma clang loop unroll(disable)
        for (; kk < k4; ++kk, wr += 4, yr += 4 * stride)
          acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(*wr, *yr, acc[n], 0, 0, 0);
      }
    }
    __syncthreads();                                       // every read of the old rows is done
    const int64_t state = (int64_t)slot * g.out_stride + (int64_t)ch * M * d;
    if (++slot == g.ring) slot = 0;
    T* ok = (T*)g.out_k + state;
    T* ov = (T*)g.out_v + state;
#pragma unroll
    for (int n = 0; n < MIX; ++n) {
      const int u = w + n * kNW;
      if (u >= mix_units) continue;
      const int st = small_div(u, 2 * ct), cu = u - st * 2 * ct;
      const bool val = cu >= ct;
      const int c = (val ? cu - ct : cu) * 16 + l15;
      if (c >= d) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + st * 16 + lk * 4 + e;
        if (i >= M) continue;
        float* row = val ? yv(i) : Xs + (pad + i) * sx;
        float v = acc[n][e];
        if (protect && i < m && ((protect[i >> 5] >> (i & 31)) & 1u)) v = row[c];   // carried over unchanged
        v = store_f(v, (val ? ov : ok) + (int64_t)i * d + c);
        if (more) row[c] = v;
      }
    }
    if (!more) break;
    // ---- the next block behind the new cache; zeros up to the end of what this step's rows used
#pragma unroll
    for (int n = 0; n < kPF; ++n) {
      if (n * kNT >= Bnext * d) break;
      const int e = tid + n * kNT;
      if (e < Bnext * d) {
        Xs[(pad + M + e / d) * sx + e % d] = pk[n];
        yv(M + e / d)[e % d] = pv[n];
      }
    }
    for (int e = tid + kPF * kNT; e < Bnext * d; e += kNT) {
      const int64_t tok = next_tok + e / d;
      Xs[(pad + M + e / d) * sx + e % d] = to_f(kb[tok * a.k.st + e % d]);
      yv(M + e / d)[e % d] = to_f(vb[tok * a.v.st + e % d]);
    }
    for (int e = tid + (M + Bnext) * d; e < Tn * d; e += kNT) {
      Xs[(pad + e / d) * sx + e % d] = 0.f;
      yv(e / d)[e % d] = 0.f;
    }
    m = M;
    Bn = Bnext;
  }
}

// ---- attention of every block of a window in one launch (Alg. 2 step 3): one wave per query row, four rows of
// a (block, head) per workgroup.  Scores: a lane per key; output: a lane per NC columns.
template <typename T, int NC>
__global__ __launch_bounds__(256) void attn_rows_k(AttnArgs a, int d, float* colsum, int ld) {
  extern __shared__ __align__(16) float sm[];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int rows4 = (a.B + 3) / 4, seg = a.seg_first + blockIdx.x / rows4, r = (blockIdx.x % rows4) * 4 + w;
  const int hq = blockIdx.y, b = blockIdx.z, hkv = hq / a.group, ch = b * a.Hkv + hkv;
  const int64_t tok0 = (int64_t)seg * a.B;
  const int Bn = (int)min((int64_t)a.B, a.L - tok0);
  if (r >= Bn) return;                               // no barrier below: waves are independent
  const bool base = seg <= a.n_fill;
  const int m = base ? a.len0 + seg * a.B : a.M, n_vis = m + r + 1;
  const int64_t hslot = base ? 0 : ((a.hist_first + (int64_t)(seg - a.n_fill - 1)) % a.hist_ring) * a.hist_stride;
  const T* ck = (base ? (const T*)a.cache_k : (const T*)a.hist_k + hslot) + (int64_t)ch * a.M * d;
  const T* cv = (base ? (const T*)a.cache_v : (const T*)a.hist_v + hslot) + (int64_t)ch * a.M * d;
  const T* kb = (const T*)a.k.p + b * a.k.sb + hkv * a.k.sh + tok0 * a.k.st;
  const T* vb = (const T*)a.v.p + b * a.v.sb + hkv * a.v.sh + tok0 * a.v.st;
  const T* q = (const T*)a.q.p + b * a.q.sb + hq * a.q.sh + (tok0 + r) * a.q.st;
  float* qs = sm + w * (d + ld);
  float* sc = qs + d;
  for (int c = l; c < d; c += 64) qs[c] = to_f(q[c]);
  wave_sync();
  float mx = -INFINITY;
  for (int j = l; j < n_vis; j += 64) {
    const T* kr = j < m ? ck + (int64_t)j * d : kb + (int64_t)(j - m) * a.k.st;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    int c = 0;
    for (; c + 4 <= d; c += 4) {
      s0 = fmaf(qs[c], to_f(kr[c]), s0);
      s1 = fmaf(qs[c + 1], to_f(kr[c + 1]), s1);
      s2 = fmaf(qs[c + 2], to_f(kr[c + 2]), s2);
      s3 = fmaf(qs[c + 3], to_f(kr[c + 3]), s3);
    }
    for (; c < d; ++c) s0 = fmaf(qs[c], to_f(kr[c]), s0);
    const float s = ((s0 + s1) + (s2 + s3)) * a.scale;
    sc[j] = s;
    mx = fmaxf(mx, s);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  float z = 0.f;
  for (int j = l; j < n_vis; j += 64) {
    const float e = expf(sc[j] - mx);
    sc[j] = e;
    z += e;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o, 64);
  wave_sync();
  if (colsum)                                        // accumulated attention per live cache slot
    for (int j = l; j < m; j += 64) atomicAdd(colsum + (int64_t)ch * a.M + j, sc[j] / z);
  T* o = (T*)a.o.p + b * a.o.sb + hq * a.o.sh + (tok0 + r) * a.o.st;
  const int mc = min(m, n_vis);
  int c[NC];
  float s0[NC], s1[NC];
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    c[n] = min(64 * n + l, d - 1);                   // (a column past d is not stored)
    s0[n] = s1[n] = 0.f;
  }
  int j = 0;
  for (; j + 4 <= mc; j += 4) {
    const float4 p = {sc[j], sc[j + 1], sc[j + 2], sc[j + 3]};
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      const T* vc = cv + (int64_t)j * d + c[n];
      s0[n] = fmaf(p.x, to_f(vc[0]), s0[n]);
      s1[n] = fmaf(p.y, to_f(vc[d]), s1[n]);
      s0[n] = fmaf(p.z, to_f(vc[2 * d]), s0[n]);
      s1[n] = fmaf(p.w, to_f(vc[3 * d]), s1[n]);
    }
  }
  for (; j < mc; ++j)
#pragma unroll
    for (int n = 0; n < NC; ++n) s0[n] = fmaf(sc[j], to_f(cv[(int64_t)j * d + c[n]]), s0[n]);
#pragma unroll 4
  for (; j < n_vis; ++j)
#pragma unroll
    for (int n = 0; n < NC; ++n) s1[n] = fmaf(sc[j], to_f(vb[(int64_t)(j - m) * a.v.st + c[n]]), s1[n]);
#pragma unroll
  for (int n = 0; n < NC; ++n)
    if (64 * n + l < d) (void)store_f((s0[n] + s1[n]) / z, o + c[n]);
}

constexpr int kRowsMaxT = 2048, kRowsMaxD = 128;

// taps resident at once with one slot tile per workgroup (0: the positions do not fit, or with the taps in chunks a wave
// would have more than one unit, whose sums it leaves in LDS between the chunks)
int taps_that_fit(int T, int d, int k, int conv_in) {
  if (2 * ((d + 15) / 16) > kNW * kMaxMix) return 0;
  for (int taps = k; taps >= 1; --taps) {
    if (taps < k && (T + 31) / 32 * planes_of((T + 31) / 32) > kNW) return 0;
    if (layout_of(T, d, k, conv_in, 1, taps).bytes <= kLds) return taps;
  }
  return 0;
}

template <typename T, int MIX, int D, int CIN>
hipError_t launch_d(const SmallArgs& g, int grid_x, hipStream_t s) {
  static bool attr_set = false;   // benign race: setting it twice is harmless
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)compress_small_k<T, MIX, D, CIN>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((compress_small_k<T, MIX, D, CIN>), dim3(grid_x, g.st.batch * g.st.Hkv), dim3(kNT), g.l.bytes, s, g);
  return hipGetLastError();
}
// A step of the smallest scans is a few hundred cycles of dependent work in each of its passes: indices that need a division by
// the head_dim or a product with a row stride are a good part of it, so the one these scans are used with has builds of its own.
template <typename T, int MIX>
hipError_t launch(const SmallArgs& g, int grid_x, hipStream_t s) {
  if (g.st.d != 64) return launch_d<T, MIX, 0, 0>(g, grid_x, s);
  return g.st.conv_in ? launch_d<T, MIX, 64, 1>(g, grid_x, s) : launch_d<T, MIX, 64, 0>(g, grid_x, s);
}

}  // namespace

// Decided for blocks of at least M tokens, so that a shorter (last) block runs on the same kernels as the others.
bool small_step_fits(int T, int M, int d, int k, int conv_in) { return taps_that_fit(std::max(T, 2 * M), d, k, conv_in) > 0; }

// All steps of a scan in one launch where one workgroup holds a whole chain: LDS, the registers of Eq. 4, and no more
// matrix work put on one compute unit per step than the launch it saves costs (12 000 cycles, about 5 us: the
// dispatch of a dependent kernel plus reading rows and filters back in).
bool small_scan_one_launch(int T, int M, int d, int k, int conv_in) {
  const int tiles = (M + 15) / 16, C4 = ((conv_in ? 2 * d : d) + 3) / 4;
  if (tiles * 2 * ((d + 15) / 16) > kNW * kMaxMix || layout_of(T, d, k, conv_in, tiles, k).bytes > kLds) return false;
  const int64_t cycles = (int64_t)tiles * ((T + 15) / 16) * C4 * k * 32 / 4;    // one 32-cycle MFMA per 4 channels, four SIMDs
  return cycles - cycles / tiles <= 12000;
}

hipError_t launch_compress_small(int dtype, const StepArgs& a, int T, int n_steps, int B, int64_t tokens_left, void* out_k,
                                 void* out_v, int64_t out_stride, int slot0, int ring, hipStream_t s) {
  SmallArgs g;
  g.st = a;
  g.n_steps = n_steps;
  g.B = B;
  g.tokens_left = tokens_left;
  g.out_k = out_k;
  g.out_v = out_v;
  g.out_stride = out_stride;
  g.slot0 = slot0;
  g.ring = ring;
  const int tiles = n_steps > 1 ? (a.M + 15) / 16 : 1;
  g.l = layout_of(T, a.d, a.k_width, a.conv_in, tiles, n_steps > 1 ? a.k_width : taps_that_fit(T, a.d, a.k_width, a.conv_in));
  const int grid_x = ((a.M + 15) / 16 + tiles - 1) / tiles;
  const bool f32 = dtype == LOCOCO_F32;
  if (tiles * 2 * ((a.d + 15) / 16) <= kNW) return f32 ? launch<float, 1>(g, grid_x, s) : launch<bf16_t, 1>(g, grid_x, s);
  return f32 ? launch<float, kMaxMix>(g, grid_x, s) : launch<bf16_t, kMaxMix>(g, grid_x, s);
}

// The walk over the values is a chain of latencies, one wave's alone, so it is made once, for at most two columns a lane.  One
// workgroup per row (attn_generic_k) is the better kernel for wider heads: 128 slots, one head, 16 tokens in fp32, with 64
// columns 11.5 us against 16.4, with 128 16.3 against 17.3 (21.2 in two walks), with 256 39.1 (four walks) against 19.9.
bool attn_rows_fits(int T, int d) { return T <= kRowsMaxT && d <= kRowsMaxD; }

hipError_t launch_attn_rows(int dtype, const AttnArgs& a, int d, float* colsum, hipStream_t s) {
  // the most positions a row can see: of a single block, its own (a large cache may have few live slots yet)
  const int ld = (a.n_seg == 1 ? a.len0 : a.M) + a.B;
  const size_t lds = (size_t)4 * (d + ld) * sizeof(float);
  const dim3 grid((unsigned)(a.n_seg * ((a.B + 3) / 4)), a.Hq, a.batch);
  auto go = [&](auto nc) {
    constexpr int NC = decltype(nc)::value;
    if (dtype == LOCOCO_F32) hipLaunchKernelGGL((attn_rows_k<float, NC>), grid, dim3(256), lds, s, a, d, colsum, ld);
    else hipLaunchKernelGGL((attn_rows_k<bf16_t, NC>), grid, dim3(256), lds, s, a, d, colsum, ld);
  };
  if (d <= 64) go(std::integral_constant<int, 1>{});
  else go(std::integral_constant<int, 2>{});
  return hipGetLastError();
}

}  // namespace lococo
