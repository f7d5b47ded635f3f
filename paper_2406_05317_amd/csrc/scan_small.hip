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
// block (63 us of each step in the 64 x 64-tiled Eq. 5, one workgroup), 104 us with compress_small_k at first, 71 us with its operand
// reads issued in groups ahead of their products and its reductions on the vector unit, 37 us with compress64_k in its place.
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
  int T;                  // the most positions of a step
  void* last_k; void* last_v;   // not null: where the last step writes its state, in place of its slot
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
        row[c] = v;
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
  // The last state goes to the caller as well, from the rows as they lie here.  (A choice of the place in the epilogue costs scalar
  // registers every step: 14 of them, 16 slots of 64, filters over [K | V], bf16, 76.5 -> 79.7 us.)
  if (g.n_steps > 1 && g.last_k) {
    __syncthreads();
    T* lk_ = (T*)g.last_k + (int64_t)ch * M * d;
    T* lv_ = (T*)g.last_v + (int64_t)ch * M * d;
    for (int e = tid; e < M * d; e += kNT) {
      const int j = e / d, c = e % d;
      store_f(Xs[(pad + j) * sx + c], lk_ + e);
      store_f(yv(j)[c], lv_ + e);
    }
  }
}

// ---- the same for single precision, head_dim 64 and filters over the keys.  Bound by the number of instructions its waves issue
// between the barriers of a step: one in some five cycles a wave, two waves to a SIMD.  So filters stay in registers in operand order
// (read once, through LDS in whole lines: from memory each lane's own touch 64 lines an instruction), operands are read 16 bytes a lane
// (four steps of the contraction, in an order both operands share), rows move four at a time, a row of Eq. 6 takes a lane as few
// positions as it has, and the four barriers of a step wait for LDS alone.  The 15 steps of the smallest scan (M = B = 16, width 3),
// in the general kernel and here: 61.3 and 29.3 us; by clock stamps 4 500 cycles a step here (970 Eq. 5, its products 770; 950 Eq. 6;
// 940 Eq. 4, its products 510).  A launch per step (8 tokens on 60 slots, width 5): 15.5 and 7.2 us, half of it before the first product;
// 22 on 95, width 9: 23.6 and 11.3, four of them products of Eq. 5.
constexpr int k64 = 64, kSx = 68;            // head_dim; row stride of X and V: 16 rows x 4 columns on 64 banks
constexpr int kPF64 = 6;                     // items of the next block a wave fetches ahead: 96 rows in all
constexpr int kParts = 4, kPosGroups = 2;    // a wave: a quarter of the channels, every second tile of 16 positions
static_assert(kParts * kPosGroups == kNW, "eight waves");
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_any;

struct Layout64 { int sl, off_v, off_l, bytes; };
__host__ __device__ inline Layout64 layout64_of(int T, int k, int tiles) {
  const int n16 = (T + 15) / 16;
  Layout64 l;
  l.sl = odd4(16 * n16);
  l.off_v = (16 * n16 + k - 1) * kSx;
  l.off_l = l.off_v + 16 * n16 * kSx;
  // (a slot tile's filters pass through on their way into the registers: rows of 64 k + 4)
  const int words = l.off_l + kParts * tiles * 16 * l.sl, filters = 16 * (k64 * k + 4);
  l.bytes = (words > filters ? words : filters) * 4;
  return l;
}

// every wave's LDS accesses are done (loads and stores of global memory may be on their way)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One workgroup: 16 TL slots of one chain.  n_steps > 1 only where those are all slots of the chain.  KW: filter width; SOFT: Eq. 6
// as a softmax (norm 0).
template <int KW, int TL, bool SOFT>
__global__ __launch_bounds__(kNT) void compress64_k(SmallArgs g) {
  extern __shared__ __align__(16) float sm[];
  const StepArgs& a = g.st;
  const int M = a.M, tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l15 = l & 15, lk = l >> 4;
  const Layout64 L = layout64_of(g.T, KW, TL);
  float* Xs = sm;
  float* Vs = sm + L.off_v;
  float* Ls = sm + L.off_l;
  constexpr int pad = (KW - 1) / 2;
  const int sl = L.sl, plane = TL * 16 * sl, ch = blockIdx.y, b = ch / a.Hkv, hkv = ch % a.Hkv, i0 = blockIdx.x * 16 * TL;
  const int part = w & 3, pg = w >> 2;
  const uint32_t* protect = a.protect ? a.protect + (int64_t)ch * a.protect_stride : nullptr;

  // Rows come four at a time, 16 bytes a lane: item u of a set of rows is rows 4 (u / 2) .. of the keys (u even) or the values.
  // Of the first state and the first block, the first eight items of a wave are asked for ahead of the filters.
  const float* kb = (const float*)a.k.p + b * a.k.sb + hkv * a.k.sh;
  const float* vb = (const float*)a.v.p + b * a.v.sb + hkv * a.v.sh;
  const int lr = l >> 4, lc = (l & 15) * 4;
  int m = a.m, Tn = m + a.Bn, n16 = (Tn + 15) / 16;
  f32x4 x8[8];
  auto request = [&](int u0) {
    const float* ck = (const float*)a.cache_k + (int64_t)ch * M * k64;
    const float* cv = (const float*)a.cache_v + (int64_t)ch * M * k64;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int u = u0 + n * kNW, j = min((u >> 1) * 4 + lr, Tn - 1);
      if ((u >> 1) * 4 >= Tn) break;
      const float* in_cache = (u & 1 ? cv : ck) + j * k64;
      const float* in_block = (u & 1 ? vb : kb) + (int64_t)(j - m) * (u & 1 ? a.v.st : a.k.st);
      x8[n] = *(const f32x4_any*)((j < m ? in_cache : in_block) + lc);
    }
  };
  auto place = [&](int u0) {
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int u = u0 + n * kNW, j = (u >> 1) * 4 + lr;
      if (j < Tn) *(f32x4*)((u & 1 ? Vs : Xs + pad * kSx) + j * kSx + lc) = x8[n];
    }
  };
  request(w);
  // this lane's filters: slot l15 of each tile, channels 16 part + 4 lk ..: consecutive in memory, [slot][channel][tap].  They come
  // in whole lines, through LDS (straight from memory a load touches 64 lines)
  float fw[TL][KW][4];
#pragma unroll
  for (int st = 0; st < TL; ++st) {
    const int s0 = i0 + st * 16, have = min(16, M - s0) * k64 * KW;      // floats of live slots (a multiple of 4)
    const float* p = (const float*)a.conv_w + hkv * a.w_head_stride + (int64_t)s0 * k64 * KW;
    constexpr int N = 16 * k64 * KW / 4, PER = (N + kNT - 1) / kNT;      // chunks of 16 bytes
    f32x4 f[PER];
#pragma unroll
    for (int n = 0; n < PER; ++n) {
      const int e = (tid + n * kNT) * 4;
      f[n] = e < have ? *(const f32x4_any*)(p + e) : f32x4_any{0.f, 0.f, 0.f, 0.f};
    }
    if (st) lds_barrier();
#pragma unroll
    for (int n = 0; n < PER; ++n) {
      const int e = (tid + n * kNT) * 4, row = e / (k64 * KW);
      if (row < 16) *(f32x4*)(sm + e + row * 4) = f[n];
    }
    lds_barrier();
    const float* q = sm + l15 * (k64 * KW + 4) + (part * 16 + lk * 4) * KW;
#pragma unroll
    for (int n = 0; n < KW; ++n) {
      const f32x4 v = *(const f32x4*)(q + 4 * n);
#pragma unroll
      for (int e = 0; e < 4; ++e) fw[st][(4 * n + e) % KW][(4 * n + e) / KW] = v[e];
    }
  }
  lds_barrier();
  place(w);
  for (int u0 = w + 8 * kNW; (u0 >> 1) * 4 < Tn; u0 += 8 * kNW) {
    request(u0);
    place(u0);
  }
  for (int r = w; r < pad; r += kNW) Xs[r * kSx + l] = 0.f;              // zeros around them
  for (int r = Tn + w; r < 16 * n16 + KW - 1 - pad; r += kNW) {
    Xs[(pad + r) * kSx + l] = 0.f;
    if (r < 16 * n16) Vs[r * kSx + l] = 0.f;
  }

  const bool val = w >= 4;                   // Eq. 4: wave w the columns 16 w .. of [K | V]
  const int col = (w & 3) * 16 + l15;
  float* const rows = val ? Vs + col : Xs + pad * kSx + col;             // row j, this lane's column: + j * kSx
  const int64_t mine = ((int64_t)ch * M + i0 + lk * 4) * k64 + col;      // of a state: this lane's first element
  // where this lane's first rows of a block come from (items w, w + 8, ..: all of one array) and go to
  const int64_t st = w & 1 ? a.v.st : a.k.st;
  const float* from = (w & 1 ? vb : kb) + (g.B + (w >> 1) * 4 + lr) * st + lc;
  float* const to = (w & 1 ? Vs : Xs + pad * kSx) + (M + (w >> 1) * 4 + lr) * kSx + lc;
  const int Blast = (int)min((int64_t)g.B, g.tokens_left - (g.n_steps - 1) * (int64_t)g.B);
  const bool whole = i0 + 16 * TL <= M;                                  // every slot is a live one
  int slot = g.slot0;
  for (int step = 0;; ++step) {
    const bool more = step + 1 < g.n_steps;
    const int Bnext = step + 2 < g.n_steps ? g.B : more ? Blast : 0;
    // the next block's first rows, in flight under this step
    f32x4 ahead[kPF64];
    if (more) {
      const int r0 = (w >> 1) * 4;
#pragma unroll
      for (int n = 0; n < kPF64; ++n) {
        if (r0 + 16 * n >= Bnext) break;
        ahead[n] = *(const f32x4_any*)(from + min(16 * n, Bnext - 1 - r0 - lr) * st);
      }
    }
    lds_barrier();
    // ---- Eq. 5: positions x slots (A: 16 positions x 16 channels at a tap's row shift, B: filters)
    auto conv = [&](auto rect) {
      for (int pt = pg; pt < n16; pt += kPosGroups) {
        f32x4 acc[TL][2];                    // (two chains of products)
#pragma unroll
        for (int st = 0; st < TL; ++st) acc[st][0] = acc[st][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        const float* xb = Xs + (pt * 16 + l15) * kSx + part * 16 + lk * 4;
#pragma unroll
        for (int t = 0; t < KW; ++t) {
          f32x4 x = *(const f32x4*)(xb + t * kSx);
          if (decltype(rect)::value)         // the rectifier in front of the convolution
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = fmaxf(x[q], 0.f);
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int st = 0; st < TL; ++st)
              acc[st][q & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q], fw[st][t][q], acc[st][q & 1], 0, 0, 0);
        }
        float* out = Ls + part * plane + l15 * sl + pt * 16 + 4 * lk;
#pragma unroll
        for (int st = 0; st < TL; ++st) *(f32x4*)(out + st * 16 * sl) = acc[st][0] + acc[st][1];
      }
    };
    if (!SOFT && a.norm == 2) conv(std::true_type{});
    else conv(std::false_type{});
    lds_barrier();
    // ---- Eq. 6: 32 lanes per slot, N positions a lane (and as many 128 positions on): a wave issues each instruction for all of
    // its lanes, so short rows take no more of them than they have positions for
    auto normalise = [&](auto width, auto halves) {
      constexpr int N = decltype(width)::value, H = decltype(halves)::value;
      typedef __attribute__((ext_vector_type(N))) float fx;
      const int c = (tid & 31) * N, row = tid >> 5, last = 16 * n16 - N;
      fx x[TL][H];
      float mx[TL], z[TL];
#pragma unroll
      for (int st = 0; st < TL; ++st) {
        const float* r = Ls + (st * 16 + row) * sl;
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const float* p = r + min(c + 128 * h, last);
          x[st][h] = (*(const fx*)p + *(const fx*)(p + plane)) + (*(const fx*)(p + 2 * plane) + *(const fx*)(p + 3 * plane));
        }
      }
      if (a.conv_b)
#pragma unroll
        for (int st = 0; st < TL; ++st) {
          const int i = i0 + st * 16 + row;
          const float bi = i < M ? ((const float*)a.conv_b)[hkv * a.b_head_stride + i] : 0.f;
#pragma unroll
          for (int h = 0; h < H; ++h) x[st][h] += bi;
        }
      constexpr float none = SOFT ? -INFINITY : 0.f;       // a protected slot's position
      if (protect)
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const int j0 = c + 128 * h;                      // (N divides 32: one word)
          const uint32_t bits = j0 < m ? protect[j0 >> 5] >> (j0 & 31) : 0;
#pragma unroll
          for (int e = 0; e < N; ++e)
#pragma unroll
            for (int st = 0; st < TL; ++st) x[st][h][e] = j0 + e < m && ((bits >> e) & 1u) ? none : x[st][h][e];
        }
      bool in[H][N];                                       // past T: zero, whatever the sum
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int e = 0; e < N; ++e) in[h][e] = c + 128 * h + e < Tn;
#pragma unroll
      for (int st = 0; st < TL; ++st)
        if (SOFT) {
          mx[st] = -INFINITY;
#pragma unroll
          for (int h = 0; h < H; ++h)
#pragma unroll
            for (int e = 0; e < N; ++e) mx[st] = fmaxf(mx[st], in[h][e] ? x[st][h][e] : -INFINITY);
          mx[st] = over32(mx[st], [](float p, float q) { return fmaxf(p, q); });
        }
#pragma unroll
      for (int st = 0; st < TL; ++st) {
        z[st] = 0.f;
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
          for (int e = 0; e < N; ++e) {
            const float y = x[st][h][e];
            const float v = SOFT ? expf(y - mx[st]) : a.norm == 1 ? fmaxf(y, 0.f) : (isfinite(y) ? y : 0.f);
            x[st][h][e] = in[h][e] ? v : 0.f;
            z[st] += x[st][h][e];
          }
      }
#pragma unroll
      for (int st = 0; st < TL; ++st) {
        z[st] = over32(z[st], [](float p, float q) { return p + q; });
        if (!SOFT && a.norm == 1) z[st] += a.eps;
        if (!SOFT && a.norm == 2 && fabsf(z[st]) < a.eps) z[st] = z[st] < 0.f ? -a.eps : a.eps;
#pragma unroll
        for (int h = 0; h < H; ++h) {
          fx v;
#pragma unroll
          for (int e = 0; e < N; ++e) v[e] = in[h][e] ? x[st][h][e] / z[st] : 0.f;
          if (c + 128 * h <= last) *(fx*)(Ls + (st * 16 + row) * sl + c + 128 * h) = v;
        }
      }
    };
    using std::integral_constant;
    if (n16 <= 2) normalise(integral_constant<int, 1>{}, integral_constant<int, 1>{});
    else if (n16 <= 4) normalise(integral_constant<int, 2>{}, integral_constant<int, 1>{});
    else if (n16 <= 8) normalise(integral_constant<int, 4>{}, integral_constant<int, 1>{});
    else normalise(integral_constant<int, 4>{}, integral_constant<int, 2>{});
    lds_barrier();
    // ---- Eq. 4a / 4b: slots x 16 columns (A: weights of 16 positions, B: their rows)
    f32x4 acc[TL][2];
    {
#pragma unroll
      for (int st = 0; st < TL; ++st) acc[st][0] = acc[st][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      const float* wr = Ls + l15 * sl + 4 * lk;
      const float* yr = rows + 4 * lk * kSx;
      auto some = [&](auto count) {          // COUNT tiles of 16 positions in flight together
        constexpr int COUNT = decltype(count)::value;
        float y[COUNT][4];
        f32x4 x[COUNT][TL];
#pragma unroll
        for (int n = 0; n < COUNT; ++n) {
#pragma unroll
          for (int q = 0; q < 4; ++q) y[n][q] = yr[(16 * n + q) * kSx];
#pragma unroll
          for (int st = 0; st < TL; ++st) x[n][st] = *(const f32x4*)(wr + 16 * n + st * 16 * sl);
        }
        wr += 16 * COUNT;
        yr += 16 * COUNT * kSx;
#pragma unroll
        for (int n = 0; n < COUNT; ++n)
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int st = 0; st < TL; ++st)
              acc[st][q & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[n][st][q], y[n][q], acc[st][q & 1], 0, 0, 0);
      };
      int p = 0;
#pragma clang loop unroll(disable)
      for (; p + 2 <= n16; p += 2) some(std::integral_constant<int, 2>{});
      if (p < n16) some(std::integral_constant<int, 1>{});
    }
    lds_barrier();                           // every read of the old rows is done
    float* const out = (!more && g.last_k ? (float*)(val ? g.last_v : g.last_k) : (float*)(val ? g.out_v : g.out_k) + (int64_t)slot * g.out_stride) + mine;
    if (++slot == g.ring) slot = 0;
#pragma unroll
    for (int st = 0; st < TL; ++st) {
      f32x4 v = acc[st][0] + acc[st][1];
      const int i = i0 + st * 16 + lk * 4;   // rows i .. i + 3
      if (protect)                           // a live protected slot is carried over unchanged
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i + e < m && ((protect[(i + e) >> 5] >> ((i + e) & 31)) & 1u)) v[e] = rows[(i + e) * kSx];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (whole || i + e < M) {
          out[(st * 16 + e) * k64] = v[e];
          rows[(i + e) * kSx] = v[e];
        }
    }
    if (!more) break;
    // ---- the next block behind the new cache; zeros up to the end of what this step's rows used
    {
      const int r0 = (w >> 1) * 4 + lr;
#pragma unroll
      for (int n = 0; n < kPF64; ++n) {
        if ((w >> 1) * 4 + 16 * n >= Bnext) break;
        if (r0 + 16 * n < Bnext) *(f32x4*)(to + 16 * n * kSx) = ahead[n];
      }
      for (int r = r0 + 16 * kPF64; r < Bnext; r += 16) *(f32x4*)(to + (r - r0) * kSx) = *(const f32x4_any*)(from + (r - r0) * st);
    }
    // (a first step of fewer live slots may be the shorter one: what a longer one reads beyond it is zeroed here as well)
    const int Tnext = M + Bnext;
    if (Tnext != Tn) {
      const int end = 16 * max(n16, (Tnext + 15) / 16);
      for (int r = Tnext + w; r < end + KW - 1 - pad; r += kNW) {
        Xs[(pad + r) * kSx + l] = 0.f;
        if (r < end) Vs[r * kSx + l] = 0.f;
      }
      Tn = Tnext;
      n16 = (Tn + 15) / 16;
    }
    m = M;
    from += g.B * st;
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

// Slot tiles a workgroup of compress64_k holds the filters and sums of without vector registers in scratch memory (with three, or norms 1
// and 2, up to 20 scalar ones lie in lanes of vector registers)
constexpr int tiles64(int k) { return k <= 5 ? 3 : k <= 11 ? 2 : 1; }
// whether compress64_k has a build for this width (every odd one from 3 to 15, and 21, the widest a workload here has; others are
// compress_small_k's) and the positions fit with `tiles` slot tiles to a workgroup
bool fits64(int dtype, int T, int d, int k, int conv_in, int tiles) {
  return dtype == LOCOCO_F32 && d == k64 && !conv_in && k >= 3 && (k <= 15 || k == 21) && tiles <= tiles64(k) && T <= 256 &&
         layout64_of(T, k, tiles).bytes <= kLds;
}

template <int KW, int TL, bool SOFT>
hipError_t launch64_as(const SmallArgs& g, int grid_x, hipStream_t s) {
  static bool attr_set = false;   // benign race: setting it twice is harmless
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)compress64_k<KW, TL, SOFT>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((compress64_k<KW, TL, SOFT>), dim3(grid_x, g.st.batch * g.st.Hkv), dim3(kNT), layout64_of(g.T, KW, TL).bytes, s, g);
  return hipGetLastError();
}
template <int KW, bool SOFT>
hipError_t launch64_tiles(const SmallArgs& g, int tiles, int grid_x, hipStream_t s) {
  if constexpr (tiles64(KW) >= 3) if (tiles == 3) return launch64_as<KW, 3, SOFT>(g, grid_x, s);
  if constexpr (tiles64(KW) >= 2) if (tiles == 2) return launch64_as<KW, 2, SOFT>(g, grid_x, s);
  return tiles == 1 ? launch64_as<KW, 1, SOFT>(g, grid_x, s) : hipErrorInvalidValue;
}
template <bool SOFT>
hipError_t launch64(const SmallArgs& g, int tiles, int grid_x, hipStream_t s) {
  switch (g.st.k_width) {
    case 3: return launch64_tiles<3, SOFT>(g, tiles, grid_x, s);
    case 5: return launch64_tiles<5, SOFT>(g, tiles, grid_x, s);
    case 7: return launch64_tiles<7, SOFT>(g, tiles, grid_x, s);
    case 9: return launch64_tiles<9, SOFT>(g, tiles, grid_x, s);
    case 11: return launch64_tiles<11, SOFT>(g, tiles, grid_x, s);
    case 13: return launch64_tiles<13, SOFT>(g, tiles, grid_x, s);
    case 15: return launch64_tiles<15, SOFT>(g, tiles, grid_x, s);
    case 21: return launch64_tiles<21, SOFT>(g, tiles, grid_x, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Decided for blocks of at least M tokens, so that a shorter (last) block runs on the same kernels as the others.
bool small_step_fits(int T, int M, int d, int k, int conv_in) { return taps_that_fit(std::max(T, 2 * M), d, k, conv_in) > 0; }

// All steps of a scan in one launch where one workgroup holds a whole chain: LDS, the registers of Eq. 4 (or of the filters), and no
// more matrix work put on one compute unit per step than the launch it saves costs (12 000 cycles, about 5 us: the
// dispatch of a dependent kernel plus reading rows and filters back in; compress64_k, 8 tokens on 28 slots, width 5, 1 900 cycles more
// by this count: 4.2 us a step, in a launch of its own 5.6 and the way from one to the next).
bool small_scan_one_launch(int dtype, int T, int M, int d, int k, int conv_in) {
  const int tiles = (M + 15) / 16, C4 = ((conv_in ? 2 * d : d) + 3) / 4;
  if (fits64(dtype, std::max(T, 2 * M), d, k, conv_in, 1)) {     // (decided like small_step_fits: a step is the same bits in either form)
    const int64_t cycles = (int64_t)tiles * ((T + 15) / 16) * 16 * k * 32 / 4;
    return fits64(dtype, std::max(T, 2 * M), d, k, conv_in, tiles) && cycles - cycles / tiles <= 12000;
  }
  if (tiles * 2 * ((d + 15) / 16) > kNW * kMaxMix || layout_of(T, d, k, conv_in, tiles, k).bytes > kLds) return false;
  const int64_t cycles = (int64_t)tiles * ((T + 15) / 16) * C4 * k * 32 / 4;    // one 32-cycle MFMA per 4 channels, four SIMDs
  return cycles - cycles / tiles <= 12000;
}

hipError_t launch_compress_small(int dtype, const StepArgs& a, int T, int n_steps, int B, int64_t tokens_left, void* out_k,
                                 void* out_v, int64_t out_stride, int slot0, int ring, hipStream_t s, void* last_k, void* last_v) {
  SmallArgs g;
  if (n_steps == 1 && last_k) {              // (a step in a launch of its own: where it goes is where it writes)
    out_k = last_k;
    out_v = last_v;
    slot0 = 0;
  }
  g.last_k = last_k;
  g.last_v = last_v;
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
  g.T = std::max(T, 2 * a.M);
  if (fits64(dtype, g.T, a.d, a.k_width, a.conv_in, 1)) {
    const int grid64 = ((a.M + 15) / 16 + tiles - 1) / tiles;
    return a.norm == 0 ? launch64<true>(g, tiles, grid64, s) : launch64<false>(g, tiles, grid64, s);
  }
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
