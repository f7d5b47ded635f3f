// Backward of the attention of every block of a window (Alg. 2 step 3), two kernels, bf16 MFMA, head_dim 128.
//
// Nothing of size queries x keys goes through memory: both kernels recompute the score tiles.
//   bwd_attn_q_k    a workgroup per 128 query rows: one walk over the keys for the row statistics (softmax reference,
//                   1 / row sum) and D = sum_j P dP, a second one for dq = dS Yk.  Leaves dO as two bf16 halves and the
//                   statistics for
//   bwd_attn_kv_k   a workgroup per 128 keys of [cache ; block]: dYk = dS^T q and dYv = P^T dO over the rows of all
//                   heads of the group.
// The fp32 operands (dO, P, dS) enter the matrix products as two bf16 halves (16 bits kept): S 1, dP 2, dq 2, dYk 2,
// dYv 3 products; with the recomputation 15 products per (query, key) pair of 128 columns.  A block whose number of
// positions is no multiple of 4, or a step whose gradients are not 16-byte aligned, enters with three parts (24 bits, nothing
// lost; dP, dq, dYk 3, dYv 6 products): those have always been computed in fp32, and errors stay at that level (3e-7 against
// 3.5e-6 with two).
// Measured, 64 blocks of 512 queries on 1024 keys, 32 heads: 5.3 ms for the whole sequence (2.1 + 3.3) against 20.0 ms as
// seven batched products and a row kernel per block with P, dS in fp32 in memory; 28 blocks of 128 on 256: 0.27 against
// 3.0 ms (launches of 15 - 23 us each that did not fill the chip).  Bound by the issue of the vector and LDS instructions
// between the products (matrix pipe 45 % busy in the first kernel, 30 % in the second).  Operands read ahead of their products,
// fragments waited for before the loops and a loop of its own for either kind of wave (no spills, whose reloads waited for
// the tiles just requested): 12 blocks of 256 queries on 512 keys, 2 x 32 heads on 8: 226 -> 216 and 339 -> 279 us.
// D is taken from P and dP, not from dO . O: the stored outputs are bf16 and would cost dS half its bits.
#include <type_traits>

#include "lococo_internal.h"
#include "mfma_util.h"

namespace lococo {
namespace {

constexpr int kD = 128;
constexpr int kTile = 64 * kD * 2;            // bytes of a tile of 64 rows
constexpr int kOrow = 3 * kD;                 // elements of a row of dO's parts in memory

struct Seg {
  const uint16_t* ck; const uint16_t* cv;     // the chain's cache rows
  int64_t start;                              // first token of the block (in the window)
  int m, Bn;
};
__device__ __forceinline__ Seg segment(const AttnArgs& a, int n, int chain) {
  Seg s;
  s.start = (int64_t)n * a.B;
  s.Bn = (int)(a.L - s.start < a.B ? a.L - s.start : a.B);
  const bool base = n <= a.n_fill;
  s.m = base ? a.len0 + n * a.B : a.M;
  const int64_t slot = base ? 0 : (int64_t)((a.hist_first + n - a.n_fill - 1) % a.hist_ring) * a.hist_stride;
  s.ck = (const uint16_t*)(base ? a.cache_k : a.hist_k) + slot + (int64_t)chain * a.M * kD;
  s.cv = (const uint16_t*)(base ? a.cache_v : a.hist_v) + slot + (int64_t)chain * a.M * kD;
  return s;
}
__device__ __forceinline__ u32x4 rows_rsrc(const void* p, int n, int64_t st_bytes) {
  return make_rsrc(p, n > 0 ? (uint32_t)((n - 1) * st_bytes + 256) : 0u);
}

// requests rows row0 .. row0 + 63 of 256 bytes (st bytes apart in memory, `off` bytes into each) into the tile at lds;
// W waves share the 16 instructions
template <int W>
__device__ __forceinline__ void request_tile(const u32x4& rsrc, uint32_t st, uint32_t row0, uint32_t lds, int w, int l) {
#pragma unroll
  for (int i = 0; i < 16 / W; ++i) {
    const int r4 = w * (16 / W) + i, r = r4 * 4 + (l >> 4);
    load_to_lds(rsrc, lds + r4 * 1024, (row0 + r) * st + (((l & 15) ^ swz(r)) << 4));
  }
}

// Fragments loaded ahead of a loop have arrived here.  (Or the compiler counts them as possibly on their way in every pass of
// the loop and waits for the tiles requested a moment ago instead: a trip to memory per tile.)
__device__ __forceinline__ void landed(bf16x8 (&f)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(f[i]));
}

template <int PARTS>
__global__ __launch_bounds__(256, PARTS == 2 ? 2 : 1) void bwd_attn_q_k(BwdAttnArgs g) {
  extern __shared__ __align__(16) unsigned char smem[];
  const AttnArgs& a = g.a;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)smem);
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int qt = item % a.qtiles, hq = (item / a.qtiles) % a.Hq, b = (item / a.qtiles / a.Hq) % a.batch;
  const int n = a.seg_first + item / a.qtiles / a.Hq / a.batch, hkv = hq / a.group, chain = b * a.Hkv + hkv, q0 = qt * 128;
  const Seg s = segment(a, n, chain);
  if (q0 >= s.Bn) return;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l31 = l & 31, lh = l >> 5;
  const int wq0 = q0 + 32 * w, qrow = wq0 + l31;
  const u32x4 rck = rows_rsrc(s.ck, s.m, 256), rcv = rows_rsrc(s.cv, s.m, 256);
  const u32x4 rbk = rows_rsrc((const uint16_t*)a.k.p + b * a.k.sb + hkv * a.k.sh + s.start * a.k.st, s.Bn, a.k.st * 2);
  const u32x4 rbv = rows_rsrc((const uint16_t*)a.v.p + b * a.v.sb + hkv * a.v.sh + s.start * a.v.st, s.Bn, a.v.st * 2);
  const int NTc = (s.m + 63) / 64, NT = NTc + (min(s.Bn, q0 + 128) + 63) / 64;
  // tile t of the walk into buffer pair t % 2 (the walk is made twice: tile t % NT)
  auto request = [&](int t) {
    if (t >= 2 * NT) return;
    const uint32_t lds = lds0 + (t & 1) * 2 * kTile;
    const int tt = t < NT ? t : t - NT;
    if (tt < NTc) {
      request_tile<4>(rck, 256, tt * 64, lds, w, l);
      request_tile<4>(rcv, 256, tt * 64, lds + kTile, w, l);
    } else {
      request_tile<4>(rbk, (uint32_t)(a.k.st * 2), (tt - NTc) * 64, lds, w, l);
      request_tile<4>(rbv, (uint32_t)(a.v.st * 2), (tt - NTc) * 64, lds + kTile, w, l);
    }
  };
  request(0);

  // ---- this lane's query and output-gradient row as operand fragments; dO also goes to memory as two halves
  const int row = min(qrow, s.Bn - 1);
  const bool live = qrow < s.Bn;
  bf16x8 fq[8], fo[8][PARTS];
  {
    const uint16_t* qp = (const uint16_t*)a.q.p + b * a.q.sb + hq * a.q.sh + (s.start + row) * a.q.st + lh * 8;
    const float* op = g.d_o + b * g.q_sb + hq * g.q_sh + (s.start + row) * kD + lh * 8;
    uint16_t* hl = g.do_hl + (((int64_t)b * a.Hq + hq) * a.L + s.start + row) * kOrow + lh * 8;
    f32x4 o0[8], o1[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      fq[ks] = *(const bf16x8*)(qp + ks * 16);
      o0[ks] = *(const f32x4_any*)(op + ks * 16);
      o1[ks] = *(const f32x4_any*)(op + ks * 16 + 4);
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const float x[8] = {o0[ks][0], o0[ks][1], o0[ks][2], o0[ks][3], o1[ks][0], o1[ks][1], o1[ks][2], o1[ks][3]};
      split_parts<PARTS>(x, fo[ks]);
      if (live)
#pragma unroll
        for (int p = 0; p < PARTS; ++p) *(bf16x8*)(hl + p * kD + ks * 16) = fo[ks][p];
    }
  }
  TileAddr ad;
  tile_addr(l, ad);
  const float c = a.scale * kLog2e, lazy_raw = 8.0f / a.scale;
  wait_loads<0>();
  landed(fq);
  __syncthreads();

  // S^T and dP^T (32 keys x this wave's queries) of half kt of the tile at K / K + kTile
  auto products = [&](const unsigned char* K, int kt, f32x16& sc, f32x16& dp) {
    const unsigned char* k0 = K + kt * 32 * 256;
    sc = zero16();
    dp = zero16();
    // (two steps' operands ahead of their products)
    bf16x8 fk[3], fv[3];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      fk[ks] = *(const bf16x8*)(k0 + ad.row[ks]);
      fv[ks] = *(const bf16x8*)(k0 + kTile + ad.row[ks]);
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      if (ks + 2 < 8) {
        fk[(ks + 2) % 3] = *(const bf16x8*)(k0 + ad.row[ks + 2]);
        fv[(ks + 2) % 3] = *(const bf16x8*)(k0 + kTile + ad.row[ks + 2]);
      }
      __builtin_amdgcn_sched_barrier(0);
      sc = mfma32(fk[ks % 3], fq[ks], sc);
#pragma unroll
      for (int p = 0; p < PARTS; ++p) dp = mfma32(fv[ks % 3], fo[ks][p], dp);
    }
  };
  // keys this lane's query does not see: score -inf, and no part in anything however bad their values are
  auto mask = [&](int t, int kt, f32x16& sc, f32x16& dp) {
    const bool blk = t >= NTc;
    const int row0 = (blk ? t - NTc : t) * 64 + kt * 32;
    if (blk ? row0 + 31 > wq0 : row0 + 32 > s.m) {
      const int lim = blk ? qrow : s.m - 1;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (row0 + (i >> 2) * 8 + lh * 4 + (i & 3) > lim) { sc[i] = -INFINITY; dp[i] = 0.f; }
    }
  };
  auto visible = [&](int t, int kt) {       // uniform: some query of this wave sees a key of this half tile
    if (t < NTc) return t * 64 + kt * 32 < s.m;
    return (t - NTc) * 64 + kt * 32 < wq0 + 32;
  };

  // ---- first walk: reference m_run (lags the maximum by at most 8), row sum and sum of p dP
  float m_run = -INFINITY, l_run = 0.f, d_run = 0.f;
  for (int t = 0; t < NT; ++t) {
    request(t + 1);
    const unsigned char* K = smem + (t & 1) * 2 * kTile;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      if (!visible(t, kt)) continue;
      f32x16 sc, dp;
      products(K, kt, sc, dp);
      mask(t, kt, sc, dp);
      float mx = sc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sc[i]);
      mx = max_halves(mx);
      if (mx > m_run + lazy_raw) {
        const float alpha = __builtin_amdgcn_exp2f((m_run - mx) * c);
        l_run *= alpha;
        d_run *= alpha;
        m_run = mx;
      }
      const float mc = m_run * c;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sc[i], c, -mc));
        l_run += p;
        d_run = fmaf(p, dp[i], d_run);
      }
    }
    wait_loads<0>();
    __syncthreads();
  }
  const float inv = 1.0f / sum_halves(l_run), D = sum_halves(d_run) * inv, mc = m_run * c;
  if (live && lh == 0) {
    float* st = g.stats + ((int64_t)b * a.Hq + hq) * a.L + s.start + qrow;
    const int64_t plane = (int64_t)a.batch * a.Hq * a.L;
    st[0] = mc;
    st[plane] = inv;
    st[2 * plane] = D;
  }
  // ---- second walk: dq^T += Yk^T dS^T
  f32x16 acc[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = zero16();
  const float ps = inv * a.scale;
  for (int t = 0; t < NT; ++t) {
    request(NT + t + 1);
    const unsigned char* K = smem + ((NT + t) & 1) * 2 * kTile;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      if (!visible(t, kt)) continue;
      f32x16 sc, dp;
      products(K, kt, sc, dp);
      mask(t, kt, sc, dp);
      float ds[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) ds[i] = __builtin_amdgcn_exp2f(fmaf(sc[i], c, -mc)) * ps * (dp[i] - D);
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        bf16x8 fd[PARTS];
        split_parts<PARTS>(ds + 8 * s2, fd);
        const unsigned char* k0 = K + (kt * 32 + s2 * 16) * 256;
        bf16x8 fk[4];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) fk[ct] = frag_tr(k0 + ad.tr[ct][0], k0 + ad.tr[ct][1]);
#pragma unroll
        for (int p = 0; p < PARTS; ++p)
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) acc[ct] = mfma32(fk[ct], fd[p], acc[ct]);
      }
    }
    wait_loads<0>();
    __syncthreads();
  }
  if (live) {
    float* out = g.d_q + b * g.q_sb + hq * g.q_sh + (s.start + qrow) * kD + lh * 4;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int gi = 0; gi < 4; ++gi)
        *(f32x4_any*)(out + ct * 32 + gi * 8) = f32x4{acc[ct][gi * 4], acc[ct][gi * 4 + 1], acc[ct][gi * 4 + 2], acc[ct][gi * 4 + 3]};
  }
}

// Eight waves, two per group of 32 keys: waves 0..3 accumulate dYv (S, P^T dO), waves 4..7 dYk (S, dP, dS^T q).  One wave
// with both would hold 384 registers of accumulators and key / value fragments; split, a wave needs under 256, each SIMD
// has one of either kind to interleave, and the price is S computed twice (72 products instead of 64 per 32 x 32 tile).
template <int PARTS>
__global__ __launch_bounds__(512, 1) void bwd_attn_kv_k(BwdAttnArgs g) {
  constexpr int kSet = 1 + PARTS;
  extern __shared__ __align__(16) unsigned char smem[];       // [2][q | parts of dO] tiles of 64 rows, [2][3][64] statistics
  const AttnArgs& a = g.a;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)smem);
  float* st_lds = (float*)(smem + 2 * kSet * kTile);
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int ktiles = (a.M + a.B + 127) / 128;
  const int chain = (item / ktiles) % (a.batch * a.Hkv), n = a.seg_first + item / ktiles / (a.batch * a.Hkv);
  const int b = chain / a.Hkv, hkv = chain % a.Hkv, j0 = (item % ktiles) * 128;
  const Seg s = segment(a, n, chain);
  const int Tn = s.m + s.Bn;
  if (j0 >= Tn) return;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l31 = l & 31, lh = l >> 5;
  const int wj = j0 + 32 * (w & 3), j = wj + l31;             // this lane's position in [cache ; block]
  const int first = j0 >= s.m ? (j0 - s.m) / 64 : 0;          // tiles of rows before it see none of the keys
  const int rtiles = (s.Bn + 63) / 64 - first, N = a.group * rtiles;
  const int64_t plane = (int64_t)a.batch * a.Hq * a.L;

  float stat = 0.f;
  auto request = [&](int it) {
    if (it >= N) return;
    const int hq = hkv * a.group + it / rtiles, r0 = (first + it % rtiles) * 64;
    const uint32_t lds = lds0 + (it & 1) * kSet * kTile;
    const u32x4 rq = rows_rsrc((const uint16_t*)a.q.p + b * a.q.sb + hq * a.q.sh + s.start * a.q.st, s.Bn, a.q.st * 2);
    const uint16_t* hl = g.do_hl + (((int64_t)b * a.Hq + hq) * a.L + s.start) * kOrow;
    const u32x4 ro = make_rsrc(hl, (uint32_t)s.Bn * (kOrow * 2u));
    request_tile<8>(rq, (uint32_t)(a.q.st * 2), r0, lds, w, l);
#pragma unroll
    for (int h = 0; h < PARTS; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r4 = w * 2 + i, r = r4 * 4 + (l >> 4);
        load_to_lds(ro, lds + (1 + h) * kTile + r4 * 1024, (r0 + r) * (kOrow * 2) + h * 256 + (((l & 15) ^ swz(r)) << 4));
      }
    if (tid < 192) {
      const int r = r0 + (tid & 63);
      stat = r < s.Bn ? g.stats[(tid >> 6) * plane + ((int64_t)b * a.Hq + hq) * a.L + s.start + r] : 0.f;
    }
  };
  auto publish_stats = [&](int it) {
    if (it < N && tid < 192) st_lds[(it & 1) * 192 + tid] = stat;
  };
  request(0);
  // either kind of wave has the loop to itself (the registers of one do not count against the other)
  auto run = [&](auto for_v_t) {
  constexpr bool for_v = decltype(for_v_t)::value;
  // key (and value) fragments of this lane's position; positions past the end are computed from the last one and dropped
  bf16x8 fk[8], fv[8];
  {
    const int jc = min(j, Tn - 1);
    const uint16_t* kp = (jc < s.m ? s.ck + (int64_t)jc * kD
                                   : (const uint16_t*)a.k.p + b * a.k.sb + hkv * a.k.sh + (s.start + jc - s.m) * a.k.st) + lh * 8;
    const uint16_t* vp = (jc < s.m ? s.cv + (int64_t)jc * kD
                                   : (const uint16_t*)a.v.p + b * a.v.sb + hkv * a.v.sh + (s.start + jc - s.m) * a.v.st) + lh * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) fk[ks] = *(const bf16x8*)(kp + ks * 16);
    if (!for_v)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) fv[ks] = *(const bf16x8*)(vp + ks * 16);
  }
  // (operand addresses of the other k steps and column blocks are these, xor a constant: registers are short here)
  int row0, tr0[2];
  {
    TileAddr ad;
    tile_addr(l, ad);
    row0 = ad.row[0];
    tr0[0] = ad.tr[0][0];
    tr0[1] = ad.tr[0][1];
  }
  const float c = a.scale * kLog2e;
  f32x16 acc[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = zero16();
  wait_loads<0>();
  landed(fk);
  if (!for_v) landed(fv);
  publish_stats(0);
  __syncthreads();

  for (int it = 0; it < N; ++it) {
    request(it + 1);
    const int r0 = (first + it % rtiles) * 64;
    const unsigned char* Q = smem + (it & 1) * kSet * kTile;
    const float* st = st_lds + (it & 1) * 192 + lh * 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int rb = r0 + h * 32;
      if (rb >= s.Bn || (wj >= s.m && rb + 31 < wj - s.m)) continue;      // no row of this half sees these keys
      const unsigned char* q0 = Q + h * 32 * 256;
      // N products of one accumulator, their operands read two ahead (left alone the compiler reads each right before its
      // product and waits for it)
      auto chain = [&](auto n_t, auto read, const bf16x8 (&f)[8], f32x16& to) {
        constexpr int N = decltype(n_t)::value;
        bf16x8 ring[3];
#pragma unroll
        for (int i = 0; i < 2; ++i) ring[i] = read(i);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          if (i + 2 < N) ring[(i + 2) % 3] = read(i + 2);
          __builtin_amdgcn_sched_barrier(0);
          to = mfma32(ring[i % 3], f[i % 8], to);
        }
      };
      f32x16 sc = zero16();
      chain(std::integral_constant<int, 8>{}, [&](int i) { return *(const bf16x8*)(q0 + (row0 ^ (i << 5))); }, fk, sc);
      __builtin_amdgcn_sched_barrier(0);
      float p[16];
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) {
        const f32x4 mcs = *(const f32x4*)(st + h * 32 + gi * 8), inv = *(const f32x4*)(st + 64 + h * 32 + gi * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) p[gi * 4 + e] = __builtin_amdgcn_exp2f(fmaf(sc[gi * 4 + e], c, -mcs[e])) * inv[e];
      }
      auto hide = [&]() {                   // pairs of a key and a query that does not see it
        if (rb + 31 >= s.Bn || (wj + 31 >= s.m && rb < wj + 31 - s.m)) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int r = rb + (i >> 2) * 8 + lh * 4 + (i & 3);
            if (r >= s.Bn || j - s.m > r) p[i] = 0.f;
          }
        }
      };
      if (for_v) hide();
      if (for_v) {
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          bf16x8 fp[PARTS];
          split_parts<PARTS>(p + 8 * s2, fp);
          const unsigned char* o0 = q0 + kTile + s2 * 16 * 256;
#pragma unroll
          for (int u = 0; u < PARTS; ++u) {
            bf16x8 fo[4];
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) fo[ct] = frag_tr(o0 + u * kTile + (tr0[0] ^ (ct << 6)), o0 + u * kTile + (tr0[1] ^ (ct << 6)));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; u + v < PARTS; ++v)
#pragma unroll
              for (int ct = 0; ct < 4; ++ct) acc[ct] = mfma32(fo[ct], fp[v], acc[ct]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else {
        f32x16 dp = zero16();
        chain(std::integral_constant<int, 8 * PARTS>{}, [&](int i) { return *(const bf16x8*)(q0 + (1 + i / 8) * kTile + (row0 ^ (i % 8 << 5))); }, fv, dp);
#pragma unroll
        for (int gi = 0; gi < 4; ++gi) {
          const f32x4 dd = *(const f32x4*)(st + 128 + h * 32 + gi * 8);
#pragma unroll
          for (int e = 0; e < 4; ++e) p[gi * 4 + e] *= (dp[gi * 4 + e] - dd[e]) * a.scale;
        }
        hide();                             // (here, so that a query that is no number stays out of later keys' gradients)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          bf16x8 fd[PARTS];
          split_parts<PARTS>(p + 8 * s2, fd);
          const unsigned char* t0 = q0 + s2 * 16 * 256;
          bf16x8 qf[4];
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) qf[ct] = frag_tr(t0 + (tr0[0] ^ (ct << 6)), t0 + (tr0[1] ^ (ct << 6)));
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < PARTS; ++u)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) acc[ct] = mfma32(qf[ct], fd[u], acc[ct]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    wait_loads<0>();
    publish_stats(it + 1);
    __syncthreads();
  }
  if (j < Tn) {
    float* dc = (for_v ? g.d_cv : g.d_ck) + ((int64_t)n * a.batch * a.Hkv + chain) * a.M * kD;
    float* db = (for_v ? g.d_v : g.d_k) + b * g.k_sb + hkv * g.k_sh + s.start * kD;
    float* out = (j < s.m ? dc + (int64_t)j * kD : db + (int64_t)(j - s.m) * kD) + lh * 4;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int gi = 0; gi < 4; ++gi)
        *(f32x4_any*)(out + ct * 32 + gi * 8) = f32x4{acc[ct][gi * 4], acc[ct][gi * 4 + 1], acc[ct][gi * 4 + 2], acc[ct][gi * 4 + 3]};
  }
  };
  if (w < 4) run(std::true_type{});
  else run(std::false_type{});
}

}  // namespace

template <int PARTS>
static hipError_t launch_parts(const BwdAttnArgs& g, hipStream_t s) {
  const AttnArgs& a = g.a;
  constexpr int lds_q = 4 * kTile, lds_kv = 2 * (1 + PARTS) * kTile + 2 * 3 * 64 * 4;
  static bool attr_set = false;   // benign race: setting it twice is harmless
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)bwd_attn_q_k<PARTS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_q);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)bwd_attn_kv_k<PARTS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_kv);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(bwd_attn_q_k<PARTS>, dim3((unsigned)(a.qtiles * a.Hq * a.batch * a.n_seg)), dim3(256), lds_q, s, g);
  const int ktiles = (a.M + a.B + 127) / 128;
  hipLaunchKernelGGL(bwd_attn_kv_k<PARTS>, dim3((unsigned)(ktiles * a.batch * a.Hkv * a.n_seg)), dim3(512), lds_kv, s, g);
  return hipGetLastError();
}

hipError_t launch_bwd_attn_mfma(BwdAttnArgs g, hipStream_t s) {
  AttnArgs& a = g.a;
  a.qtiles = (a.B + 127) / 128;
  // runs of blocks of one form: all of them as a rule, or all but a ragged last one
  auto parts = [&](int n) {
    const int64_t left = a.L - (int64_t)n * a.B;
    return g.three_parts || ((n <= a.n_fill ? a.len0 + n * a.B : a.M) + (int)(left < a.B ? left : a.B)) % 4 ? 3 : 2;
  };
  const int n_all = a.n_seg;
  hipError_t e = hipSuccess;
  for (int n = 0; n < n_all && e == hipSuccess; n += a.n_seg) {
    a.seg_first = n;
    for (a.n_seg = 1; n + a.n_seg < n_all && parts(n + a.n_seg) == parts(n);) ++a.n_seg;
    e = parts(n) == 2 ? launch_parts<2>(g, s) : launch_parts<3>(g, s);
  }
  return e;
}

}  // namespace lococo
