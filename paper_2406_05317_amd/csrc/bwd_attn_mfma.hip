// Backward of the attention of every block of a window (Alg. 2 step 3), two kernels, bf16 MFMA, head_dim 128.
//
// Nothing of size queries x keys goes through memory: both kernels recompute the score tiles.
//   bwd_attn_q_k    a workgroup per 128 query rows: one walk over the keys for the row statistics (softmax reference,
//                   1 / row sum) and D = sum_j P dP, a second one for dq = dS Yk.  Leaves dO as two bf16 halves and the
//                   statistics for
//   bwd_attn_kv_k   a workgroup per 128 keys of [cache ; block]: dYk = dS^T q and dYv = P^T dO over the rows of all
//                   heads of the group.
// The fp32 operands (dO, P, dS) enter the matrix products as two bf16 halves (16 bits kept): S 1, dP 2, dq 2, dYk 2,
// dYv 3 products; with the recomputation (S and dP three times each) 16 products per (query, key) pair of 128 columns.  A block
// whose number of positions is no multiple of 4, or a step whose gradients are not 16-byte aligned, enters with three parts (24
// bits, nothing lost; dP, dq, dYk 3, dYv 6 products): those have always been computed in fp32, and errors stay at that level (3e-7
// against 3.5e-6 with two).
// Measured, 64 blocks of 512 queries on 1024 keys, 32 heads: 4.1 ms for the whole sequence (1.9 + 2.2) against 20.0 ms as
// seven batched products and a row kernel per block with P, dS in fp32 in memory; 28 blocks of 128 on 256: 0.21 against
// 3.0 ms (launches of 15 - 23 us each that did not fill the chip).  Bound by the issue of the vector and LDS instructions
// between the products (matrix pipe 43 % busy in the first kernel, 33 % in the second).  The second kernel took 2.8 ms and 144 us
// with one workgroup of eight waves to a compute unit, four for dYv and four for dYk with S computed twice: of a workgroup's
// 90 000 cycles 14 000 went by before its first product and 20 000 in its stores, and the kinds waited for each other 1 800 of
// 8 200 a tile.  One such workgroup with both sums in every wave still took 2.7 ms, but is the faster form where there are no more
// workgroups than compute units (see two_waves).
// D is taken from P and dP, not from dO . O: the stored outputs are bf16 and would cost dS half its bits.
#include <algorithm>

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

// A wave accumulates dYk and dYv of 32 keys: 128 of its 256 registers are sums, so key and value fragments lie in LDS in part,
// in fragment order: as many as it takes to spill none (a reload waits for the tiles requested before it).  The rows of all heads
// are walked in tiles of 32.
// HV 1: a workgroup is four waves, one per 32 keys, and two share a compute unit: one's first loads and last stores, a third of
// its life, fall beside the other's products.  (Three parts: fewer fragments find room in LDS, and dP's operands are read one
// product ahead instead of two for it.  4097 tokens in blocks of 303 on 687 keys, 32 heads: 296 us, with eight waves 350; 1528
// in blocks of 191 on 383, 128 heads: 255 and 321.)
// HV 2: eight waves, two per 32 keys that take every second tile and add up at the end: half as many tiles in series, for launches
// that leave compute units idle.
template <int PARTS, int HV>
struct Kv {
  static constexpr int tile = 32 * 256, set = HV * (1 + PARTS) * tile;                // [half] tiles of q | parts of dO
  // k steps whose value, key fragments are in LDS
  static constexpr int VL = HV == 1 ? (PARTS == 2 ? 4 : 0) : (PARTS == 2 ? 5 : 4), KL = 3;
  static constexpr int f_at = 2 * set, st_at = f_at + (VL + KL) * 4 * 1024, end = st_at + 2 * HV * 3 * 32 * 4;
  static constexpr int sums = HV == 1 ? 0 : 8 * 64 * 64 * 4, lds = end > sums ? end : sums;   // (handed over behind the walk)
  static_assert(lds <= 80 * 1024 * HV, "two workgroups of four waves, one of eight");
};
template <int PARTS, int HV>
__global__ __launch_bounds__(256 * HV, 2) void bwd_attn_kv_k(BwdAttnArgs g) {
  using X = Kv<PARTS, HV>;
  constexpr int VL = X::VL, KL = X::KL;
  extern __shared__ __align__(16) unsigned char smem[];       // [2][HV] tiles, fragments, [2][HV][3][32] statistics
  const AttnArgs& a = g.a;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)smem);
  float* st_lds = (float*)(smem + X::st_at);
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int ktiles = (a.M + a.B + 127) / 128;
  const int chain = (item / ktiles) % (a.batch * a.Hkv), n = a.seg_first + item / ktiles / (a.batch * a.Hkv);
  const int b = chain / a.Hkv, hkv = chain % a.Hkv, j0 = (item % ktiles) * 128;
  const Seg s = segment(a, n, chain);
  const int Tn = s.m + s.Bn;
  if (j0 >= Tn) return;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l31 = l & 31, lh = l >> 5;
  const int kg = w & 3, half = w >> 2;
  const int wj = j0 + 32 * kg, j = wj + l31;                  // this lane's position in [cache ; block]
  const int first = j0 >= s.m ? (j0 - s.m) / 32 : 0;          // tiles of rows before it see none of the keys
  const int rtiles = (s.Bn + 31) / 32 - first, N = (a.group * rtiles + HV - 1) / HV;
  const int64_t plane = (int64_t)a.batch * a.Hq * a.L;

  // requests tile u (q, then the parts of dO) of this half's next rows, behind the last of them the walk moves on
  float stat = 0.f;
  int rn = half, hn = 0, buf = 0;           // these rows: tile `first + rn` of head hn
  auto wrap = [&](int& r, int& h) {
#pragma unroll
    for (int i = 0; i < HV; ++i)
      if (r >= rtiles) { r -= rtiles; ++h; }
  };
  wrap(rn, hn);
  int rt = rn, ht = hn;                     // the rows whose products come next
  auto request = [&](int u) {
    if (hn >= a.group) return;
    int l = tid & 63;
    asm volatile("" : "+v"(l));             // (offsets are worked out again every time, not kept in registers)
    const int hq = hkv * a.group + hn, r0 = (first + rn) * 32;
    const uint32_t lds = lds0 + buf * X::set + (half * (1 + PARTS) + u) * X::tile;
    const uint16_t* hl = g.do_hl + (((int64_t)b * a.Hq + hq) * a.L + s.start) * kOrow;
    const u32x4 rs = u == 0 ? rows_rsrc((const uint16_t*)a.q.p + b * a.q.sb + hq * a.q.sh + s.start * a.q.st, s.Bn, a.q.st * 2)
                            : make_rsrc(hl, (uint32_t)s.Bn * (kOrow * 2u));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r4 = kg * 2 + i, r = r4 * 4 + (l >> 4), c = ((l & 15) ^ swz(r)) << 4;
      load_to_lds(rs, lds + r4 * 1024, u == 0 ? (r0 + r) * (uint32_t)(a.q.st * 2) + c : (r0 + r) * (kOrow * 2) + (u - 1) * 256 + c);
    }
    if (u == 0 && (tid & 255) < 96) {
      const int r = r0 + tid % 32;
      stat = r < s.Bn ? g.stats[(tid & 255) / 32 * plane + ((int64_t)b * a.Hq + hq) * a.L + s.start + r] : 0.f;
    }
    if (u == PARTS) {
      buf ^= 1;
      rn += HV;
      wrap(rn, hn);
    }
  };
  auto publish_stats = [&](int at) {
    if ((tid & 255) < 96) st_lds[(at * HV + half) * 96 + (tid & 255)] = stat;
  };
#pragma unroll
  for (int u = 0; u <= PARTS; ++u) request(u);
  // key and value fragments of this lane's position; positions past the end are computed from the last one and dropped
  bf16x8 fk[8], fv[8];                      // [KL ..], [VL ..]: those that stay in registers
  unsigned char* const vf = smem + X::f_at + kg * 1024 + l * 16;
  unsigned char* const kf = vf + VL * 4096;
  {
    const int jc = min(j, Tn - 1);
    const uint16_t* kp = (jc < s.m ? s.ck + (int64_t)jc * kD
                                   : (const uint16_t*)a.k.p + b * a.k.sb + hkv * a.k.sh + (s.start + jc - s.m) * a.k.st) + lh * 8;
    const uint16_t* vp = (jc < s.m ? s.cv + (int64_t)jc * kD
                                   : (const uint16_t*)a.v.p + b * a.v.sb + hkv * a.v.sh + (s.start + jc - s.m) * a.v.st) + lh * 8;
#pragma unroll
    for (int ks = KL; ks < 8; ++ks) fk[ks] = *(const bf16x8*)(kp + ks * 16);
#pragma unroll
    for (int ks = VL; ks < 8; ++ks) fv[ks] = *(const bf16x8*)(vp + ks * 16);
    if (HV == 1 || half == 0)
#pragma unroll
      for (int ks = 0; ks < VL; ++ks) *(bf16x8*)(vf + ks * 4096) = *(const bf16x8*)(vp + ks * 16);
    if (HV == 1 || half == 1)
#pragma unroll
      for (int ks = 0; ks < KL; ++ks) *(bf16x8*)(kf + ks * 4096) = *(const bf16x8*)(kp + ks * 16);
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
  f32x16 av[4], ak[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) av[ct] = ak[ct] = zero16();
  wait_loads<0>();
#pragma unroll
  for (int ks = KL; ks < 8; ++ks) asm volatile("" : "+v"(fk[ks]));     // (see landed)
#pragma unroll
  for (int ks = VL; ks < 8; ++ks) asm volatile("" : "+v"(fv[ks]));
  publish_stats(0);
  __syncthreads();

  for (int it = 0; it < N; ++it) {
    request(0);
    const int rb = (first + rt) * 32;
    const float* st = st_lds + ((it & 1) * HV + half) * 96 + lh * 4;
    const bool seen = ht < a.group && !(wj >= s.m && rb + 31 < wj - s.m);   // else there is no row that sees these keys
    rt += HV;
    wrap(rt, ht);
    if (seen) {
      asm volatile("" : "+v"(row0), "+v"(tr0[0]), "+v"(tr0[1]));       // (or the xors are kept in registers of their own)
      const unsigned char* q0 = smem + (it & 1) * X::set + half * (1 + PARTS) * X::tile;
      const bool hidden = rb + 31 >= s.Bn || (wj + 31 >= s.m && rb < wj + 31 - s.m);
      auto hide = [&](float (&p)[16]) {     // pairs of a key and a query that does not see it
        if (hidden) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int r = rb + (i >> 2) * 8 + lh * 4 + (i & 3);
            if (r >= s.Bn || j - s.m > r) p[i] = 0.f;
          }
        }
      };
      auto pin = [&]() { __builtin_amdgcn_sched_barrier(0); };
      auto transposed = [&](const unsigned char* t, int ct) { return frag_tr(t + (tr0[0] ^ (ct << 6)), t + (tr0[1] ^ (ct << 6))); };
      f32x16 sc, dp;
      // S and dP, operands read two products ahead (left alone the compiler reads each right before its product and waits for it)
      auto scores = [&]() {
        bf16x8 ring[3], rk[3];
        auto read = [&](int i) {
          ring[i % 3] = *(const bf16x8*)(q0 + (row0 ^ (i << 5)));
          rk[i % 3] = i < KL ? *(const bf16x8*)(kf + i * 4096) : fk[i];
        };
        sc = zero16();
        read(0);
        read(1);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (i + 2 < 8) read(i + 2);
          pin();
          sc = mfma32(ring[i % 3], rk[i % 3], sc);
        }
        pin();
      };
      auto weights_grad = [&]() {
        constexpr int R = PARTS == 3 && HV == 1 ? 2 : 3;
        bf16x8 ring[R], rv[2];
        auto read = [&](int i) {            // product i: part i % PARTS of k step i / PARTS
          const int ks = i / PARTS;
          ring[i % R] = *(const bf16x8*)(q0 + (1 + i % PARTS) * X::tile + (row0 ^ (ks << 5)));
          if (i % PARTS == 0) rv[ks % 2] = ks < VL ? *(const bf16x8*)(vf + ks * 4096) : fv[ks];
        };
        dp = zero16();
#pragma unroll
        for (int i = 0; i < R - 1; ++i) read(i);
#pragma unroll
        for (int i = 0; i < 8 * PARTS; ++i) {
          if (i + R - 1 < 8 * PARTS) read(i + R - 1);
          pin();
          dp = mfma32(ring[i % R], rv[i / PARTS % 2], dp);
        }
        pin();
      };
      if (HV == 2 && half) weights_grad();             // (the two waves of a SIMD: one's products beside the other's exponentials)
      scores();
      request(1);
      pin();
      bf16x8 ring[2];
      auto read_o = [&](int i) {            // fragment i: column block i % 4 of part i / 4 % PARTS, rows 16 (i / 4 / PARTS) ..
        if (i < 8 * PARTS) ring[i % 2] = transposed(q0 + (1 + i / 4 % PARTS) * X::tile + i / 4 / PARTS * 16 * 256, i % 4);
      };
      read_o(0);
      float p[16];
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) {
        const f32x4 mcs = *(const f32x4*)(st + gi * 8), inv = *(const f32x4*)(st + 32 + gi * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) p[gi * 4 + e] = __builtin_amdgcn_exp2f(fmaf(sc[gi * 4 + e], c, -mcs[e])) * inv[e];
        if (PARTS == 3 && gi == 1) pin();   // (registers)
      }
      hide(p);
      bf16x8 part[PARTS];
#pragma unroll
      for (int i = 0; i < 8 * PARTS; ++i) {
        if (i % (4 * PARTS) == 0) split_parts<PARTS>(p + i / 4 / PARTS * 8, part);
        read_o(i + 1);
        pin();
#pragma unroll
        for (int v = 0; i / 4 % PARTS + v < PARTS; ++v) av[i % 4] = mfma32(ring[i % 2], part[v], av[i % 4]);
        pin();
      }
#pragma unroll
      for (int u = 2; u <= PARTS; ++u) request(u);
      pin();
      if (HV == 1 || !half) weights_grad();
      auto read_q = [&](int i) {
        if (i < 8) ring[i % 2] = transposed(q0 + i / 4 * 16 * 256, i % 4);
      };
      read_q(0);
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) {
        const f32x4 dd = *(const f32x4*)(st + 64 + gi * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) p[gi * 4 + e] *= (dp[gi * 4 + e] - dd[e]) * a.scale;
      }
      hide(p);                              // (again, so that a query that is no number stays out of later keys' gradients)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (i % 4 == 0) split_parts<PARTS>(p + i / 4 * 8, part);
        read_q(i + 1);
        pin();
#pragma unroll
        for (int u = 0; u < PARTS; ++u) ak[i % 4] = mfma32(ring[i % 2], part[u], ak[i % 4]);
        pin();
      }
    }
    if (!seen)
#pragma unroll
      for (int u = 1; u <= PARTS; ++u) request(u);
    wait_loads<0>();
    publish_stats(~it & 1);
    __syncthreads();
  }
  float* const dc = (half ? g.d_ck : g.d_cv) + ((int64_t)n * a.batch * a.Hkv + chain) * a.M * kD;
  float* const db = (half ? g.d_k : g.d_v) + b * g.k_sb + hkv * g.k_sh + s.start * kD;
  float* const out = (j < s.m ? dc + (int64_t)j * kD : db + (int64_t)(j - s.m) * kD) + lh * 4;
  auto quad = [](const f32x16 (&x)[4], int i) {
    return f32x4{x[i >> 2][(i & 3) * 4], x[i >> 2][(i & 3) * 4 + 1], x[i >> 2][(i & 3) * 4 + 2], x[i >> 2][(i & 3) * 4 + 3]};
  };
  if constexpr (HV == 1) {
    float* const ko = (j < s.m ? g.d_ck + (((int64_t)n * a.batch * a.Hkv + chain) * a.M + j) * kD
                               : g.d_k + b * g.k_sb + hkv * g.k_sh + (s.start + j - s.m) * kD) + lh * 4;
    if (j < Tn)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        *(f32x4_any*)(out + (i >> 2) * 32 + (i & 3) * 8) = quad(av, i);
        *(f32x4_any*)(ko + (i >> 2) * 32 + (i & 3) * 8) = quad(ak, i);
      }
  } else {                                  // the two halves trade: waves 0..3 finish dYv of their keys, waves 4..7 dYk
    f32x4* const give = (f32x4*)smem + w * 1024 + l;
    const f32x4* const take = (const f32x4*)smem + (w ^ 4) * 1024 + l;
    auto hand_over = [&](const f32x16 (&x)[4]) {
#pragma unroll
      for (int i = 0; i < 16; ++i) give[i * 64] = quad(x, i);
    };
    if (half) hand_over(av);
    else hand_over(ak);
    __syncthreads();
    auto finish = [&](const f32x16 (&x)[4]) {
#pragma unroll
      for (int i = 0; i < 16; ++i) *(f32x4_any*)(out + (i >> 2) * 32 + (i & 3) * 8) = quad(x, i) + take[i * 64];
    };
    if (j < Tn) {
      if (half) finish(ak);
      else finish(av);
    }
  }
}

}  // namespace

// block n of a window: live slots before it, tokens
static int live_before(const AttnArgs& a, int n) { return n <= a.n_fill ? a.len0 + n * a.B : a.M; }
static int tokens_of(const AttnArgs& a, int n) { return (int)std::min<int64_t>(a.B, a.L - (int64_t)n * a.B); }

// Two waves per 32 keys where the longest walk is four tiles or more, and the workgroups fill no more than a compute unit each.
// They are counted by what they walk, three tiles on top for loads and stores, in units of the longest: most of a block's keys are
// seen by few of its rows.  One step, us, one wave and two: 8 key heads of 32 query heads, 128 tokens on 256 keys 48.0 and 34.0, 16
// on 144 18.2 and 16.3; 32 heads, 128 tokens 19.2 and 17.0, 96 15.7 and 15.7, 32 10.6 and 12.5; 64 chains, 512 tokens 71 and 83;
// three parts, 8 of 32 heads, 127 tokens on 255 keys 59 and 45; 32 heads, one token 11.8 and 13.7; 64 chains, 77 on 589 keys 30 and 38;
// 32 chains, 514 on 1026, 288 workgroups, 76 and 53.  Over 150 steps of 160 - 700 workgroups the form not taken is at best 6 % the
// faster one, 0.1 % on average (their plain number on either side of the compute units: 31 and 0.9 %).
static bool two_waves(const AttnArgs& a) {
  const int longest = a.group * ((tokens_of(a, a.seg_first) + 31) / 32);
  if (longest < 4) return false;
  const int64_t room = (int64_t)cu_count() * (longest + 3), chains = (int64_t)a.batch * a.Hkv;
  int64_t work = 0;
  for (int n = a.seg_first; n < a.seg_first + a.n_seg; ++n) {
    const int m = live_before(a, n), Bn = tokens_of(a, n);
    for (int j = 0; j < m + Bn; j += 128) {
      work += chains * (a.group * ((Bn + 31) / 32 - std::max(0, (j - m) / 32)) + 3);
      if (work > room) return false;
    }
  }
  return true;
}

template <int PARTS, int HV>
static hipError_t launch_kv(const BwdAttnArgs& g, hipStream_t s) {
  const AttnArgs& a = g.a;
  constexpr int lds = Kv<PARTS, HV>::lds;
  static bool attr_set = false;   // benign race: setting it twice is harmless
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute((const void*)bwd_attn_kv_k<PARTS, HV>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int ktiles = (a.M + a.B + 127) / 128;
  hipLaunchKernelGGL((bwd_attn_kv_k<PARTS, HV>), dim3((unsigned)(ktiles * a.batch * a.Hkv * a.n_seg)), dim3(256 * HV), lds, s, g);
  return hipGetLastError();
}

template <int PARTS>
static hipError_t launch_parts(const BwdAttnArgs& g, hipStream_t s) {
  const AttnArgs& a = g.a;
  constexpr int lds_q = 4 * kTile;
  static bool attr_set = false;   // benign race: setting it twice is harmless
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute((const void*)bwd_attn_q_k<PARTS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_q);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(bwd_attn_q_k<PARTS>, dim3((unsigned)(a.qtiles * a.Hq * a.batch * a.n_seg)), dim3(256), lds_q, s, g);
  return two_waves(a) ? launch_kv<PARTS, 2>(g, s) : launch_kv<PARTS, 1>(g, s);
}

hipError_t launch_bwd_attn_mfma(BwdAttnArgs g, hipStream_t s) {
  AttnArgs& a = g.a;
  a.qtiles = (a.B + 127) / 128;
  // runs of blocks of one form: all of them as a rule, or all but a ragged last one
  auto parts = [&](int n) { return g.three_parts || (live_before(a, n) + tokens_of(a, n)) % 4 ? 3 : 2; };
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
