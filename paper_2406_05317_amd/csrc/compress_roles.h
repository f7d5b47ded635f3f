// The work of one workgroup of the fused compression kernel on a tile of 32 slots (the method, the two walks over a [K | V]
// bank, the layouts and the template parameters are described in compress_tile.h).
//
// Two roles.  A step of 32 slots is a chain of short position tiles, and with one wave per SIMD that does everything a tile took
// 2 055 cycles for 1 216 of matrix work: the wave issues some 300 instructions a tile, and whatever it waits for, the matrix
// pipe waits for too.  So the workgroup has eight waves, a SIMD one of either kind:
//   logit waves (0 .. 3)    hold the filter slice, a quarter of the channels each, and do nothing but the logit products of
//                           one tile after the other, leaving their partial sums in LDS;
//   mixing waves (4 .. 7)   stage the tiles, add up the partial logits, run the softmax and mix, 64 columns of [K | V] each.
// In stage i the logit waves work on tile i + 1 and the mixing waves on the softmax of tile i and the mixing of tile i - 1;
// partial logits, probabilities and rescale factors are double-buffered, so one barrier ends a stage.  A wave has 256 registers;
// builds without protected slots keep everything in them, but for those that share out the positions of a step.  What bounds a
// stage now is LDS, some 1 760 cycles of operand reads, partial logits and staging.
// Measured against one role, whole calls, width 21 over [K | V] with 32 heads: the compressor as printed, 3.5 K tokens, M = 128:
// 723 -> 559 us.  Where every (chain, slot tile) has one workgroup to itself, 3.5 K tokens, M = 256: 664 -> 637 us, one token
// 36.7 -> 33.5, 77 tokens 47.3 -> 43.7.  Several chains per workgroup: 4 x 2 K tokens, M = 128: 861 -> 825 us; 4 K tokens,
// M = 512: 1322 -> 1269; 8 x 33 tokens, M = 128: 83.1 -> 80.4.  54 such shapes, widths 15 and 21, with and without protected
// slots: 1.02 - 1.37 times as fast.
// Filters over the keys, single steps: 77 tokens on a cache of 256, 8 kv heads: 18.9 -> 16.7 us; one token of 32
// heads on 128 slots: 11.9 -> 11.2 us.  Scans with filters over the keys stay with compress_mfma_k, whose stages take as long there
// (3.5 K tokens: 312 against 316 us) and whose prologue is shorter.
#pragma once

#include "compress_tile.h"

namespace lococo {
namespace compress_detail {

constexpr int kRoleThreads = 2 * kThreads;

template <int KW>
struct Roles {
  using G = Geo<32, KW>;
  static constexpr int LDS = G::LDS + G::SBYTES;     // (the partial logits twice)
  static_assert(LDS <= 160 * 1024, "LDS budget");
};

template <int KW, int NORM, int PROT, int MULTI, int SPLIT, int CIN>
__device__ __forceinline__ void compress_roles(const ScanArgs& sa, const uint16_t* wp, int64_t wp_head_stride, unsigned char* smem,
                                               uint32_t wg_id, uint32_t wg_count) {
  constexpr int BM = 32;
  using G = Geo<BM, KW>;
  static_assert(!SPLIT || !MULTI, "the splits are built for one chain per workgroup");
  constexpr bool PSPLIT = SPLIT == 1, PIPE = SPLIT == 2;
  // Who stages key tile 0 of a walk.  With the loops over passes and chains of a workgroup that has its tile to itself, the logit
  // waves of width 21 (168 registers of filters) had no room for the tile's addresses: they came back from scratch memory in
  // front of every walk.  The mixing waves have the room, and request it with tiles 1 - 3, under the logit waves' filter load.
  // (one token of four sequences, M = 128, width 21: 42.2 -> 39.5 us; 4 x 2 K tokens: 864 -> 840; M = 512: 1278 -> 1274)
  constexpr bool kMixersStageAll = SPLIT == 0;
  const StepArgs& a = sa.st;
  unsigned char* Xs0 = smem;                                    // NXBUF key tiles (with halo)
  unsigned char* Vs0 = Xs0 + G::NXBUF * G::XBYTES;              // NVBUF value tiles
  float* Sred0 = (float*)(Vs0 + G::NVBUF * G::VBYTES);          // 2 x 4 partial-logit tiles [wave][slot][pos]
  unsigned char* Ps0 = (unsigned char*)Sred0 + 2 * G::SBYTES;   // 2 probability tiles [slot][pos], bf16
  float* alphas0 = (float*)(Ps0 + 2 * G::PBYTES);               // 2 x rescale factor per slot
  float* lsum = alphas0 + 2 * BM;                               // final row sums
  __shared__ int bail;                       // a chain wait timed out: leave
  __shared__ int same_l2;
  __shared__ int i_merge;                    // (PSPLIT) this part completes the count
  __shared__ int split_fast;

  // tid, w: inside the role; the wave index as a scalar
  const int wg_tid = threadIdx.x, tid = wg_tid & (kThreads - 1), w = __builtin_amdgcn_readfirstlane(wg_tid >> 6) & 3, l = wg_tid & 63;
  const int l31 = l & 31, lh = l >> 5;
  const bool mixer = __builtin_amdgcn_readfirstlane(wg_tid >> 8) != 0;
  // Workgroups are dealt to the 8 XCDs round-robin by their linear id.  The slot tiles of one chain
  // all read the same keys and values, so they are given ids that land on one XCD (one L2).
  int item = wg_id;
  {
    const int per = wg_count / 8;
    if (item < per * 8) item = (item % 8) * per + item / 8;
  }
  const int tiles = a.M / BM;
  // splits: consecutive work items are the workgroups of one (chain, slot tile), so they land on one XCD
  const int P = SPLIT ? sa.psplit : 1;
  const int part = SPLIT ? item % P : 0;
  if (SPLIT) item /= P;
  // A workgroup owns one slot tile of the chains grp, grp + groups, grp + 2 groups, ...  (one chain
  // when the launch has a workgroup per chain and tile).  Where filters or biases differ between
  // kv heads the host picks `groups` as a multiple of Hkv, so all of them belong to head hkv0.
  const int grp = item / tiles, groups = wg_count / (tiles * P), n_chains = a.batch * a.Hkv;
  const int hkv0 = grp % a.Hkv;
  const int i0 = (item % tiles) * BM;
  if (wg_tid == 0) { bail = 0; same_l2 = 0; }
  __syncthreads();
  // ---- meeting point of the slot tiles of a chain between two steps of the one-launch scan:
  // a counter per chain.  A tile signals when its rows of the new cache are written and waits,
  // before it reads the chain's cache for the next step, until the counter says that every tile
  // has signalled: round r is complete at tiles * (r + 1).  A workgroup with several chains goes
  // through them in the same order as the other tiles of its group, so by the time it comes back to a
  // chain the others have long signalled and the wait costs one load; with one chain per
  // workgroup the wait follows the signal directly.
  //
  // General form: workgroup barrier, thread 0 does a device-scope release increment (which writes
  // the L2 back: every dirty line of the XCD, about 3 us per step on the 32 K-token workload);
  // the wait polls, then a device-scope acquire, then a workgroup barrier.  One wave pays for the
  // cache maintenance.
  //
  // When all tiles of the chain run on one XCD they share one L2, and nothing has to be written
  // back or invalidated there: stores go through the CU's L1 to the L2 and have arrived when the
  // wave's store counter reaches zero, and the cache rows are read at device scope (see
  // load_cat16).  So each wave waits for its stores, the workgroup meets, thread 0 increments with
  // a relaxed device-scope atomic and polls with relaxed loads.  Whether the tiles share an XCD is
  // not assumed from the workgroup numbering: round 0, before the first step, is a general-form
  // meeting in which every tile reports the XCD it runs on.
  auto chain_signal = [&](int c) {
    const bool fast = same_l2 != 0;          // LDS word written before the previous workgroup barrier
    if (fast) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (wg_tid == 0) {
      if (fast) __hip_atomic_fetch_add(sa.sync + c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else __hip_atomic_fetch_add(sa.sync + c, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  auto chain_wait = [&](int c, int round) -> bool {
    if (wg_tid == 0) {
      // round 0 (the census) is signalled by every workgroup of the chain, later rounds by the one
      // workgroup per slot tile that writes the rows
      const uint32_t target = (uint32_t)(tiles * P) + (uint32_t)tiles * (uint32_t)round;
      int polls = 0;
      while (__hip_atomic_load(sa.sync + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        __builtin_amdgcn_s_sleep(2);
        if (++polls > sa.spin_limit) {         // bounded: never spin forever on a workgroup that is not there
          __hip_atomic_store(sa.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          bail = 1;
          break;
        }
      }
      if (same_l2 == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    return bail == 0;
  };
  if (PSPLIT && wg_tid == 0) {
    // every part registers the XCD it runs on in the census word of its (chain, tile); read at the hand-off
    const uint32_t xcd = __builtin_amdgcn_s_getreg(20 | ((4 - 1) << 11)) & 7u;
    __hip_atomic_fetch_add(sa.psync + 2 * (grp * tiles + i0 / BM) + 1, 1u << (3u * xcd), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  }
  if (sa.n_steps > 1) {
    uint32_t* xcd_mask = sa.sync + n_chains + 1;
    if (wg_tid == 0) {
      const uint32_t xcd = __builtin_amdgcn_s_getreg(20 | ((4 - 1) << 11));   // XCC_ID, bits [3:0]
      for (int c = grp; c < n_chains; c += groups)
        __hip_atomic_fetch_or(xcd_mask + c, 1u << xcd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int c = grp; c < n_chains; c += groups) chain_signal(c);
    bool one_xcd = true;
    for (int c = grp; c < n_chains; c += groups) {
      if (!chain_wait(c, 0)) return;
      if (wg_tid == 0) {
        const uint32_t mask = __hip_atomic_load(xcd_mask + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        one_xcd = one_xcd && (mask & (mask - 1)) == 0;
      }
    }
    if (wg_tid == 0) same_l2 = one_xcd && sa.same_l2_allowed;
    __syncthreads();
  }

  const int n_mine = MULTI ? (n_chains - grp + groups - 1) / groups : 1;

  // One walk's work, one step's and one launch's, written once and compiled for either role: the loops, the waits and the
  // barriers are the same, what lies between them is not.
  auto run = [&](auto mixer_t) {
  constexpr bool MIX = decltype(mixer_t)::value;
  // per-step and per-chain quantities, set at the top of the loops
  int T = 0, m = 0, NT = 0;
  int jbase = 0;            // first position of the range at hand (0 unless the positions are split or walked in legs)
  CatRows cat_k, cat_v;
  // protected-slot bits of the chain at hand (see lococo_cache.protect), or null
  const uint32_t* pwords = nullptr;

  // ---- logit waves: this wave's slice of the filter bank, resident in registers (for the whole kernel, or for a pass over a
  // [K | V] bank): lane (slot l31, channels 32w + 16h + 8*lh ..) for every tap
  bf16x8 wreg[MIX ? 1 : KW][2];
  auto load_filters = [&](int half_of_bank) {          // 0: the bank (or its key half), 1: its value half
    if constexpr (!MIX) {
      const uint16_t* wb = wp + hkv0 * wp_head_stride + (CIN ? (int64_t)half_of_bank * a.M * (KW * kD) : 0) + ((int64_t)(i0 / 32) * 4 + w) * (KW * 1024);
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)wb, 0, KW * 2048, 0x00020000);
#pragma unroll
      for (int t = 0; t < KW; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          wreg[t][h] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, l * 16, (t * 2 + h) * 1024, 0));
    }
  };
  auto pin_filters = [&]() {                 // here they have arrived, and from here on they stay
    if constexpr (!MIX) {
#pragma unroll
      for (int t = 0; t < KW; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) asm volatile("" : "+v"(wreg[t][h]));
    }
  };
  if (!CIN) {
    load_filters(0);
    pin_filters();
  }

  // ---- mixing waves
  // key-side logits of one tile as this lane left them in the first walk (CIN only)
  f32x4 pre = {0.f, 0.f, 0.f, 0.f};
  __amdgpu_buffer_rsrc_t pre_rows = __builtin_amdgcn_make_buffer_rsrc((void*)sa.prelogits, 0, 0, 0x00020000);
  // mixing accumulator, transposed: lane = slot l31, rows = columns 64w + ct*32 + (i/4)*8 + lh*4 + i%4
  f32x16 oacc[2];
  // softmax state of the slot this lane helps with (replicated over the LPR lanes of the slot)
  const int srow = w * G::RPW + l / G::LPR;
  const int sp0 = (l % G::LPR) * G::EPL;
  static_assert(G::EPL == 4, "a lane has four positions of a tile");
  float m_run = 0.f, l_run = 0.f;
  // (a softmax over the positions does not see a per-slot constant: the bias only enters the relu-sum form)
  const float bias =
      MIX && a.conv_b ? __uint_as_float((uint32_t)((const uint16_t*)a.conv_b)[hkv0 * a.b_head_stride + i0 + srow] << 16) : 0.f;
  // staging: global -> registers -> LDS (key tile with halo, value tile; both row-major)
  Cat16 xreg[G::XPER];
  Cat16 vreg[G::VPER];
  auto x_chunk = [&](int it, int j0) {
    const int item = tid + it * kThreads;
    return load_cat16(cat_k, j0 - G::PAD + (item >> 4), item & 15);
  };
  auto load_v = [&](int it, int j0) {
    const int item = tid + it * kThreads;
    vreg[it] = load_cat16(cat_v, j0 + (item >> 4), item & 15);
  };
  auto put_x = [&](int it, unsigned char* Xs, const Cat16& r) {
    const int item = tid + it * kThreads;
    *(u32x4*)(Xs + (item >> 4) * G::XSTRIDE + (item & 15) * 16) = r.from_cache | r.from_blk;
  };
  auto store_v = [&](int it, unsigned char* Vs) {
    const int item = tid + it * kThreads;
    *(u32x4*)(Vs + (item >> 4) * G::VSTRIDE + (item & 15) * 16) = vreg[it].from_cache | vreg[it].from_blk;
  };

  // ---- logit waves: the logits of tile c over this wave's channels, left in partial-logit buffer c % 2.
  // Ring of key operands, fetched kRing - 1 contraction steps ahead; kRing divides the number of steps, so the last steps of
  // a tile fetch the first operands of the next one.  acc: lane = slot l31, rows = positions (i/4)*8 + lh*4 + i%4.
  constexpr int kRing = G::NS % 10 == 0 ? 10 : (G::NS % 6 == 0 ? 6 : 7);
  static_assert(G::NS % kRing == 0, "the operand ring must wrap at the end of a tile");
  bf16x8 xv[MIX ? 1 : kRing];
  auto operand = [&](int c, int st) -> bf16x8 {
    const unsigned char* x = Xs0 + (c % G::NXBUF) * G::XBYTES + l31 * G::XSTRIDE + (32 * w + lh * 8) * 2;
    return *(const bf16x8*)(x + (st >> 1) * G::XSTRIDE + (st & 1) * 32);
  };
  auto logits_begin = [&]() {
    if constexpr (!MIX) {
#pragma unroll
      for (int st = 0; st < kRing - 1; ++st) xv[st] = operand(0, st);
    }
  };
  auto logits_of = [&](int c) {
    if constexpr (!MIX) {
      f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < G::NS; ++st) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv[st % kRing], wreg[st >> 1][st & 1], acc, 0, 0, 0);
        const int next = st + kRing - 1;     // (the ring slot of step st - 1 is free now)
        xv[next % kRing] = next < G::NS ? operand(c, next) : operand(c + 1, next - G::NS);
        __builtin_amdgcn_sched_barrier(0);
      }
      float* S = Sred0 + (c & 1) * (G::SBYTES / 4) + (w * BM + l31) * G::SSTRIDE + lh * 4;
#pragma unroll
      for (int g = 0; g < 4; ++g) *(f32x4*)(S + g * 8) = f32x4{acc[g * 4], acc[g * 4 + 1], acc[g * 4 + 2], acc[g * 4 + 3]};
    }
  };

  // ---- mixing waves: stage i.  PH: 0 = the one walk of a bank over the keys; 1 = first walk of a [K | V] bank (the summed logits
  // go to the workspace, nothing is mixed); 2 = its second walk.
  auto mix_stage = [&](int i, bool soft, bool mix, auto ph_t) {
    constexpr int PH = decltype(ph_t)::value;
    if constexpr (MIX) {
      const int j0 = jbase + i * BN;
      const unsigned char* Xprev = Xs0 + ((i + G::NXBUF - 1) % G::NXBUF) * G::XBYTES;
      const unsigned char* Vprev = Vs0 + ((i + 1) & 1) * G::VBYTES;
      f32x4 p4[4];
      if (soft) {
        const float* S = Sred0 + (i & 1) * (G::SBYTES / 4);
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) p4[ww] = *(const f32x4*)(S + (ww * BM + srow) * G::SSTRIDE + sp0);
      }
      // mixing of tile i - 1: operand fragments
      const int s16 = l & 15, g2 = (l >> 4) & 1;
      s16x4 y0[2][2], y1[2][2];
      bf16x8 pv[2];
      float al = 1.f;
      if (PH != 1 && mix) {
        const unsigned char* Pprev = Ps0 + ((i + 1) & 1) * G::PBYTES;
        al = alphas0[((i + 1) & 1) * BM + l31];
        const int ystride = w < 2 ? G::XSTRIDE : G::VSTRIDE;
        const unsigned char* ybase =
            (w < 2 ? Xprev + (G::PAD + lh * 8 + (s16 >> 2)) * G::XSTRIDE + (64 * w) * 2
                   : Vprev + (lh * 8 + (s16 >> 2)) * G::VSTRIDE + (64 * (w - 2)) * 2) + (16 * g2 + 4 * (s16 & 3)) * 2;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          pv[ks] = *(const bf16x8*)(Pprev + l31 * G::PSTRIDE + (ks * 16 + lh * 8) * 2);
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) {
            const unsigned char* yp = ybase + (ks * 16) * ystride + (ct * 32) * 2;
            y0[ks][ct] = lds_read_tr(yp);
            y1[ks][ct] = lds_read_tr(yp + 4 * ystride);
          }
        }
      }
      if (soft) {
        // the chunks requested a stage ago (key tile i + 3, value tile i) go to LDS, then the same registers receive key
        // tile i + 4 and value tile i + 1
        unsigned char* Xstage = Xs0 + ((i + 3) % G::NXBUF) * G::XBYTES;
#pragma unroll
        for (int it = 0; it < G::XPER; ++it) {
          put_x(it, Xstage, xreg[it]);
          xreg[it] = x_chunk(it, j0 + 4 * BN);
        }
        if (PH != 1) {
          unsigned char* Vstage = Vs0 + (i & 1) * G::VBYTES;
#pragma unroll
          for (int it = 0; it < G::VPER; ++it) {
            store_v(it, Vstage);
            load_v(it, j0 + BN);
          }
        }
      }
      if (PH != 1 && mix) {
        // (rarely) rescale the accumulators before tile i - 1 is mixed in
        if (__any(al != 1.0f)) {
#pragma unroll
          for (int ct = 0; ct < 2; ++ct)
#pragma unroll
            for (int q = 0; q < 16; ++q) oacc[ct][q] *= al;
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) {
            const s16x4 a0 = y0[ks][ct], a1 = y1[ks][ct];
            const s16x8 yy = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
            oacc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, yy), pv[ks], oacc[ct], 0, 0, 0);
          }
      }
      if (!soft) return;
      float sv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sv[e] = (PH == 2 ? pre[e] : 0.f) + (NORM == 0 || PH == 1 ? p4[0][e] + p4[1][e] : bias + p4[0][e] + p4[1][e]);
        sv[e] = sv[e] + p4[2][e] + p4[3][e];
      }
      if (PH == 1) {
        // first walk: this lane's four sums go to the workspace; the second walk reads them back (same lane, at device
        // scope: from the L2 the store went through to, whatever this CU's L1 holds from a step ago)
        const f32x4 v = {sv[0], sv[1], sv[2], sv[3]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), pre_rows, ((j0 / BN) * (BM * BN) + tid * 4) * 4, 0, 0);
        return;
      }
      if (PH == 2)                           // the next tile's, a whole stage before they are added
        pre = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(pre_rows, ((j0 / BN + 1) * (BM * BN) + tid * 4) * 4, 0, kDeviceScope));
      if (j0 + BN > T) {                     // tail tile: positions past T carry no weight
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j0 + sp0 + e >= T) sv[e] = NORM == 0 ? -INFINITY : 0.f;
      }
      if (PROT && j0 < m) {                  // neither do the positions of live protected slots (BN = 32: one mask word)
        uint32_t pmask = pwords[j0 >> 5];
        if (j0 + BN > m) pmask &= (1u << (m - j0)) - 1u;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((pmask >> (sp0 + e)) & 1u) sv[e] = NORM == 0 ? -INFINITY : 0.f;
      }
      float alpha = 1.f;
      if (NORM == 0) {
        // The reference only moves when the row maximum outgrows it by kLazy, so exp(s - ref) stays below e^kLazy and the
        // accumulators are rescaled rarely.  Every tile has a position < T, so mx is finite -- unless all 32 positions of
        // the tile are protected slots: such a tile adds nothing and leaves the reference alone.
        const float mx = group_max<G::LPR>(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])));
        const bool dead = PROT && mx == -INFINITY;
        const bool bump = !dead && mx > m_run + kLazy;
        const float m_new = bump ? mx : m_run;
        alpha = bump ? __expf(m_run - m_new) : 1.0f;
        const float mc = dead ? 0.f : m_new * kLog2e;
        m_run = m_new;
#pragma unroll
        for (int e = 0; e < 4; ++e) sv[e] = __builtin_amdgcn_exp2f(fmaf(sv[e], kLog2e, -mc));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) sv[e] = fmaxf(sv[e], 0.f);
      }
      float psum = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) psum += sv[e];
      l_run = l_run * alpha + group_sum<G::LPR>(psum);
      const u32x2 pk = {pack_bf16(sv[0], sv[1]), pack_bf16(sv[2], sv[3])};
      *(u32x2*)(Ps0 + (i & 1) * G::PBYTES + srow * G::PSTRIDE + sp0 * 2) = pk;
      if ((l % G::LPR) == 0) alphas0[(i & 1) * BM + srow] = alpha;
    }
  };
  // ends a stage: what was written to LDS is there (loads on their way stay on their way)
  auto meet = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  // a walk over tiles 0 .. NT - 1 of the range at hand.  Key tiles 0 (by either kind of wave), 1 and 2 are staged first, all loads
  // issued before the first store; key tile 3 and value tile 0 are on their way.
  auto walk = [&](auto ph_t) {
    constexpr int PH = decltype(ph_t)::value;
    if constexpr (MIX) {
      Cat16 x0[kMixersStageAll ? G::XPER : 1], x1[G::XPER], x2[G::XPER];
      if constexpr (kMixersStageAll) {
#pragma unroll
        for (int it = 0; it < G::XPER; ++it) x0[it] = x_chunk(it, jbase);
      }
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) x1[it] = x_chunk(it, jbase + BN);
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) x2[it] = x_chunk(it, jbase + 2 * BN);
      if (PH == 2) pre = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(pre_rows, ((jbase / BN) * (BM * BN) + tid * 4) * 4, 0, kDeviceScope));
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) xreg[it] = x_chunk(it, jbase + 3 * BN);
      if (PH != 1) {
#pragma unroll
        for (int it = 0; it < G::VPER; ++it) load_v(it, jbase);
      }
      if constexpr (kMixersStageAll) {
#pragma unroll
        for (int it = 0; it < G::XPER; ++it) put_x(it, Xs0, x0[it]);
      }
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) put_x(it, Xs0 + G::XBYTES, x1[it]);
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) put_x(it, Xs0 + 2 * G::XBYTES, x2[it]);
    } else if constexpr (!kMixersStageAll) {
      Cat16 x0[G::XPER];
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) x0[it] = x_chunk(it, jbase);
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) put_x(it, Xs0, x0[it]);
    }
    meet();
    logits_begin();
    logits_of(0);
    meet();
    for (int i = 0; i < NT; ++i) {
      if (i + 1 < NT) logits_of(i + 1);
      mix_stage(i, true, i > 0, ph_t);
      meet();
    }
    if (PH != 1) mix_stage(NT, false, true, ph_t);
  };

  constexpr std::integral_constant<int, 1> first{};
  constexpr std::integral_constant<int, CIN ? 2 : 0> main_walk{};
  for (int step = 0; step < sa.n_steps; ++step) {
  if (PIPE && (step & 1) != part) continue;            // the partner's step
  // A bank over [K | V] is walked twice, with the key half of the filters in the registers, then with the value half.  With
  // several chains per workgroup the first walks of all of them come first, so that a step costs two loads of a filter slice.
  // A pair of workgroups walks each range of a step twice instead (but for its first step): the range that does not wait for the
  // step before is then behind it when the chain is met.
  constexpr int kPasses = CIN && !PIPE ? 2 : 1;
  for (int pass = 0; pass < kPasses; ++pass) {
  if (CIN && !PIPE) {
    load_filters(pass);
    pin_filters();
  }
  for (int ci = 0; ci < n_mine; ++ci) {
  const int ch = grp + ci * groups;
  // ---- the step reads what every slot tile of this chain wrote in the step before
  if (!PIPE && pass == 0 && step > 0 && !chain_wait(ch, step)) return;
  int first_blk = 0, NT_all = 0;
  // ---- this step's inputs: source state, occupancy, block
  {
    const int b = ch / a.Hkv, hkv = ch % a.Hkv;
    if (PROT) pwords = a.protect + (int64_t)ch * a.protect_stride;
    const int64_t tok = (int64_t)step * sa.B;
    const int Bn = step == 0 ? a.Bn : (int)(sa.tokens_left - tok < sa.B ? sa.tokens_left - tok : sa.B);
    m = step == 0 ? a.m : a.M;
    T = m + Bn;
    NT = (T + BN - 1) / BN;
    if (PIPE) {                        // tiles from first_blk on read block rows only, halo included
      NT_all = NT;
      first_blk = (m + G::PAD + BN - 1) / BN;
      if (first_blk > NT_all) first_blk = NT_all;
    }
    if (PSPLIT) {                      // this part's range of position tiles (possibly empty)
      const int per = (NT + P - 1) / P, lo = part * per;
      const int hi = lo + per < NT ? lo + per : NT;
      jbase = lo * BN;
      NT = hi > lo ? hi - lo : 0;
    }
    const int64_t prev = (int64_t)((sa.slot0 + step - 1) % sa.ring) * sa.out_stride;   // (unused for step 0)
    const uint16_t* src_k = step == 0 ? (const uint16_t*)a.cache_k : (const uint16_t*)sa.out_k + prev;
    const uint16_t* src_v = step == 0 ? (const uint16_t*)a.cache_v : (const uint16_t*)sa.out_v + prev;
    cat_k = make_cat(src_k + (int64_t)ch * a.M * kD, m,
                     (const uint16_t*)a.k.p + b * a.k.sb + hkv * a.k.sh + tok * a.k.st, a.k.st, Bn);
    cat_v = make_cat(src_v + (int64_t)ch * a.M * kD, m,
                     (const uint16_t*)a.v.p + b * a.v.sb + hkv * a.v.sh + tok * a.v.st, a.v.st, Bn);
  }
  // (the two workgroups of a pair work on different steps at the same time: an area each)
  if (CIN)
    pre_rows = __builtin_amdgcn_make_buffer_rsrc((void*)(sa.prelogits + (int64_t)((ch * tiles + i0 / BM) * (PIPE ? 2 : 1) + (PIPE ? part : 0)) * sa.pre_stride), 0,
                                                 (int)sa.pre_stride * 4, 0x00020000);
  auto zero_state = [&]() {
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[ct][i] = 0.f;
    m_run = -INFINITY;
    l_run = 0.f;
  };
  // in the second walk the value rows are where the key rows were and the other way round
  auto trade = [&]() { const CatRows t = cat_k; cat_k = cat_v; cat_v = t; };
  if constexpr (PIPE) {
    zero_state();
    // first the tiles of the block alone, then, once the chain has been met, those that touch the cache
    if constexpr (CIN) {
      // Each is walked twice.  But a step that has nobody to wait for (the first of a launch) takes the first walk of all its
      // tiles at once: two loads of a filter slice and three walks instead of four of either (a step of 64 tokens on 64 slots,
      // 8 heads, width 21: 21.9 -> 18.7 us, 96 on 96: 25.4 -> 22.3; either way the same sums in the same order).
      const bool alone = step == 0;
      for (int leg = 0; leg < 2; ++leg) {
        const bool both = !(alone && leg == 1);
        if (both) load_filters(0);
        if (leg == 1) {
          if (step > 0 && !chain_wait(ch, step)) return;
        }
        jbase = alone || leg == 1 ? 0 : first_blk * BN;
        NT = alone ? NT_all : leg == 0 ? NT_all - first_blk : first_blk;
        if (both && NT > 0) {
          pin_filters();
          walk(first);
          load_filters(1);
          __syncthreads();                   // the next prologue writes the tiles this walk read last
          pin_filters();
          trade();
        }
        jbase = leg == 0 ? first_blk * BN : 0;
        NT = leg == 0 ? NT_all - first_blk : first_blk;
        if (NT > 0) {
          walk(main_walk);
          if (!alone) trade();
        }
        if (leg == 0) __syncthreads();
      }
      if (!alone) trade();
    } else {
      for (int leg = 0; leg < 2; ++leg) {
        if (leg == 1) {
          if (step > 0 && !chain_wait(ch, step)) return;
        }
        jbase = leg == 0 ? first_blk * BN : 0;
        NT = leg == 0 ? NT_all - first_blk : first_blk;
        if (NT > 0) walk(main_walk);
        if (leg == 0) __syncthreads();
      }
    }
  } else {
    if (CIN && pass == 0) {
      if (NT > 0) walk(first);
      __syncthreads();                       // (as above)
      continue;
    }
    if (CIN) trade();
    zero_state();                            // (a part without positions hands in an empty result)
    if (NT > 0) walk(main_walk);
  }

  uint16_t* nk;
  uint16_t* nv;
  {
    const int64_t out_at = (int64_t)((sa.slot0 + step) % sa.ring) * sa.out_stride + ((int64_t)ch * a.M + i0) * kD;
    // (after the second walk of a [K | V] bank the accumulator's first d columns are the value rows)
    nk = (uint16_t*)(CIN ? sa.out_v : sa.out_k) + out_at;
    nv = (uint16_t*)(CIN ? sa.out_k : sa.out_v) + out_at;
  }
  if constexpr (PSPLIT) {
    // ---- this part's result goes to the workspace: accumulators [slot][2 d] as they are
    // (unnormalised, relative to this part's reference), then the references, then the row sums
    float* mine = sa.partials + ((int64_t)(ch * tiles + i0 / BM) * P + part) * G::PART_FLOATS;
    if constexpr (MIX) {
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = {oacc[ct][g * 4 + 0], oacc[ct][g * 4 + 1], oacc[ct][g * 4 + 2], oacc[ct][g * 4 + 3]};
        *(f32x4*)(mine + l31 * (2 * kD) + 64 * w + ct * 32 + g * 8 + lh * 4) = v;
      }
    if ((l % G::LPR) == 0) {
      mine[BM * 2 * kD + srow] = m_run;
      mine[BM * 2 * kD + BM + srow] = l_run;
    }
    }
    // ---- hand-off.  The parts of a (chain, tile) count themselves in; the one that completes the
    // count merges.  Two forms, as for the meeting of a chain: when all parts run on one XCD they
    // share its L2, so a part's stores have arrived once its store counter is at zero and the merging
    // part reads them at device scope (from the L2); otherwise device-scope release / acquire.  Which
    // form applies is read from the census word of the (chain, tile), where every part registered
    // its XCD when the kernel started: P registrations, all in this workgroup's field.  (A part that
    // looks before everybody has registered takes the general form, which is always safe.)
    uint32_t* cnt = sa.psync + 2 * (ch * tiles + i0 / BM);
    if (wg_tid == 0) {
      const uint32_t xcd = __builtin_amdgcn_s_getreg(20 | ((4 - 1) << 11)) & 7u;   // XCC_ID
      split_fast = sa.same_l2_allowed &&
                   __hip_atomic_load(cnt + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ((uint32_t)P << (3u * xcd));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const bool fast = split_fast != 0;
    if (wg_tid == 0) {
      const uint32_t old = fast ? __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                : __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      i_merge = (old + 1u) % (uint32_t)P == 0u;
    }
    __syncthreads();
    if (!i_merge) continue;              // the merging part signals the chain; this one goes on to the next step
    // ---- merge: reference = the largest of the parts' references; every part's sums and
    // accumulators are scaled to it and added in the order of the parts.  All loads are issued
    // before the first is used: one trip to the L2 for the lot.
    float* scale_s = Sred0;              // [part][slot]
    float* inv_s = Sred0 + 4 * BM;        // 1 / row sum
    const __amdgpu_buffer_rsrc_t parts = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(sa.partials + (int64_t)(ch * tiles + i0 / BM) * P * G::PART_FLOATS), 0, P * G::PART_FLOATS * 4, 0x00020000);
    constexpr int kIters = BM * (2 * kD / 4) / kRoleThreads;      // (slot, four columns of [K | V]) chunks per thread
    u32x4 raw[kIters][4];
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const int e = wg_tid + it * kRoleThreads, slot = e / (2 * kD / 4), c4 = e % (2 * kD / 4);
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P)
          raw[it][p] = __builtin_amdgcn_raw_buffer_load_b128(parts, (p * G::PART_FLOATS + slot * (2 * kD) + c4 * 4) * 4, 0, kDeviceScope);
    }
    if (wg_tid < BM) {
      float mp[4], lp[4], mstar = -INFINITY;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P) {
          mp[p] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(parts, (p * G::PART_FLOATS + BM * 2 * kD + wg_tid) * 4, 0, kDeviceScope));
          lp[p] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(parts, (p * G::PART_FLOATS + BM * 2 * kD + BM + wg_tid) * 4, 0, kDeviceScope));
        }
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P) mstar = fmaxf(mstar, mp[p]);
      float lsum_all = 0.f;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P) {
          const float sc = (NORM == 0) ? (mp[p] == -INFINITY ? 0.f : __expf(mp[p] - mstar)) : 1.0f;
          scale_s[p * BM + wg_tid] = sc;
          lsum_all += sc * lp[p];
        }
      inv_s[wg_tid] = 1.0f / (NORM == 0 ? lsum_all : lsum_all + a.eps);
    }
    __syncthreads();
    uint32_t keep = 0;                     // live protected slots keep their old rows (BM = 32: one mask word)
    if (PROT && i0 < m) {
      keep = pwords[i0 >> 5];
      if (i0 + 32 > m) keep &= (1u << (m - i0)) - 1u;
    }
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const int e = wg_tid + it * kRoleThreads, slot = e / (2 * kD / 4), c4 = e % (2 * kD / 4);
      if (PROT && ((keep >> slot) & 1u)) continue;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P) {
          const float sc = scale_s[p * BM + slot];
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[q] = fmaf(sc, __uint_as_float(raw[it][p][q]), acc[q]);
        }
      const float inv = inv_s[slot];
      u32x2 pk;
      pk[0] = pack_bf16(acc[0] * inv, acc[1] * inv);
      pk[1] = pack_bf16(acc[2] * inv, acc[3] * inv);
      uint16_t* dst = (c4 < kD / 4 ? nk : nv) + (int64_t)slot * kD + (c4 % (kD / 4)) * 4;
      *(u32x2*)dst = pk;
    }
    if (PROT && keep) {
#pragma unroll
      for (int it = 0; it < 2 * BM * 16 / kRoleThreads; ++it) {
        const int e = wg_tid + it * kRoleThreads;
        const int kv = e / (BM * 16), r = (e >> 4) % BM, c16 = e & 15;
        if ((keep >> r) & 1u) {
          const int off = (i0 + r) * (kD * 2) + c16 * 16;
          *(u32x4*)((kv ? nv : nk) + (int64_t)r * kD + c16 * 8) =
              __builtin_amdgcn_raw_buffer_load_b128(kv ? cat_v.cache : cat_k.cache, off, 0, kDeviceScope);
        }
      }
    }
  } else {
  // ---- normalise by the row sums and store the new cache rows.  A lane holds 4 columns of a
  // slot at a time; the rows are put together in the key-tile area of LDS (free after the last
  // stage) and leave as whole rows, 1 KB of contiguous memory per wave instruction.
  if (MIX && (l % G::LPR) == 0) lsum[srow] = l_run;
  __syncthreads();
  unsigned char* Orows = Xs0;                // [K rows of the tile ; V rows of the tile][XSTRIDE]
  static_assert(2 * BM * G::XSTRIDE <= G::NXBUF * G::XBYTES, "the output rows fit the key-tile area");
  uint32_t keep = 0;                         // a live protected slot keeps its old row (copied below) instead of Eq. 4a / 4b
  if (PROT && i0 < m) {
    keep = pwords[i0 >> 5];
    if (i0 + 32 > m) keep &= (1u << (m - i0)) - 1u;
  }
  if constexpr (MIX) {
    const float inv = 1.0f / (NORM == 0 ? lsum[l31] : lsum[l31] + a.eps);
    unsigned char* orow = Orows + ((w >> 1) * BM + l31) * G::XSTRIDE + (64 * (w & 1)) * 2;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        u32x2 pk;
        pk[0] = pack_bf16(oacc[ct][g * 4 + 0] * inv, oacc[ct][g * 4 + 1] * inv);
        pk[1] = pack_bf16(oacc[ct][g * 4 + 2] * inv, oacc[ct][g * 4 + 3] * inv);
        *(u32x2*)(orow + (ct * 32 + g * 8 + lh * 4) * 2) = pk;
      }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 2 * BM * 16 / kRoleThreads; ++it) {  // (K or V, slot, 16-byte chunk)
    const int e = wg_tid + it * kRoleThreads;
    const int kv = e / (BM * 16), r = (e >> 4) % BM, c16 = e & 15;
    uint16_t* dst = (kv ? nv : nk) + (int64_t)r * kD + c16 * 8;
    if (PROT && ((keep >> r) & 1u)) {                        // live protected slot: inside the cache resources
      const int off = (i0 + r) * (kD * 2) + c16 * 16;
      *(u32x4*)dst = __builtin_amdgcn_raw_buffer_load_b128(kv ? cat_v.cache : cat_k.cache, off, 0, kDeviceScope);
    } else {
      *(u32x4*)dst = *(const u32x4*)(Orows + (kv * BM + r) * G::XSTRIDE + c16 * 16);
    }
  }
  }  // not split

  // ---- the rows are on their way: tell the other tiles of the chain.  (The barrier also keeps
  // the next prologue's LDS stores behind the copy-out above.)
  if (step + 1 < sa.n_steps) chain_signal(ch);
  else __syncthreads();
  }  // chains
  }  // passes
  }  // steps
  };
  if (mixer) run(std::true_type{});
  else run(std::false_type{});
}

}  // namespace compress_detail
}  // namespace lococo
