// The work of one workgroup of the fused compression kernel, included as the body of the kernels that have it (template
// parameters BM, KW, NORM, PROT, MULTI, SPLIT, LOG, as described in compress_tile.h).  In scope: ScanArgs sa, wp,
// wp_head_stride, smem (Geo<BM, KW>::LDS bytes), and wg_id of wg_count.  It is text and not an inlined function because the
// 64-slot builds use all 512 registers: as a function the same code spilled differently and the 32 K-token scan took 4 % longer.
  using G = Geo<BM, KW>;
  static_assert(!SPLIT || (BM == 32 && !MULTI), "the splits are built for 32-slot tiles, one chain per workgroup");
  constexpr bool PSPLIT = SPLIT == 1, PIPE = SPLIT == 2;
  const StepArgs& a = sa.st;
  unsigned char* Xs0 = smem;                                    // NXBUF key tiles (with halo)
  unsigned char* Vs0 = Xs0 + G::NXBUF * G::XBYTES;              // NVBUF value tiles
  float* Sred = (float*)(Vs0 + G::NVBUF * G::VBYTES);           // 4 partial-logit tiles [wave][slot][pos]
  unsigned char* Ps0 = (unsigned char*)Sred + G::SBYTES;        // 2 probability tiles [slot][pos], bf16
  float* alphas0 = (float*)(Ps0 + 2 * G::PBYTES);               // 2 x rescale factor per slot
  float* lsum = alphas0 + 2 * BM;                               // final row sums

  // (the wave index as a scalar: everything derived from it stays on the scalar unit, and the
  // choices between the key and the value side of the mixing are uniform branches)
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, l31 = l & 31, lh = l >> 5;
  // Workgroups are dealt to the 8 XCDs round-robin by their linear id.  The slot tiles of one chain
  // all read the same keys and values, so they are given ids that land on one XCD (one L2).
  int item = wg_id;
  {
    const int per = wg_count / 8;
    if (item < per * 8) item = (item % 8) * per + item / 8;
  }
  const int tiles = a.M / BM;
  // position split: consecutive work items are the parts of one (chain, slot tile), so they land on one XCD
  const int P = SPLIT ? sa.psplit : 1;
  const int part = SPLIT ? item % P : 0;
  if (SPLIT) item /= P;
  // A workgroup owns one slot tile of the chains grp, grp + groups, grp + 2 groups, ...  (one chain
  // when the launch has a workgroup per chain and tile).  Where filters or biases differ between
  // kv heads the host picks `groups` as a multiple of Hkv, so all of them belong to head hkv0.
  const int grp = item / tiles, groups = wg_count / (tiles * P), n_chains = a.batch * a.Hkv;
  const int hkv0 = grp % a.Hkv;
  const int i0 = (item % tiles) * BM;
  // per-step and per-chain quantities, set at the top of the loops
  int T = 0, m = 0, NT = 0;
  int jbase = 0;            // first position of this workgroup's range (0 unless the positions are split)
  CatRows cat_k, cat_v;
  // protected-slot bits of the chain at hand (see lococo_cache.protect), or null
  const uint32_t* pwords = nullptr;

  // ---- this wave's slice of the filter bank, resident in registers for the whole kernel:
  // lane (slot l31 of tile rt, channels 32w + 16h + 8*lh ..) for every tap
  bf16x8 wreg[G::RT][KW][2];
  {
    const uint16_t* wb = wp + hkv0 * wp_head_stride;
#pragma unroll
    for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
      for (int t = 0; t < KW; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          wreg[rt][t][h] =
              *(const bf16x8*)(wb + ((((int64_t)(i0 / 32 + rt) * 4 + w) * KW + t) * 2 + h) * 512 + l * 8);
    // Pin the filters to the accumulation-register half of the register file: the MFMA reads
    // them from there directly, which leaves the other 256 registers to everything else.
#pragma unroll
    for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
      for (int t = 0; t < KW; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) asm volatile("" : "+a"(wreg[rt][t][h]));
  }
  __amdgpu_buffer_rsrc_t log_rows = __builtin_amdgcn_make_buffer_rsrc((void*)sa.logits, 0, 0, 0x00020000);

  // mixing accumulator, transposed: lane = slot rt*32 + l31, rows = columns 64w + ct*32 + (i/4)*8 + lh*4 + i%4
  f32x16 oacc[2][G::RT];

  // softmax state of the slot this lane helps with (replicated over the LPR lanes of the slot)
  const int srow = w * G::RPW + l / G::LPR;
  const int sp0 = (l % G::LPR) * G::EPL;
  float m_run = 0.f, l_run = 0.f;
  // (a softmax over the positions does not see a per-slot constant: the bias only enters the relu-sum form)
  const float bias =
      a.conv_b ? __uint_as_float((uint32_t)((const uint16_t*)a.conv_b)[hkv0 * a.b_head_stride + i0 + srow] << 16)
               : 0.f;

  // ---- staging: global -> registers -> LDS (key tile with halo, value tile; both row-major)
  Cat16 xreg[G::XPER];
  Cat16 vreg[G::VPER];
  auto load_x = [&](int it, int j0) {
    const int item = tid + it * kThreads;
    xreg[it] = load_cat16(cat_k, j0 - G::PAD + (item >> 4), item & 15);
  };
  auto load_v = [&](int it, int j0) {
    const int item = tid + it * kThreads;
    vreg[it] = load_cat16(cat_v, j0 + (item >> 4), item & 15);
  };
  // the two halves of a chunk's fetch on their own, for stages that give each a slot of its own
  auto load_half = [&](Cat16& r, const CatRows& c, int p, int chunk, bool blk) {
    if (blk) r.from_blk = __builtin_amdgcn_raw_buffer_load_b128(c.blk, (p - c.m) * c.blk_stride + chunk * 16, 0, 0);
    else r.from_cache = __builtin_amdgcn_raw_buffer_load_b128(c.cache, p * (kD * 2) + chunk * 16, 0, kDeviceScope);
  };
  auto store_x = [&](int it, int j0, unsigned char* Xs) {
    const int item = tid + it * kThreads;
    (void)j0;
    *(u32x4*)(Xs + (item >> 4) * G::XSTRIDE + (item & 15) * 16) = xreg[it].from_cache | xreg[it].from_blk;
  };
  auto store_v = [&](int it, int j0, unsigned char* Vs) {
    const int item = tid + it * kThreads;
    (void)j0;
    *(u32x4*)(Vs + (item >> 4) * G::VSTRIDE + (item & 15) * 16) = vreg[it].from_cache | vreg[it].from_blk;
  };

  // Ring of key operands of the logit MFMAs, fetched kRing-1 contraction steps ahead.  kRing
  // divides the number of steps, so the last steps of a stage fetch the first operands of the
  // next stage into the slots that stage expects and the matrix pipe never waits at a stage start.
  constexpr int kRing = G::NS % 5 == 0 ? 5 : (G::NS % 6 == 0 ? 6 : 7);
  static_assert(G::NS % kRing == 0, "operand ring must wrap exactly at a stage boundary");
  bf16x8 xv[kRing];

  // Partial logits of one tile, summed over this wave's channel quarter:
  // sacc[rt] lane = slot rt*32 + l31, rows = positions (i/4)*8 + lh*4 + i%4.
  f32x16 sacc[G::RT];
  // Publish them: 16-byte stores, 4 consecutive positions of one slot each.
  auto write_partials = [&]() {
#pragma unroll
    for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = {sacc[rt][g * 4 + 0], sacc[rt][g * 4 + 1], sacc[rt][g * 4 + 2], sacc[rt][g * 4 + 3]};
        *(f32x4*)(Sred + (w * BM + rt * 32 + l31) * G::SSTRIDE + g * 8 + lh * 4) = v;
      }
  };

  // One pipeline stage.  With tile index i it runs, interleaved:
  //   DoConv:    logits of tile i+1 (key tile buffer (i+1)%5) into sacc, published at the end;
  //   DoSoftmax: reduction + softmax of tile i (partials in Sred) into Ps[i&1], alphas[i&1];
  //              staging of key tile i+3 and value tile i (loaded during the previous stage);
  //   DoMix:     mixing of tile i-1 (Ps[(i-1)&1], key tile buffer (i-1)%5, value buffer (i-1)&1).
  //
  // Issue model.  A wave issues in order and the matrix pipe takes one MFMA every 32 cycles, so
  // after each MFMA there is room for about seven other instructions before the next MFMA can
  // issue anyway.  Everything that is not a logit MFMA is therefore cut into micro-slices of a few
  // instructions, one per MFMA ("slot" 2*st + rt), with every load issued several slots before
  // the slice that consumes it.
  //
  // Barriers.  B1 (slot 5) publishes what the previous stage wrote to LDS -- partial logits,
  // probabilities, rescale factors, staged tiles -- so everything read before it (the key tile of
  // this stage's logits) was staged two stages ago.  B2 (slot 19) comes after every wave has
  // consumed this tile's partial logits; the buffer is rewritten at the end of the stage.
  // Neither needs outstanding global loads to finish, so they are plain barriers preceded by a
  // wait on the LDS counter only.
  // RI: the tile index modulo the period of the buffer rings (key tiles: NXBUF; values, probabilities,
  // rescale factors: 2) where the caller knows it at compile time, so that every buffer address of the
  // stage is a constant; -1: computed from i.
  auto stage = [&](int i, auto do_conv, auto do_softmax, auto do_mix_t, auto ring_t) {
    constexpr bool DoConv = decltype(do_conv)::value, DoSoftmax = decltype(do_softmax)::value;
    constexpr bool DoMix = decltype(do_mix_t)::value;
    constexpr int RI = decltype(ring_t)::value;
    const int ib = RI >= 0 ? RI + 2 * G::NXBUF : i;      // (kept positive: ib - 1 enters a remainder)
    const int j0 = (SPLIT ? jbase : 0) + i * BN;
    const unsigned char* Xnext = Xs0 + ((ib + 1) % G::NXBUF) * G::XBYTES;
    const unsigned char* Xnext2 = Xs0 + ((ib + 2) % G::NXBUF) * G::XBYTES;
    const unsigned char* Xprev = Xs0 + ((ib + G::NXBUF - 1) % G::NXBUF) * G::XBYTES;
    unsigned char* Xstage = Xs0 + ((ib + 3) % G::NXBUF) * G::XBYTES;
    const unsigned char* Vprev = Vs0 + ((ib - 1) & 1) * G::VBYTES;
    unsigned char* Vstage = Vs0 + (ib & 1) * G::VBYTES;
    unsigned char* Pcur = Ps0 + (ib & 1) * G::PBYTES;
    const unsigned char* Pprev = Ps0 + ((ib - 1) & 1) * G::PBYTES;
    float* alpha_cur = alphas0 + (ib & 1) * BM;
    const float* alpha_prev = alphas0 + ((ib - 1) & 1) * BM;

    // logits: operands of step st come from this stage's key tile, those of steps >= NS are the
    // first operands of the next stage's tile
    const int xlane = l31 * G::XSTRIDE + (32 * w + lh * 8) * 2;
    auto fetch = [&](int st) {
      const unsigned char* xb = (st < G::NS ? Xnext : Xnext2) + xlane;
      const int s2 = st < G::NS ? st : st - G::NS;
      xv[st % kRing] = *(const bf16x8*)(xb + (s2 >> 1) * G::XSTRIDE + (s2 & 1) * 32);
    };
    // protected positions of tile i (bits of live protected slots; BN = 32 = one mask word)
    uint32_t pmask = 0;
    if (PROT && DoSoftmax && j0 < m) {
      pmask = pwords[j0 >> 5];
      if (j0 + BN > m) pmask &= (1u << (m - j0)) - 1u;
    }
    // softmax of tile i
    constexpr int E4 = G::EPL / 4;
    f32x4 part[4][E4];
    float sv[G::EPL];
    float mx = 0.f, m_new = 0.f, mc = 0.f, alpha = 1.f, psum = 0.f;
    bool bump = false;
    uint32_t packed[G::EPL / 2];
    auto sm_issue = [&](int ww) {
#pragma unroll
      for (int e4 = 0; e4 < E4; ++e4)
        part[ww][e4] = *(const f32x4*)(Sred + (ww * BM + srow) * G::SSTRIDE + sp0 + e4 * 4);
    };
    auto sm_add = [&](int ww0, int e4) {      // 4 positions: + partials ww0 and ww0+1
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sv[e4 * 4 + e] = ww0 == 0 ? (NORM == 0 ? part[0][e4][e] + part[1][e4][e] : bias + part[0][e4][e] + part[1][e4][e])
                                  : sv[e4 * 4 + e] + part[ww0][e4][e] + part[ww0 + 1][e4][e];
    };
    auto sm_exp = [&](int e) {
      sv[e] = NORM == 0 ? __builtin_amdgcn_exp2f(fmaf(sv[e], kLog2e, -mc)) : fmaxf(sv[e], 0.f);
    };
    // mixing of tile i-1: operand fragments, fetched ahead of the MFMAs that follow the loop
    const int s16 = l & 15, g2 = (l >> 4) & 1;
    const unsigned char* ybase =
        (w < 2 ? Xprev + (G::PAD + lh * 8 + (s16 >> 2)) * G::XSTRIDE + (64 * w) * 2
               : Vprev + (lh * 8 + (s16 >> 2)) * G::VSTRIDE + (64 * (w - 2)) * 2) +
        (16 * g2 + 4 * (s16 & 3)) * 2;
    const int ystride = w < 2 ? G::XSTRIDE : G::VSTRIDE;
    bf16x8 pv[2][G::RT];
    s16x4 y0[2][2], y1[2][2];
    float al[G::RT];
    auto mix_fetch_p = [&](int ks) {
#pragma unroll
      for (int rt = 0; rt < G::RT; ++rt)
        pv[ks][rt] = *(const bf16x8*)(Pprev + (rt * 32 + l31) * G::PSTRIDE + (ks * 16 + lh * 8) * 2);
    };
    auto mix_fetch_y = [&](int ks, int ct) {
      const unsigned char* yp = ybase + (ks * 16) * ystride + (ct * 32) * 2;
      y0[ks][ct] = lds_read_tr(yp);
      y1[ks][ct] = lds_read_tr(yp + 4 * ystride);
    };
    auto mix_mfma = [&](int ks, int ct) {
      const s16x4 a0 = y0[ks][ct], a1 = y1[ks][ct];
      const s16x8 yy = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
      const bf16x8 yv = __builtin_bit_cast(bf16x8, yy);
#pragma unroll
      for (int rt = 0; rt < G::RT; ++rt)
        oacc[ct][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(yv, pv[ks][rt], oacc[ct][rt], 0, 0, 0);
    };

    // The micro-slices.  `slot` counts logit MFMAs of the stage: 0 .. RT*NS-1.
    constexpr int kSlots = G::RT * G::NS;
    constexpr int S = G::RT;                   // slots per contraction step
    auto micro = [&](int slot) {
      if (slot == 2 * S + S - 1) {             // B1
        __builtin_amdgcn_s_waitcnt(0xc07f);    // lgkmcnt(0): this wave's LDS stores of the last stage landed
        __builtin_amdgcn_s_barrier();
      }
      if (DoSoftmax) {
        // partial logits of tile i: four 16/32-byte reads, then the sums, a few steps later
        if (slot >= 3 * S && slot < 3 * S + 4) sm_issue(slot - 3 * S);
        // staging: the chunks loaded during the previous stage (key tile i+3, value tile i) go to
        // LDS, then the same registers receive key tile i+4 and value tile i+1: a whole stage
        // of latency cover, enough for a first touch that has to come from HBM
        // With 60 slots in a stage the 15 pieces (LDS store, cache-side fetch, block-side fetch of each
        // chunk) get a slot each, in the slots the softmax leaves free at the end of the stage: one LDS
        // store or one load fits the shadow of an MFMA, a store and two loads together do not.
        constexpr int kPieces = 3 * (G::XPER + G::VPER);
        constexpr bool kSpread = kSlots - kPieces - 1 >= kSlots * 3 / 5 + 8;   // behind the softmax and the mixing fetches
        if (kSpread) {
          constexpr int Z0 = kSlots - kPieces - 1;
          if (slot >= Z0 && slot < Z0 + kPieces) {
            const int piece = slot - Z0, it = piece / 3, what = piece % 3;
            if (it < G::XPER) {
              const int item = tid + it * kThreads, jn = j0 + 4 * BN;
              if (what == 0) store_x(it, j0 + 3 * BN, Xstage);
              else load_half(xreg[it], cat_k, jn - G::PAD + (item >> 4), item & 15, what == 2);
            } else {
              const int iv = it - G::XPER, item = tid + iv * kThreads;
              if (what == 0) store_v(iv, j0, Vstage);
              else load_half(vreg[iv], cat_v, j0 + BN + (item >> 4), item & 15, what == 2);
            }
          }
        } else {
          if (slot >= 5 * S && slot < 5 * S + G::XPER) {
            store_x(slot - 5 * S, j0 + 3 * BN, Xstage);
            load_x(slot - 5 * S, j0 + 4 * BN);
          }
          if (slot >= 5 * S + G::XPER && slot < 5 * S + G::XPER + G::VPER) {
            store_v(slot - 5 * S - G::XPER, j0, Vstage);
            load_v(slot - 5 * S - G::XPER, j0 + BN);
          }
        }
        if (slot >= 8 * S && slot < 8 * S + E4) sm_add(0, slot - 8 * S);
        if (slot >= 8 * S + E4 && slot < 8 * S + 2 * E4) sm_add(2, slot - 8 * S - E4);
        if (slot == 8 * S + 2 * E4) __builtin_amdgcn_s_barrier();   // B2: the partial logits have been consumed
        if (LOG == 1 && slot == 8 * S + 2 * E4 + 1) {       // the logits as they are, for the backward pass
#pragma unroll
          for (int e4 = 0; e4 < E4; ++e4) {
            const f32x4 v = {sv[e4 * 4], sv[e4 * 4 + 1], sv[e4 * 4 + 2], sv[e4 * 4 + 3]};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), log_rows, (srow * sa.logits_ld + sp0 + e4 * 4) * 4, j0 * 4, 0);
          }
        }
        if (slot == 8 * S + 2 * E4 + 1) {
          if (j0 + BN > T) {                   // tail tile: positions past T carry no weight
#pragma unroll
            for (int e = 0; e < G::EPL; ++e)
              if (j0 + sp0 + e >= T) sv[e] = NORM == 0 ? -INFINITY : 0.f;
          }
          if (PROT && pmask) {                 // neither do the positions of protected slots
#pragma unroll
            for (int e = 0; e < G::EPL; ++e)
              if ((pmask >> (sp0 + e)) & 1u) sv[e] = NORM == 0 ? -INFINITY : 0.f;
          }
          if (NORM == 0) {
            mx = sv[0];
#pragma unroll
            for (int e = 1; e < G::EPL; ++e) mx = fmaxf(mx, sv[e]);
          }
        }
        if (NORM == 0 && slot == 8 * S + 2 * E4 + 2) mx = group_max<G::LPR>(mx);
        if (NORM == 0 && slot == 8 * S + 2 * E4 + 3) {
          // The reference only moves when the row maximum outgrows it by kLazy, so exp(s - ref)
          // stays below e^kLazy and the accumulators are rescaled rarely.  Every tile has a
          // position < T, so mx is finite -- unless all 32 positions of the tile are protected
          // slots: such a tile adds nothing and leaves the reference alone.
          const bool dead = PROT && mx == -INFINITY;
          bump = !dead && mx > m_run + kLazy;
          m_new = bump ? mx : m_run;
          alpha = bump ? __expf(m_run - m_new) : 1.0f;
          mc = dead ? 0.f : m_new * kLog2e;
        }
        constexpr int X0 = 8 * S + 2 * E4 + 4;   // one exponential per slot
        if (slot >= X0 && slot < X0 + G::EPL) sm_exp(slot - X0);
        if (slot == X0 + G::EPL) {
#pragma unroll
          for (int e = 0; e < G::EPL; ++e) psum += sv[e];
        }
        if (slot == X0 + G::EPL + 1) {
          psum = group_sum<G::LPR>(psum);
          l_run = l_run * alpha + psum;
          m_run = m_new;
        }
        if (slot == X0 + G::EPL + 2) {
#pragma unroll
          for (int e2 = 0; e2 < G::EPL / 2; ++e2) packed[e2] = pack_bf16(sv[2 * e2], sv[2 * e2 + 1]);
        }
        if (slot == X0 + G::EPL + 3) {
#pragma unroll
          for (int e4 = 0; e4 < E4; ++e4) {
            const u32x2 pk = {packed[2 * e4], packed[2 * e4 + 1]};
            *(u32x2*)(Pcur + srow * G::PSTRIDE + (sp0 + e4 * 4) * 2) = pk;
          }
          if ((l % G::LPR) == 0) alpha_cur[srow] = alpha;
        }
      }
      if (DoMix) {
        constexpr int M0 = kSlots * 3 / 5;       // operand fragments of tile i-1's mixing, one fetch per slot
        if (slot == M0) {
#pragma unroll
          for (int rt = 0; rt < G::RT; ++rt) al[rt] = alpha_prev[rt * 32 + l31];
        }
        if (slot == M0 + 1) mix_fetch_p(0);
        if (slot == M0 + 2) mix_fetch_p(1);
        if (slot == M0 + 3) mix_fetch_y(0, 0);
        if (slot == M0 + 4) mix_fetch_y(0, 1);
        if (slot == M0 + 5) mix_fetch_y(1, 0);
        if (slot == M0 + 6) mix_fetch_y(1, 1);
        // (rarely) rescale the accumulators before tile i-1 is mixed in
        if (slot == M0 + 7) {
          bool any = false;
#pragma unroll
          for (int rt = 0; rt < G::RT; ++rt) any |= al[rt] != 1.0f;
          if (__any(any)) {
#pragma unroll
            for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
              for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                for (int q = 0; q < 16; ++q) oacc[ct][rt][q] *= al[rt];
          }
        }
      }
    };

    if (DoConv && i < 0) {                     // only the very first stage has nobody to fetch for it
#pragma unroll
      for (int st = 0; st < kRing - 1; ++st) fetch(st);
    }
    __builtin_amdgcn_sched_barrier(0);

#pragma unroll
    for (int st = 0; st < G::NS; ++st) {
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int rt = 0; rt < G::RT; ++rt) {
        if (DoConv) {
          sacc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv[st % kRing], wreg[rt][st >> 1][st & 1],
                                                             st == 0 ? zero : sacc[rt], 0, 0, 0);
          if (rt == G::RT - 1) fetch(st + kRing - 1);   // the ring slot of step st-1 is free now
        }
        micro(st * S + rt);
        __builtin_amdgcn_sched_barrier(0);     // pin the order: MFMA, then this slot's slice
      }
    }
    // Mixing MFMAs of tile i-1 run while the last logit MFMAs drain; the partial logits are
    // published in between.  The next stage's B1 makes them visible.
    if (DoMix && DoConv) {
      // one partial-logit store behind each mixing MFMA: the stores issue in the shadow of the matrix
      // pipe instead of as one burst
      int nw = 0;
      auto one_write = [&]() {
        const int rt = nw / 4, g = nw % 4;
        if (rt < G::RT) {
          const f32x4 v = {sacc[rt][g * 4 + 0], sacc[rt][g * 4 + 1], sacc[rt][g * 4 + 2], sacc[rt][g * 4 + 3]};
          *(f32x4*)(Sred + (w * BM + rt * 32 + l31) * G::SSTRIDE + g * 8 + lh * 4) = v;
        }
        ++nw;
      };
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          const s16x4 a0 = y0[ks][ct], a1 = y1[ks][ct];
          const s16x8 yy = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
          const bf16x8 yv = __builtin_bit_cast(bf16x8, yy);
#pragma unroll
          for (int rt = 0; rt < G::RT; ++rt) {
            oacc[ct][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(yv, pv[ks][rt], oacc[ct][rt], 0, 0, 0);
            one_write();
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      while (nw < 4 * G::RT) one_write();
    } else {
      if (DoMix) { mix_mfma(0, 0); mix_mfma(0, 1); }
      if (DoConv) write_partials();
      if (DoMix) { mix_mfma(1, 0); mix_mfma(1, 1); }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

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
  __shared__ int bail;                       // a chain wait timed out: leave
  __shared__ int same_l2;
  if (tid == 0) { bail = 0; same_l2 = 0; }
  __syncthreads();
  auto chain_signal = [&](int c) {
    const bool fast = same_l2 != 0;          // LDS word written before the previous workgroup barrier
    if (fast) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      if (fast) __hip_atomic_fetch_add(sa.sync + c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else __hip_atomic_fetch_add(sa.sync + c, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  auto chain_wait = [&](int c, int round) -> bool {
    if (tid == 0) {
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
  if (PSPLIT && tid == 0) {
    // every part registers the XCD it runs on in the census word of its (chain, tile); read at the hand-off
    const uint32_t xcd = __builtin_amdgcn_s_getreg(20 | ((4 - 1) << 11)) & 7u;
    __hip_atomic_fetch_add(sa.psync + 2 * (grp * tiles + i0 / BM) + 1, 1u << (3u * xcd), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  }
  if (sa.n_steps > 1) {
    uint32_t* xcd_mask = sa.sync + n_chains + 1;
    if (tid == 0) {
      const uint32_t xcd = __builtin_amdgcn_s_getreg(20 | ((4 - 1) << 11));   // XCC_ID, bits [3:0]
      for (int c = grp; c < n_chains; c += groups)
        __hip_atomic_fetch_or(xcd_mask + c, 1u << xcd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int c = grp; c < n_chains; c += groups) chain_signal(c);
    bool one_xcd = true;
    for (int c = grp; c < n_chains; c += groups) {
      if (!chain_wait(c, 0)) return;
      if (tid == 0) {
        const uint32_t mask = __hip_atomic_load(xcd_mask + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        one_xcd = one_xcd && (mask & (mask - 1)) == 0;
      }
    }
    if (tid == 0) same_l2 = one_xcd && sa.same_l2_allowed;
    __syncthreads();
  }

  const int n_mine = MULTI ? (n_chains - grp + groups - 1) / groups : 1;
  for (int step = 0; step < sa.n_steps; ++step) {
  if (PIPE && (step & 1) != part) continue;            // the partner's step
  for (int ci = 0; ci < n_mine; ++ci) {
  const int ch = grp + ci * groups;
  // ---- the step reads what every slot tile of this chain wrote in the step before
  if (!PIPE && step > 0 && !chain_wait(ch, step)) return;
  // PIPE: the chain is met between the two legs of the walk
  const bool meet_between = PIPE && step > 0;
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
    if (LOG == 1)
      log_rows = __builtin_amdgcn_make_buffer_rsrc((void*)(sa.logits + step * sa.logits_stride + ((int64_t)ch * a.M + i0) * sa.logits_ld), 0,
                                                   BM * sa.logits_ld * 4, 0x00020000);
    const int64_t prev = (int64_t)((sa.slot0 + step - 1) % sa.ring) * sa.out_stride;   // (unused for step 0)
    const uint16_t* src_k = step == 0 ? (const uint16_t*)a.cache_k : (const uint16_t*)sa.out_k + prev;
    const uint16_t* src_v = step == 0 ? (const uint16_t*)a.cache_v : (const uint16_t*)sa.out_v + prev;
    cat_k = make_cat(src_k + (int64_t)ch * a.M * kD, m,
                     (const uint16_t*)a.k.p + b * a.k.sb + hkv * a.k.sh + tok * a.k.st, a.k.st, Bn);
    cat_v = make_cat(src_v + (int64_t)ch * a.M * kD, m,
                     (const uint16_t*)a.v.p + b * a.v.sb + hkv * a.v.sh + tok * a.v.st, a.v.st, Bn);
  }
  // ---- prologue of a walk: key tiles 0, 1 and 2 staged; key tile 3 and value tile 0 on their way.  All
  // loads are issued before the first store (the accumulators' registers are free here), so the
  // walk starts after one memory latency, not three.
  auto prologue = [&]() {
    const int jb = SPLIT ? jbase : 0;
    Cat16 xpro[3][G::XPER];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) {
        const int item = tid + it * kThreads;
        xpro[t][it] = load_cat16(cat_k, jb + t * BN - G::PAD + (item >> 4), item & 15);
      }
#pragma unroll
    for (int it = 0; it < G::XPER; ++it) load_x(it, jb + 3 * BN);
#pragma unroll
    for (int it = 0; it < G::VPER; ++it) load_v(it, jb);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int it = 0; it < G::XPER; ++it) {
        const int item = tid + it * kThreads;
        *(u32x4*)(Xs0 + t * G::XBYTES + (item >> 4) * G::XSTRIDE + (item & 15) * 16) =
            xpro[t][it].from_cache | xpro[t][it].from_blk;
      }
    __syncthreads();
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  constexpr std::integral_constant<int, -1> dyn{};
  // The steady stages with the phase of the buffer rings known at compile time: one copy of the stage per
  // residue of the tile index modulo 2 * NXBUF, chained, so that the ring addresses are constants (about 30
  // scalar and 14 vector instructions per stage otherwise).  Ten copies of a stage still fit the instruction
  // cache.  Built where the register allocation takes it without spilling (32-slot tiles, width 15, filters over
  // the keys; measured: 3 % on the smaller and 9 % on the larger of the shapes that run on pairs of workgroups);
  // the 64-slot builds answered with spills inside the copies and ran 1.6 times as long (two copies, with only the
  // parity of the index a constant, did not spill and gained 0.7 %, but the launch then fetched 18 % more from
  // HBM), so they and every other build keep the one copy.
  constexpr bool RINGU = BM == 32 && KW == 15 && SPLIT != 1 && !(PROT && SPLIT == 2);
  auto steady_unrolled = [&]() {
    int i = 1;
    auto one = [&](auto r_t) {
      if (!(i + 1 < NT)) return false;
      stage(i, yes, yes, yes, r_t);
      ++i;
      return true;
    };
    for (;;) {
      if (!one(std::integral_constant<int, 1>{})) break;
      if (!one(std::integral_constant<int, 2>{})) break;
      if (!one(std::integral_constant<int, 3>{})) break;
      if (!one(std::integral_constant<int, 4>{})) break;
      if (!one(std::integral_constant<int, 5>{})) break;
      if (!one(std::integral_constant<int, 6>{})) break;
      if (!one(std::integral_constant<int, 7>{})) break;
      if (!one(std::integral_constant<int, 8>{})) break;
      if (!one(std::integral_constant<int, 9>{})) break;
      if (!one(std::integral_constant<int, 0>{})) break;
    }
  };
  static_assert(G::NXBUF == 5 && G::NVBUF == 2, "the unrolled steady stages assume a ring period of ten");
  if constexpr (PIPE) {
  // ---- a step in two legs: the same sequence of stages as the one-walk form below, as functions of the
  // leg's range.  The two forms are kept apart on purpose: the one-walk builds' register allocation is
  // tight (all 512 registers in use) and has answered to small changes of this code with spills inside the
  // stage loop, so they keep their code as it was.
  // the walk that mixes: pipeline fill, steady state, drain
  auto walk_main = [&]() {
    prologue();
    if constexpr (RINGU) {
      stage(-1, yes, no, no, std::integral_constant<int, 9>{});
      if (NT > 1) {
        stage(0, yes, yes, no, std::integral_constant<int, 0>{});
        steady_unrolled();
        stage(NT - 1, no, yes, yes, dyn);
      } else {
        stage(0, no, yes, no, std::integral_constant<int, 0>{});
      }
      stage(NT, no, no, yes, dyn);
      return;
    }
    stage(-1, yes, no, no, dyn);                          // logits of tile 0 only
    if (NT > 1) {
      stage(0, yes, yes, no, dyn);
      for (int i = 1; i + 1 < NT; ++i) stage(i, yes, yes, yes, dyn);
      stage(NT - 1, no, yes, yes, dyn);
    } else {
      stage(0, no, yes, no, dyn);
    }
    stage(NT, no, no, yes, dyn);
  };
  auto zero_state = [&]() {
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[ct][rt][i] = 0.f;
    m_run = -INFINITY;
    l_run = 0.f;
  };
  // PIPE: the range of a leg of the walk; the chain is met before the leg that touches the cache
  auto set_leg = [&](int leg) -> bool {
    if (leg == 0) {
      jbase = first_blk * BN;
      NT = NT_all - first_blk;
    } else {
      if (meet_between && !chain_wait(ch, step)) return false;
      jbase = 0;
      NT = first_blk;
    }
    return true;
  };
  zero_state();
  for (int leg = 0; leg < 2; ++leg) {
    if (!set_leg(leg)) return;
    if (NT > 0) walk_main();
    if (leg == 0) __syncthreads();
  }

  } else {
  if (!SPLIT || NT > 0) {
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[ct][rt][i] = 0.f;
  m_run = -INFINITY;
  l_run = 0.f;
  prologue();
  if constexpr (RINGU) {
  stage(-1, yes, no, no, std::integral_constant<int, 9>{});
  if (NT > 1) {
    stage(0, yes, yes, no, std::integral_constant<int, 0>{});
    steady_unrolled();
    stage(NT - 1, no, yes, yes, dyn);
  } else {
    stage(0, no, yes, no, std::integral_constant<int, 0>{});
  }
  stage(NT, no, no, yes, dyn);
  } else {
  stage(-1, yes, no, no, dyn);                          // logits of tile 0 only

  // ---- pipeline fill, steady state, drain
  if (NT > 1) {
    stage(0, yes, yes, no, dyn);
    for (int i = 1; i + 1 < NT; ++i) stage(i, yes, yes, yes, dyn);
    stage(NT - 1, no, yes, yes, dyn);
  } else {
    stage(0, no, yes, no, dyn);
  }
  stage(NT, no, no, yes, dyn);
  }
  } else {                                 // a part without positions hands in an empty result
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int rt = 0; rt < G::RT; ++rt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[ct][rt][i] = 0.f;
    m_run = -INFINITY;
    l_run = 0.f;
  }

  }   // one walk per step

  uint16_t* nk;
  uint16_t* nv;
  {
    const int64_t out_at = (int64_t)((sa.slot0 + step) % sa.ring) * sa.out_stride + ((int64_t)ch * a.M + i0) * kD;
    nk = (uint16_t*)sa.out_k + out_at;
    nv = (uint16_t*)sa.out_v + out_at;
    if constexpr (LOG == 2 || last_to_caller(BM, KW, MULTI)) {
      if (step > 0 && step + 1 == sa.n_steps && sa.last_k) {   // (a single step looks no further)
        nk = (uint16_t*)sa.last_k + ((int64_t)ch * a.M + i0) * kD;
        nv = (uint16_t*)sa.last_v + ((int64_t)ch * a.M + i0) * kD;
      }
    }
  }
  if constexpr (PSPLIT) {
    // ---- this part's result goes to the workspace: accumulators [slot][2 d] as they are
    // (unnormalised, relative to this part's reference), then the references, then the row sums
    float* mine = sa.partials + ((int64_t)(ch * tiles + i0 / BM) * P + part) * G::PART_FLOATS;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = {oacc[ct][0][g * 4 + 0], oacc[ct][0][g * 4 + 1], oacc[ct][0][g * 4 + 2], oacc[ct][0][g * 4 + 3]};
        *(f32x4*)(mine + l31 * (2 * kD) + 64 * w + ct * 32 + g * 8 + lh * 4) = v;
      }
    if ((l % G::LPR) == 0) {
      mine[BM * 2 * kD + srow] = m_run;
      mine[BM * 2 * kD + BM + srow] = l_run;
    }
    // ---- hand-off.  The parts of a (chain, tile) count themselves in; the one that completes the
    // count merges.  Two forms, as for the meeting of a chain: when all parts run on one XCD they
    // share its L2, so a part's stores have arrived once its store counter is at zero and the merging
    // part reads them at device scope (from the L2); otherwise device-scope release / acquire.  Which
    // form applies is read from the census word of the (chain, tile), where every part registered
    // its XCD when the kernel started: P registrations, all in this workgroup's field.  (A part that
    // looks before everybody has registered takes the general form, which is always safe.)
    __shared__ int i_merge;
    __shared__ int split_fast;
    uint32_t* cnt = sa.psync + 2 * (ch * tiles + i0 / BM);
    if (tid == 0) {
      const uint32_t xcd = __builtin_amdgcn_s_getreg(20 | ((4 - 1) << 11)) & 7u;   // XCC_ID
      split_fast = sa.same_l2_allowed &&
                   __hip_atomic_load(cnt + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ((uint32_t)P << (3u * xcd));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const bool fast = split_fast != 0;
    if (tid == 0) {
      const uint32_t old = fast ? __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                : __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      i_merge = (old + 1u) % (uint32_t)P == 0u;
    }
    __syncthreads();
    if (!i_merge) continue;              // the merging part signals the chain; this one goes on to the next step
    // ---- merge: reference = the largest of the parts' references; every part's sums and
    // accumulators are scaled to it and added in the order of the parts.  All loads are issued
    // before the first is used: one trip to the L2 for the lot.
    float* scale_s = Sred;               // [part][slot]
    float* inv_s = Sred + 4 * BM;        // 1 / row sum
    const __amdgpu_buffer_rsrc_t parts = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(sa.partials + (int64_t)(ch * tiles + i0 / BM) * P * G::PART_FLOATS), 0, P * G::PART_FLOATS * 4, 0x00020000);
    constexpr int kIters = BM * (2 * kD / 4) / kThreads;      // (slot, four columns of [K | V]) chunks per thread
    u32x4 raw[kIters][4];
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const int e = tid + it * kThreads, slot = e / (2 * kD / 4), c4 = e % (2 * kD / 4);
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P)
          raw[it][p] = __builtin_amdgcn_raw_buffer_load_b128(parts, (p * G::PART_FLOATS + slot * (2 * kD) + c4 * 4) * 4, 0, kDeviceScope);
    }
    if (tid < BM) {
      float mp[4], lp[4], mstar = -INFINITY;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P) {
          mp[p] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(parts, (p * G::PART_FLOATS + BM * 2 * kD + tid) * 4, 0, kDeviceScope));
          lp[p] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(parts, (p * G::PART_FLOATS + BM * 2 * kD + BM + tid) * 4, 0, kDeviceScope));
        }
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P) mstar = fmaxf(mstar, mp[p]);
      float lsum_all = 0.f;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (p < P) {
          const float sc = (NORM == 0) ? (mp[p] == -INFINITY ? 0.f : __expf(mp[p] - mstar)) : 1.0f;
          scale_s[p * BM + tid] = sc;
          lsum_all += sc * lp[p];
        }
      inv_s[tid] = 1.0f / (NORM == 0 ? lsum_all : lsum_all + a.eps);
    }
    __syncthreads();
    uint32_t keep = 0;                     // live protected slots keep their old rows (BM = 32: one mask word)
    if (PROT && i0 < m) {
      keep = pwords[i0 >> 5];
      if (i0 + 32 > m) keep &= (1u << (m - i0)) - 1u;
    }
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const int e = tid + it * kThreads, slot = e / (2 * kD / 4), c4 = e % (2 * kD / 4);
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
      for (int it = 0; it < 2 * BM * 16 / kThreads; ++it) {
        const int e = tid + it * kThreads;
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
  if ((l % G::LPR) == 0) lsum[srow] = l_run;
  __syncthreads();
  unsigned char* Orows = Xs0;                // [K rows of the tile ; V rows of the tile][XSTRIDE]
  static_assert(2 * BM * G::XSTRIDE <= G::NXBUF * G::XBYTES, "the output rows fit the key-tile area");
  uint32_t keep[G::RT];
#pragma unroll
  for (int rt = 0; rt < G::RT; ++rt) {
    // a live protected slot keeps its old row (copied below) instead of Eq. 4a / 4b
    keep[rt] = 0;
    if (PROT && i0 + rt * 32 < m) {
      keep[rt] = pwords[(i0 >> 5) + rt];
      if (i0 + rt * 32 + 32 > m) keep[rt] &= (1u << (m - i0 - rt * 32)) - 1u;
    }
    const int slot = rt * 32 + l31;
    const float inv = 1.0f / (NORM == 0 ? lsum[slot] : lsum[slot] + a.eps);
    unsigned char* orow = Orows + ((w >> 1) * BM + slot) * G::XSTRIDE + (64 * (w & 1)) * 2;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        u32x2 pk;
        pk[0] = pack_bf16(oacc[ct][rt][g * 4 + 0] * inv, oacc[ct][rt][g * 4 + 1] * inv);
        pk[1] = pack_bf16(oacc[ct][rt][g * 4 + 2] * inv, oacc[ct][rt][g * 4 + 3] * inv);
        *(u32x2*)(orow + (ct * 32 + g * 8 + lh * 4) * 2) = pk;
      }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 2 * BM * 16 / kThreads; ++it) {      // (K or V, slot, 16-byte chunk)
    const int e = tid + it * kThreads;
    const int kv = e / (BM * 16), r = (e >> 4) % BM, c16 = e & 15;
    uint16_t* dst = (kv ? nv : nk) + (int64_t)r * kD + c16 * 8;
    if (PROT && ((keep[r >> 5] >> (r & 31)) & 1u)) {         // live protected slot: inside the cache resources
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
  }  // steps
