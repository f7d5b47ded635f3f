// Fused compression kernel for gfx950: Eq. 5 (convolution logits), Eq. 6
// (softmax over positions) and Eq. 4a/4b (fusion of K and V with shared
// weights) in one pass, bf16 MFMA with fp32 accumulation.  The logits and the
// normalised weights never leave the compute unit.
//
// Two kernels do this work: the one described next (compress_tile.inl), whose four waves all do the same, and one whose eight
// waves have two roles (compress_roles.h), for filters over [K | V] and for single steps on the builds with two workgroups per
// pair.  This file has what they share: the method, the layouts in LDS, the resources.
//
// Structure.  The step is "attention with a convolution for scores": for a
// tile of BM cache slots the kernel walks the T = m + B positions of
// [cache ; block] in tiles of 32, computes the logits as an implicit GEMM
// with inner dimension C*k (each filter tap is a row-shifted view of the key
// tile held in LDS), keeps a running reference / row sum per slot (online
// softmax), and accumulates [K | V]^T P^T into a 2d x BM fp32 accumulator.
//
// Register-stationary filters.  The filter bank is the same for every
// position, chain and step, and a compute unit's register file (512 KB) is
// larger than its slice of the bank, so each workgroup loads its BM x (C*k)
// filter slice into registers once and streams only keys/values through LDS.
// The four waves split the inner dimension by channel quarter (wave w owns
// channels [32w, 32w+32) of every tap); their partial logits are summed
// through LDS before the softmax.  For the mixing GEMM wave w owns output
// columns [64w, 64w+64) of [K | V].
//
// Transposed tiles.  Both GEMMs are computed transposed (positions x slots,
// then columns x slots) so that an MFMA lane always belongs to one slot: the
// partial logits leave the registers as 16-byte stores, the rescale factor is
// a per-lane scalar and the new cache rows are stored 8 bytes at a time.
//
// Software pipeline.  One wave per SIMD leaves nothing to switch to while a
// wave waits, so the loop is pipelined by hand, three tiles deep: while the
// MFMAs of tile i+1's logits issue, the wave works through tile i's reduction
// and softmax, tile i-1's mixing MFMAs and the staging of later tiles, all cut
// into small slices pinned between the logit MFMAs (loads are issued a few
// steps before they are consumed).  The two workgroup barriers of a tile sit
// inside that MFMA stream as well, so no barrier is waited for with the matrix
// pipe idle.
//
// Filters over [K | V] (C = 2d, the compressor as Eq. 5 prints it).  A slot tile's slice of such a
// bank is twice what the registers hold, and the logit is a sum of a convolution over the keys
// and one over the values, so the walk is done twice: with the key half of the filters resident
// the kernel leaves the summed key-side logits of every position tile in the workspace (4 KB per
// tile, each lane writing the four values it will read back itself); then the value half takes the
// registers' place and the second walk runs with the value rows as the convolution's input,
// the stored key-side logits added where the logit waves' partial sums meet.  In that walk
// the two row tiles swap roles (values with halo, keys without), so the accumulator's first d
// columns are the new value rows and the pointers are swapped where the rows are written.
//
// Shapes taken: head_dim = 128, bf16, width 15 (64- or 32-slot tiles) or 21 (32-slot tiles) over the
// keys, or either width over [K | V] (32-slot tiles), either normalisation, M a multiple of BM;
// any T (tail positions are masked), any m.
#pragma once

#include <type_traits>

#include "lococo_internal.h"

namespace lococo {
namespace compress_detail {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

constexpr int kD = 128;            // head_dim = conv channels
constexpr int kThreads = 256;
constexpr int BN = 32;             // positions per tile

// Whether a build's last step always can write its state to the caller (ScanArgs::last_k) in place of its slot.  The choice costs
// registers in the epilogue of every step and saves a copy a call.  In the 32-slot, one-chain builds of width 15 it puts six vector
// registers (softmax, pairs) into scratch memory: 132 steps on 512 slots, 8 chains, 3147 us without it and 3193 with, 102 on 160, 32
// chains, 1452 and 1463, 126 on 128, 64 chains, 1815 and 1833.  In the others it is free or better: width 21, 65 on 352, 8 chains, 1452
// without and 1436 with; 64 slots a workgroup, 53 on 512, 32 chains, 2823 and 2795; several chains, 62 on 128, 1562 and 1553.
constexpr bool last_to_caller(int bm, int kw, bool multi) { return bm == 64 || kw != 15 || multi; }
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLazy = 8.0f;      // the softmax reference lags the row maximum by at most this much

template <int BM, int KW>
struct Geo {
  static constexpr int RT = BM / 32;                 // 32-slot MFMA tiles per workgroup
  static constexpr int NS = KW * 2;                  // contraction steps of a logit tile: (tap, channel half)
  static constexpr int PAD = (KW - 1) / 2;
  static constexpr int XROWS = BN + KW - 1;          // key tile rows incl. halo
  static constexpr int XSTRIDE = kD * 2 + 16;        // bytes per key-tile row (conflict-free 16-byte reads)
  static constexpr int VSTRIDE = kD * 2 + 64;        // bytes per value-tile row (conflict-free transposing reads)
  static constexpr int SSTRIDE = BN + 4;             // floats per slot row of a partial-logit buffer
  static constexpr int PSTRIDE = BN * 2 + 16;        // bytes per slot row of the bf16 probability tile
  static constexpr int XITEMS = XROWS * 16;          // 16-byte chunks of the key tile
  static constexpr int XPER = (XITEMS + kThreads - 1) / kThreads;
  static constexpr int XALLOC = XPER * kThreads / 16;  // rows allocated: every thread stores XPER chunks
  static constexpr int XBYTES = XALLOC * XSTRIDE;
  static constexpr int VPER = BN * 16 / kThreads;    // 16-byte chunks of the value tile per thread
  static constexpr int VBYTES = BN * VSTRIDE;
  static constexpr int SBYTES = 4 * BM * SSTRIDE * 4;
  static constexpr int PBYTES = BM * PSTRIDE;
  static constexpr int NXBUF = 5, NVBUF = 2;           // key tiles i-1 .. i+3, value tiles i-1, i
  static constexpr int LDS = NXBUF * XBYTES + NVBUF * VBYTES + SBYTES + 2 * PBYTES + 3 * BM * 4;
  static constexpr int RPW = BM / 4;                 // slots a wave owns in the softmax phase
  static constexpr int LPR = 64 / RPW;               // lanes per slot there
  static constexpr int EPL = BN / LPR;               // positions per lane there
  static_assert(BM == 32 || BM == 64, "BM");
  static constexpr int PART_FLOATS = BM * 2 * kD + 2 * BM;   // a part's accumulators [slot][2 d], references, row sums
  static_assert(EPL % 4 == 0, "softmax lanes read whole float4s");
  static_assert(NS >= 26, "the slices of the pipelined loop are laid out over 26 contraction steps");
  static_assert(LDS <= 160 * 1024, "LDS budget");
};

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {   // v_cvt_pk_bf16_f32, RNE
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Cross-lane exchange inside groups of 4 / 8 lanes on the VALU (DPP), no LDS round trip.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7 - i within 8 lanes
template <int LPR>
__device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, dpp<kDppXor1>(v));
  v = fmaxf(v, dpp<kDppXor2>(v));
  if (LPR == 8) v = fmaxf(v, dpp<kDppHalfMirror>(v));
  return v;
}
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp<kDppXor1>(v);
  v += dpp<kDppXor2>(v);
  if (LPR == 8) v += dpp<kDppHalfMirror>(v);
  return v;
}

// Transposing LDS read (ds_read_b64_tr_b16).  Within each group of 16 lanes, lane s supplies the
// address of 4 consecutive 16-bit elements; lane i of the group receives element (i % 4) of the
// chunks addressed by lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12.  With lane s pointing at
// (row r0 + s/4, column c0 + 4*(s%4)) of a row-major tile, lane i ends up with column c0 + i of
// rows r0 .. r0+3: an operand fragment (column, 4 contraction rows) straight from a row-major tile.
__device__ __forceinline__ s16x4 lds_read_tr(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p);
}

// [cache ; block] rows are read through two raw buffer resources, one over the live cache rows and
// one over the block rows.  A row index outside a resource's range (negative offsets wrap to huge
// unsigned ones) reads as zero without touching memory, so OR-ing the two loads yields row p of the
// concatenation for 0 <= p < T and zeros elsewhere: no clamps, no selects, no masks.
struct CatRows {
  __amdgpu_buffer_rsrc_t cache, blk;
  int m;            // rows in the cache part
  int blk_stride;   // bytes between block rows
};
__device__ __forceinline__ CatRows make_cat(const uint16_t* cache_rows, int m, const uint16_t* blk_rows,
                                            int64_t blk_st, int Bn) {
  CatRows c;
  c.cache = __builtin_amdgcn_make_buffer_rsrc((void*)cache_rows, 0, m * kD * 2, 0x00020000);
  c.blk = __builtin_amdgcn_make_buffer_rsrc((void*)blk_rows, 0, (int)((Bn - 1) * blk_st + kD) * 2,
                                            0x00020000);
  c.m = m;
  c.blk_stride = (int)blk_st * 2;
  return c;
}
// The two halves are OR-ed only when the data is stored to LDS, many steps after the loads were issued.
struct Cat16 { u32x4 from_cache, from_blk; };
// Cache rows are read at device scope (sc1: served by the L2, never by this CU's L1): in the
// one-launch scan they were written by other workgroups a step ago, and every row is read once per
// workgroup anyway.
constexpr int kDeviceScope = 1 << 4;
__device__ __forceinline__ Cat16 load_cat16(const CatRows& c, int p, int chunk) {
  Cat16 r;
  r.from_cache = __builtin_amdgcn_raw_buffer_load_b128(c.cache, p * (kD * 2) + chunk * 16, 0, kDeviceScope);
  r.from_blk = __builtin_amdgcn_raw_buffer_load_b128(c.blk, (p - c.m) * c.blk_stride + chunk * 16, 0, 0);
  return r;
}

// wp: filters repacked in register order, [bank][M/32][wave][tap][half][lane] x 8 channels: lane l of
// wave w holds slot (32-slot tile)*32 + l%32, channels 32w + 16*half + 8*(l/32) .. +7, so that every
// load instruction of the prologue reads 1 KB of contiguous memory.
// NORM = 0: softmax over the positions; NORM = 1: relu(W) / (sum of relu(W) + eps) (Eq. 6 as printed,
// with the rectifier of the convolution head in front of it).
// PROT = 1: the cache carries protected slots (lococo_cache.protect); a build of its own so that the
// common case pays neither the registers nor the instructions.
// MULTI = 1: a workgroup may own several chains (see below); also a build of its own, because the
// register allocation of the one-chain build is tight and the 32 K-token workload runs on it.
// SPLIT = 1: the positions of a step are shared out between sa.psplit workgroups per (chain, slot
// tile) -- for shapes whose (chain, tile) pairs would leave compute units idle.  Each part walks its
// range of position tiles with the same pipeline and leaves its running reference, row sum and
// unnormalised accumulators in the workspace; the part that arrives last merges them in a fixed
// order (so the result does not depend on who is last) and writes the rows.
// SPLIT = 2: two workgroups per (chain, slot tile) take the steps of a scan in turn.  A step of such a
// build is walked in two legs that share the running softmax and the accumulators (the order of the
// positions does not matter to either): first the tiles that lie wholly in the block, halo included --
// they do not depend on the step before, so the workgroup whose turn is next works through them while
// its partner finishes that step -- then, after the chain has been met, the tiles that touch the cache.
// Only the second leg is on the chain's critical path.  (Single-step launches walk the same two legs, one
// workgroup of each pair idle, so that results do not depend on the kind of launch.)
// LOG = 1 (compress_tile.inl): the logits of Eq. 5 also go to memory, step by step [chains, M, ld], for the backward pass of a
// scan (no protected slots, filters over the keys).
// LOG = 2: no logits, but the last step can write to the caller, where the build without cannot (see last_to_caller).
// CIN = 1 (compress_roles.h): filters over [K | V] (two walks, see the head of the file); wp then holds the key half of
// every bank's slices followed by the value half, each in the order above.

}  // namespace compress_detail
}  // namespace lococo
