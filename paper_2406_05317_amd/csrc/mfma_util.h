// Device helpers shared by the backward kernels on the matrix cores: vector types, splitting fp32 values into two
// bf16 halves, buffer resources, loads that write LDS directly, swizzled tiles and their two kinds of operand read.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lococo {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_any;      // the caller's gradients: any float address
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ f32x16 zero16() {
  return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// two fp32 values -> their bf16 roundings (packed) and the bf16 roundings of what those left over: about 16 bits of
// the values kept
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  const f32x2 v = {x0, x1};
  hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  const f32x2 e = {x0 - __uint_as_float(hi << 16), x1 - __uint_as_float(hi & 0xffff0000u)};
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(e, bf16x2));
}
// PARTS = 2: the same for eight values, as operands.  PARTS = 3: what those two leave over as well, 24 bits in all: nothing is lost.
template <int PARTS>
__device__ __forceinline__ void split_parts(const float* x, bf16x8 (&part)[PARTS]) {
  float r[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = x[i];
#pragma unroll
  for (int p = 0; p < PARTS; ++p) {
    u32x4 h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x2 v = {r[2 * i], r[2 * i + 1]};
      h[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
      r[2 * i] -= __uint_as_float(h[i] << 16);
      r[2 * i + 1] -= __uint_as_float(h[i] & 0xffff0000u);
    }
    part[p] = __builtin_bit_cast(bf16x8, h);
  }
}
// a value combined with the one the lane 32 away holds (v_permlane32_swap: no trip through the LDS crossbar)
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// raw buffer resource over `bytes` bytes: what lies beyond reads as zero and is not touched
__device__ __forceinline__ u32x4 make_rsrc(const void* p, uint32_t bytes) {
  const uint64_t base = (uint64_t)p;
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
  r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
  r[2] = __builtin_amdgcn_readfirstlane(bytes);
  r[3] = 0x00020000u;
  return r;
}
// 64 lanes x 16 bytes straight into the 1 KB of LDS at lds_addr (lane l writes cell l).  Counted by vmcnt; the
// compiler does not know that LDS is written: the wait and the barrier that publish the data are written by hand.
// (M0, the LDS address, is an operand the compiler sets; the s_nop is the wait state such a load wants behind it.)
__device__ __forceinline__ void load_to_lds(const u32x4& rsrc, uint32_t lds_addr, uint32_t voff) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "{m0}"(lds_addr), "v"(voff), "s"(rsrc) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() {     // at most N of the newest loads still on their way
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// Transposing LDS read: within each group of 16 lanes, lane s supplies the address of 4 consecutive 16-bit elements
// and lane i receives element i % 4 of the chunks addressed by lanes i / 4 + {0, 4, 8, 12}; with lane s pointing at
// (row s / 4, column 4 (s % 4)) of a 4 x 16 patch every lane gets one column of the patch, 4 rows deep.
__device__ __forceinline__ bf16x8 frag_tr(const unsigned char* p0, const unsigned char* p1) {
  const s16x4 a0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p0);
  const s16x4 a1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p1);
  const s16x8 v = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// Tiles of 128-element bf16 rows in LDS, unpadded (256 bytes a row), 16-byte chunk c of row r in cell c ^ swz(r).
// swz runs through all 16 values over 16 rows, and through 4 times 0..3 (xor a constant) over four rows: both kinds of
// operand read, 16 bytes of 16 rows and the transposing 64 bytes of 4 rows, fall on 64 different banks.
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// Addresses of the operand reads inside such a tile (row and column offsets that are multiples of 16 rows are plain
// byte offsets on top).
struct TileAddr {
  int row[8];          // 16-byte reads: lane (row l % 32), k step ks: columns 16 ks + 8 (l / 32) ..
  int tr[4][2];        // transposing reads, column block ct of 32: rows 4 (l / 32) .. + 3, and 8 rows on
};
__device__ __forceinline__ void tile_addr(int l, TileAddr& t) {
  const int l31 = l & 31, lh = l >> 5, s16 = l & 15, g2 = (l >> 4) & 1;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) t.row[ks] = l31 * 256 + (((2 * ks + lh) ^ swz(l31)) << 4);
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = lh * 4 + (s16 >> 2) + 8 * h, chunk = 4 * ct + 2 * g2 + ((s16 & 3) >> 1);
      t.tr[ct][h] = r * 256 + ((chunk ^ swz(r)) << 4) + (s16 & 1) * 8;
    }
}

// work items renumbered so that consecutive ones run on one XCD (workgroup ids are dealt round-robin to the eight)
__device__ __forceinline__ int xcd_item(int id, int total) {
  const int per = total / 8;
  return id < per * 8 ? (id % 8) * per + id / 8 : id;
}

}  // namespace lococo
