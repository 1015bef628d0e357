// Shared device helpers for the tiled contrastive-loss kernels (gfx950 only).
//
// Conventions used by both sweeps
//   - Matrix products run on the 32x32x16 bf16 or fp16 MFMA (fp32 accumulate),
//     those of fp32 inputs as six products of bf16 parts (split3).  Fragments of both 16-bit types are carried
//     in bf16x8 registers; only the MFMA opcode and the conversions differ.  For a 32x32 output block, lane L holds column
//     n = L % 32 and rows m = 8*(r/4) + 4*(L/32) + r%4 for accumulator r = 0..15.
//     Operand fragments: lane L holds row L % 32 and the 8 consecutive
//     contraction slots 8*(L/32) .. 8*(L/32)+7 of a 16-wide contraction step.
//   - Log-sum-exp statistics are kept in base 2: y = s*log2(e)*<a, b>, a
//     running pair (R, l) stands for log2(l) + R, and exp2 maps to v_exp_f32.
//   - Tiles are staged in LDS in 16-byte chunks with an XOR swizzle of the chunk
//     index so that both the row-fragment reads and the transposing reads of
//     the backward pass are bank-conflict free.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace infcl {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

#define INFCL_LDS __attribute__((address_space(3)))
#define INFCL_GLOBAL __attribute__((address_space(1)))

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// A per-tile partial sum above this bound, or a non-finite one, sends a tile
// through the exact (max-rescaled) path.  With at most 2^22 terms per sum the
// accumulated value stays below 2^86, far from float overflow.
constexpr float kLazyBound = 18446744073709551616.0f;  // 2^64

__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ f32x16 mfma_bf16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// 16-bit MFMA on fragments held as bf16x8: bf16 operands, or fp16 (F16).
template <bool F16>
__device__ __forceinline__ f32x16 mfma16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                  0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// float -> 16-bit element, round to nearest even (bf16, or the bits of fp16)
template <bool F16>
__device__ __forceinline__ __bf16 to16(float x) {
  if constexpr (F16)
    return __builtin_bit_cast(__bf16, (_Float16)x);
  else
    return (__bf16)x;
}
// 16-bit element (bf16, or fp16 bits) -> float, exact
template <bool F16>
__device__ __forceinline__ float from16(__bf16 x) {
  if constexpr (F16)
    return (float)__builtin_bit_cast(_Float16, x);
  else
    return (float)x;
}
// An fp32 operand fragment as three bf16 fragments, x = p0 + p1 + p2: each
// part is the remainder so far rounded to nearest, and the remainders are exact,
// so the parts carry x's 24 bits (8 + 8 + 8, with the signs).  The parts of
// magnitudes below 2^-110 are subnormal; the conversion and the MFMA keep those,
// down to 2^-133, so that such an x is right to within 2^-134.  A product of two
// operands is six bf16 MFMAs (mfma_split): of the three products left out,
// p1 q2 and p2 q1 reach 2^-25 of the full one each, all three 2^-24 (over random
// mantissas 2^-27.5 in the root mean square, 2^-26.5 next to 1), as much as
// fp32's own rounding of it; every bf16 product is exact in the fp32
// accumulator.  Six 32x32x16 bf16 MFMAs take 192 cycles where eight 32x32x2 fp32
// ones take 512.
struct split3 {
  bf16x8 p[3];
};
// two floats to packed bf16 (one v_cvt_pk_bf16_f32), round to nearest even
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// At the start of a kernel that splits its inputs: conversions to 16-bit types
// limit finite values to the largest one instead of rounding them to infinity
// (MODE.FP16_OVFL; it covers bf16 too).  Entries from 2^128 - 2^119 on would
// otherwise have an infinite first part and NaN for the others; this way the
// remainders stay exact.  Limiting the values by two instructions per pair
// cost 3 to 5% (forward b = 8192, d = 256 235 -> 247 us).  An infinite entry
// still has an infinite first part and NaN products.
__device__ __forceinline__ void split_limit_parts() {
  __builtin_amdgcn_s_setreg(0 << 11 | 23 << 6 | 1, 1);  // one bit at 23 of HW_REG_MODE
}
// one pair of values into element pair e of the three parts; eleven instructions
__device__ __forceinline__ void split_pair(float u, float v, int e, u32x4 (&p)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t q = pk_bf16(u, v);
    p[k][e] = q;
    u -= __uint_as_float(q << 16);
    v -= __uint_as_float(q & 0xFFFF0000u);
  }
}
__device__ __forceinline__ split3 split_f32(const float (&x)[8]) {
  u32x4 p[3];
#pragma unroll
  for (int e = 0; e < 4; ++e) split_pair(x[2 * e], x[2 * e + 1], e, p);
  split3 s;
#pragma unroll
  for (int k = 0; k < 3; ++k) s.p[k] = __builtin_bit_cast(bf16x8, p[k]);
  return s;
}
__device__ __forceinline__ split3 split_f32(f32x4 lo, f32x4 hi) {
  const float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return split_f32(x);
}
// c0 + c1 += a b, in two independent accumulation chains
__device__ __forceinline__ void mfma_split(const split3& a, const split3& b, f32x16& c0, f32x16& c1) {
  c0 = mfma_bf16(a.p[2], b.p[0], c0);
  c1 = mfma_bf16(a.p[0], b.p[2], c1);
  c0 = mfma_bf16(a.p[1], b.p[1], c0);
  c1 = mfma_bf16(a.p[1], b.p[0], c1);
  c0 = mfma_bf16(a.p[0], b.p[1], c0);
  c1 = mfma_bf16(a.p[0], b.p[0], c1);
}

__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Asynchronous 16-byte buffer -> LDS copies, issued from inline assembly with a
// raw descriptor over [base, base + nbytes) (rsrc_words; loads past the end
// return 0; rebased per tile so that 32-bit per-lane offsets address inputs of
// any size).  Lane L writes LDS bytes [lds_base + 16 L, +16).  The compiler does
// not see this as a write to LDS, so it never stalls later LDS reads on it: the
// caller waits for completion explicitly (wait_dma) before the written buffer is
// read.  m0 holds the wave-uniform LDS base.  The compiler's hazard checks do not look inside
// inline assembly, and it may restore an operand right before it (an SGPR of
// the descriptor with v_readlane, the offset with v_accvgpr_read): the five
// wait states cover a VALU-written SGPR read by a vector memory instruction,
// which is the longest of those requirements (and the one of m0).
__device__ __forceinline__ u32x4 rsrc_words(const void* base, int64_t nbytes) {
  const int64_t n = nbytes < 0 ? 0 : (nbytes > 0xFFFFFFF0ll ? 0xFFFFFFF0ll : nbytes);
  const uint64_t a = (uint64_t)base;
  u32x4 r;
  r[0] = (uint32_t)a;
  r[1] = (uint32_t)(a >> 32) & 0xFFFFu;  // stride 0
  r[2] = (uint32_t)n;                    // num_records (bytes)
  r[3] = 0x00020000u;
  return r;
}
__device__ __forceinline__ void dma16_asm(const u32x4& rs, const INFCL_LDS void* lds_base, uint32_t voff) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds_base);
  asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voff), "s"(rs), "{m0}"(m0v));
}
// ... with a wave-uniform byte offset soff added to every lane's offset.
__device__ __forceinline__ void dma16_asm(const u32x4& rs, const INFCL_LDS void* lds_base, uint32_t voff,
                                          uint32_t soff) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds_base);
  const uint32_t so = __builtin_amdgcn_readfirstlane(soff);
  asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rs), "s"(so), "{m0}"(m0v));
}

// The same with one wait state only (m0 written by a scalar instruction just
// before), for bursts whose other operands are set up well ahead; the build's
// wait-state check verifies every use.
__device__ __forceinline__ void dma16_asm_w1(const u32x4& rs, const INFCL_LDS void* lds_base, uint32_t voff) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds_base);
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voff), "s"(rs), "{m0}"(m0v));
}
__device__ __forceinline__ void dma16_asm_w1(const u32x4& rs, const INFCL_LDS void* lds_base, uint32_t voff,
                                             uint32_t soff) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds_base);
  const uint32_t so = __builtin_amdgcn_readfirstlane(soff);
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rs), "s"(so), "{m0}"(m0v));
}

// Merge of two base-2 log-sum-exp pairs (R, l) -> (max R, rescaled sum).
__device__ __forceinline__ void lse2_merge(float& R, float& l, float R2, float l2) {
  float M = fmaxf(R, R2);
  if (M == -__builtin_inff()) return;  // both empty
  l = l * exp2_hw(R - M) + l2 * exp2_hw(R2 - M);
  R = M;
}

__device__ __forceinline__ bool lazy_ok(float t) { return t <= kLazyBound; }  // false for NaN/inf

// Cross-lane helpers (full 64-lane wave).
__device__ __forceinline__ float shfl_xor(float v, int mask) {
  int l = __lane_id();
  return __int_as_float(__builtin_amdgcn_ds_bpermute((l ^ mask) << 2, __float_as_int(v)));
}
__device__ __forceinline__ float shfl_idx(float v, int src) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src << 2, __float_as_int(v)));
}
__device__ __forceinline__ bool wave_any(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

}  // namespace infcl
