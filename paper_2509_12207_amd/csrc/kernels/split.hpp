// FP32 products on the BF16 matrix cores of gfx950, with FP32 accuracy (the
// three-way bfloat16 split of Henry, Tang and Heinecke, 2019).
//
// An FP32 value is exactly the sum of three bfloat16 values: h is x rounded
// to nearest, m is x - h rounded to nearest, l is the rest (24 = 3 x 8
// significant bits; both differences are exact).  Of the nine products of two
// split values the six of relative size 2^-16 and more are formed:
//   hh | mh hm | lh hl mm
// and hm, mh, lh, hl, mm are accumulated apart from hh.  What is left out (lm,
// ml, ll) is below 2^-25 of the product, with no sign of its own.  BF16 x BF16
// is exact in FP32; the matrix instruction rounds its FP32 accumulator once
// per 16 products, where the FP32 instruction rounds once per product, so the
// sum is closer to the exact one: against fp64 the error (rms) of a K-long
// product is 0.28-0.40 of the FP32 instruction's for uniform and normal values
// and K = 32 to 4096, and 0.36-0.48 where all products are positive; from
// three terms on it is smaller (kSplitMinTerms).  A sum with one term that is
// not zero errs by up to 1.63 x 2^-24 of it, where the FP32 instruction rounds
// it correctly (the split too, if a factor has at most eight significant bits:
// a permutation's one).
//
// Rate: six v_mfma_f32_32x32x16_bf16 (32 cycles each) take the place of eight
// v_mfma_f32_32x32x2_f32 (64 cycles each): 2.67 times fewer matrix cycles.
// The split costs six and a half vector instructions per staged element, paid
// once per element and workgroup tile.
//
// Values are multiplied by 2^16 as they are split and the sums by 2^-32 at the
// end: a multiple of 2^-149 becomes one of 2^-133, the last bit of a subnormal
// bfloat16, so that the three pieces hold every FP32 value, subnormal ones
// too (the matrix instruction takes subnormal operands as they are).  Without
// the factor values below 2^-109 had none, and a tile that held one, as every
// tile of a softmax output with a spread of 75 in its logits does, was
// computed twice.
//
// What has no split is noticed by a result that is not finite: operands that
// are infinite, NaN or 2^112 and more, and sums of 2^96 and more.  The
// workgroup then computes its tile again with the FP32 instruction.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "mfma.hpp"

namespace ug {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16 mfma_bf16(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {   // nearest even
  const f32x2_t v = {x, y};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// Sums of fewer products are left to the FP32 instruction: what the split
// leaves out is more than the roundings it saves (error in 2^-24 of the sum of
// |products|, largest / rms, FP32 against split, normal values: one product
// 1.00 / 0.425 against 1.63 / 0.435, two 1.87 / 0.429 against 2.43 / 0.368,
// three 2.21 / 0.438 against 2.07 / 0.325).
constexpr int kSplitMinTerms = 3;

constexpr float kSplitScale = 0x1p16f;      // of the values split
constexpr float kSplitUnscale = 0x1p-32f;   // of their products

// Splits a pair.
__device__ __forceinline__ void split2(float x, float y, uint32_t* h, uint32_t* m, uint32_t* l) {
  x *= kSplitScale;
  y *= kSplitScale;
  *h = pack_bf16(x, y);
  const float rx = x - __uint_as_float(*h << 16);
  const float ry = y - __uint_as_float(*h & 0xffff0000u);
  *m = pack_bf16(rx, ry);
  const uint32_t lx = __float_as_uint(rx - __uint_as_float(*m << 16));
  const uint32_t ly = __float_as_uint(ry - __uint_as_float(*m & 0xffff0000u));
  *l = __builtin_amdgcn_perm(ly, lx, 0x07060302u);
}

__device__ __forceinline__ bool finite16(f32x16 v) {
  bool ok = true;
#pragma unroll
  for (int r = 0; r < 16; ++r) ok = ok && (__float_as_uint(v[r]) & 0x7f800000u) != 0x7f800000u;
  return ok;
}

// Meets the workgroup once this wavefront's LDS accesses are done.  Unlike
// __syncthreads it leaves global loads in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

}  // namespace ug
