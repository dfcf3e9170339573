// fp32 products on bf16 matrix instructions: a number is the sum of three bf16 numbers (each the rounding of what the ones before
// left: 24 bits), a product of two numbers six products of pieces; those left out are below 2^-24 of it.  Six
// v_mfma_f32_16x16x32_bf16 take 96 cycles where eight v_mfma_f32_16x16x4_f32 take 256.  The pieces' products are exact and 32 of
// them are summed at once, so a sum over K numbers is nearer to 64 bits than the chain of fp32 instructions: error of K = 128 /
// 1024 / 16384 random products 0.7 / 0.8 / 0.9 of it, of positive ones 0.5 / 0.5 / 0.6.  A number that is not finite gives NaN;
// below 2^-109 the last pieces leave the exponent range.
#pragma once
#include "fs_common.h"

namespace fs {

typedef __attribute__((ext_vector_type(8))) float f32x8_t;

struct Split3 { bf16x8 h, m, l; };

__device__ __forceinline__ Split3 split3(f32x4 a, f32x4 b) {
  const f32x8_t x = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  Split3 s;
  s.h = __builtin_convertvector(x, bf16x8);
  const f32x8_t r = x - __builtin_convertvector(s.h, f32x8_t);
  s.m = __builtin_convertvector(r, bf16x8);
  s.l = __builtin_convertvector(r - __builtin_convertvector(s.m, f32x8_t), bf16x8);
  return s;
}

__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// c + a b, small products first.
__device__ __forceinline__ f32x4 mfma3(const Split3& a, const Split3& b, f32x4 c) {
  c = mfma_bf16(a.l, b.h, c);
  c = mfma_bf16(a.h, b.l, c);
  c = mfma_bf16(a.m, b.m, c);
  c = mfma_bf16(a.m, b.h, c);
  c = mfma_bf16(a.h, b.m, c);
  return mfma_bf16(a.h, b.h, c);
}

// The same for the transposed product: the pieces in the order of mfma3(b, a, .), so that both round alike.
__device__ __forceinline__ f32x4 mfma3_t(const Split3& a, const Split3& b, f32x4 c) {
  c = mfma_bf16(a.h, b.l, c);
  c = mfma_bf16(a.l, b.h, c);
  c = mfma_bf16(a.m, b.m, c);
  c = mfma_bf16(a.h, b.m, c);
  c = mfma_bf16(a.m, b.h, c);
  return mfma_bf16(a.h, b.h, c);
}

// Piece p (0, 1, 2) of a number, for operand images written number by number.
__device__ __forceinline__ void split3_store(uint16_t* at, size_t piece_stride, float v) {
  const uint16_t h = f32_to_bf16_bits(v);
  const float r = v - bf16_bits_to_f32(h);
  const uint16_t m = f32_to_bf16_bits(r);
  at[0] = h;
  at[piece_stride] = m;
  at[2 * piece_stride] = f32_to_bf16_bits(r - bf16_bits_to_f32(m));
}

}  // namespace fs
