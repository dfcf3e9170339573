// fp32 products on bf16 matrix instructions: a number is the sum of three bf16 numbers (each the rounding of what the ones before
// left: 24 bits), a product of two numbers six products of pieces; those left out are below 2^-24 of it.  Six
// v_mfma_f32_16x16x32_bf16 take 96 cycles where eight v_mfma_f32_16x16x4_f32 take 256.  The pieces' products are exact and 32 of
// them are summed at once, so a sum over K numbers is nearer to 64 bits than the chain of fp32 instructions: error of K = 128 /
// 1024 / 16384 random products 0.7 / 0.8 / 0.9 of it, of positive ones 0.5 / 0.5 / 0.6.  A number that is not finite gives NaN.  Below
// 2^-109 the last pieces leave the exponent range (subnormal pieces count: a number is then off by up to 2^-134): the kernels scale what
// they split so that nothing that matters is left there.
#pragma once
#include "fs_common.h"

namespace fs {

typedef __attribute__((ext_vector_type(8))) float f32x8_t;

struct Split3 { bf16x8 h, m, l; };

typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;

// x less its first piece, for two numbers: the dot product of their pieces with (-1, 0) or (0, -1), which is exact.  (Seven instructions
// for the pieces of two numbers where shifts and subtractions take eleven.  A number that is not finite makes its neighbour NaN:
// for numbers that are summed anyway.  The pairs are kept in registers: as an inline constant of the instruction the first one is
// read as the second.)
__device__ __forceinline__ f32x2_t less_piece(f32x2_t x, bf16x2_t h) {
  uint32_t low = 0xbf80u, high = 0xbf800000u;
  asm("" : "+s"(low));
  asm("" : "+s"(high));
  return f32x2_t{__builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2_t, low), x[0], false),
                 __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2_t, high), x[1], false)};
}
__device__ __forceinline__ Split3 split3(f32x4 a, f32x4 b) {
  const f32x2_t x[4] = {{a[0], a[1]}, {a[2], a[3]}, {b[0], b[1]}, {b[2], b[3]}};
  bf16x2_t h[4], m[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = __builtin_convertvector(x[i], bf16x2_t);
    const f32x2_t r = less_piece(x[i], h[i]);
    m[i] = __builtin_convertvector(r, bf16x2_t);
    l[i] = __builtin_convertvector(less_piece(r, m[i]), bf16x2_t);
  }
  auto join = [](const bf16x2_t (&v)[4]) {
    return __builtin_bit_cast(bf16x8, u32x4{__builtin_bit_cast(uint32_t, v[0]), __builtin_bit_cast(uint32_t, v[1]), __builtin_bit_cast(uint32_t, v[2]),
                                            __builtin_bit_cast(uint32_t, v[3])});
  };
  return {join(h), join(m), join(l)};
}
// The same number by number (numbers of different rows or columns of a result).
__device__ __forceinline__ Split3 split3_each(f32x4 a, f32x4 b) {
  const f32x8_t x = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  Split3 s;
  s.h = __builtin_convertvector(x, bf16x8);
  const f32x8_t r = x - __builtin_convertvector(s.h, f32x8_t);
  s.m = __builtin_convertvector(r, bf16x8);
  s.l = __builtin_convertvector(r - __builtin_convertvector(s.m, f32x8_t), bf16x8);
  return s;
}

// PART: which numbers of an operand are summed over, all eight of a lane or the four of its low or high half (the others need not be
// finite then).
enum { ALL = 0, LOW = 1, HIGH = 2 };
template <int PART = ALL>
__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) {
  typedef __attribute__((ext_vector_type(4))) short s16x4;
  if constexpr (PART == ALL) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  } else {
    auto half = [](bf16x8 v) {
      const u32x4 u = __builtin_bit_cast(u32x4, v);
      return __builtin_bit_cast(s16x4, PART == LOW ? u32x2{u[0], u[1]} : u32x2{u[2], u[3]});
    };
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(half(a), half(b), c, 0, 0, 0);
  }
}

// c + a b, small products first.
template <int PART = ALL>
__device__ __forceinline__ f32x4 mfma3(const Split3& a, const Split3& b, f32x4 c) {
  c = mfma_bf16<PART>(a.l, b.h, c);
  c = mfma_bf16<PART>(a.h, b.l, c);
  c = mfma_bf16<PART>(a.m, b.m, c);
  c = mfma_bf16<PART>(a.m, b.h, c);
  c = mfma_bf16<PART>(a.h, b.m, c);
  return mfma_bf16<PART>(a.h, b.h, c);
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
