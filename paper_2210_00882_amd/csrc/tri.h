// fp32 products on the bf16 matrix pipe.
//
// The fp32 MFMA runs at a sixteenth of the bf16 one's rate, and with it the fp32 networks spend most of their time on
// the matrix pipe.  So every fp32 operand is taken apart into three bf16 pieces,
//     x = x0 + x1 + x2,   x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1)   (round to nearest even),
// which is exact (3 x 8 significant bits hold the 24 of an fp32 value; the two differences are exact in fp32), and a
// product becomes six bf16 MFMAs into one fp32 accumulator,
//     w x = w2 x0 + w1 x0 + w1 x1 + w0 x0 + w0 x1 + w0 x2.
// The three products left out are below 2^-24 of w x (|x1| <= 2^-8 |x|, |x2| <= 2^-17 |x|), i.e. below the rounding
// of the fp32 product they stand in for, and 16 inputs enter the accumulator per rounding instead of two.  Six bf16
// MFMAs of 16 inputs take 192 cycles where eight fp32 ones take 512.
#pragma once
#include "dev_common.h"

namespace msrl {

typedef float f32x8 __attribute__((ext_vector_type(8)));

// one operand: 8 values of a row as three bf16 pieces
struct Tri {
  u32x4 p[3];
};

__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {  // round to nearest even, a in the low half
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// v minus the low / high half of a bf16 pair: one dot product with (-1, 0) or (0, -1), exact here like the
// subtraction it stands for (the difference of a value and its rounding has no more bits than the value).  The
// constants are hidden from the compiler, which would turn the first into the inline constant -1.0, a value of
// the high half.
__device__ __forceinline__ float minus_low(float v, uint32_t w) {
  uint32_t c = 0x0000BF80u;
  asm("" : "+s"(c));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, c), v, false);
}
__device__ __forceinline__ float minus_high(float v, uint32_t w) {
  uint32_t c = 0xBF800000u;
  asm("" : "+s"(c));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, c), v, false);
}

// the pieces of values a, b as pair `i` of an operand
__device__ __forceinline__ void tri_pair(float a, float b, Tri& o, int i) {
  const uint32_t p0 = bf16_pair(a, b);
  a = minus_low(a, p0);
  b = minus_high(b, p0);
  const uint32_t p1 = bf16_pair(a, b);
  o.p[0][i] = p0;
  o.p[1][i] = p1;
  o.p[2][i] = bf16_pair(minus_low(a, p1), minus_high(b, p1));
}
// the network's input (observations): an infinity has no pieces (its remainder would be NaN) and takes part as the
// largest bf16 value, which saturates the same units; a NaN stays one
__device__ __forceinline__ Tri tri_operand(const f32x8& f) {
  Tri o;
#pragma unroll
  for (int i = 0; i < 4; ++i) tri_pair(bf16_range(f[2 * i]), bf16_range(f[2 * i + 1]), o, i);
  return o;
}
__device__ __forceinline__ f32x16 mma_piece(const u32x4& w, const u32x4& x, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
}
// piece of the weight / of the operand in MFMA m of a k tile; the pieces of the weight are used up in the order 2, 1, 0
// (two accumulators in turn, one for the three smallest products, were measured: 2 to 6 % slower, the chain of
// dependent MFMAs is no bound)
constexpr int TRI_W[6] = {2, 1, 1, 0, 0, 0}, TRI_X[6] = {0, 0, 1, 0, 1, 2};

}  // namespace msrl
