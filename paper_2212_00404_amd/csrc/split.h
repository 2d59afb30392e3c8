// fp32 operands on the bf16 matrix cores: each value is split into three
// bf16 values, and a product of two values becomes six bf16 products.
//
// gfx950's bf16 matrix instructions run sixteen times the rate of its fp32
// ones, so six of them per product are 2.7 times as fast.  The operands are
// held exactly:
//   2^16 x = h + m + l,  h = bf16(2^16 x), m = bf16(2^16 x - h),
//   l = bf16(2^16 x - h - m)
// (round to nearest each time; both differences exact) for every fp32 value
// below 2^112: 24 significant bits in three times 8, and the smallest fp32
// value, 2^-149, at the smallest bf16 one, 2^-133 (without the factor every
// value below 2^-110 lost low bits, those below 2^-134 all of them).  The sum
// is divided by 2^32 at the end, exactly.  With |m| <= 2^-8 |h| and
// |l| <= 2^-17 |h|, the three products left out of  (h+m+l)(h'+m'+l')
// (m l', l m', l l') are below 2^-24 of h h' in all, a rounding of the product.
// Products of bf16 values are exact in the matrix core, which adds in fp32
// with round to nearest and keeps denormals.  The sum rounds once per
// instruction (16 or 32 terms) and not once per term or two; the corrections
// go to an accumulator of their own, so that their small roundings stay small.
// Against 64-bit sums of 32 to 4608 random terms the result measured 0.3 to
// 0.4 times the error of the fp32 matrix instructions.
//
// Infinities, NaN and large values: the difference from h is NaN where h is
// infinite, so a non-finite operand, one of 2^112 and above, or a zero of a
// padded operand against it, makes the result non-finite; a sum of 2^96 and
// above may overflow.  Each kernel tests its results and sums a non-finite one
// again from memory with fp32 FMAs, which gives what the fp32 kernels give.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace dconv {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

// Two floats to packed bf16, round to nearest (one instruction); a in the
// low half.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const floatx2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ float bf16_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// The three bf16 parts of eight scaled fp32 values: a lane's operands of the 16x16x32
// and 32x32x16 instructions (eight consecutive k).
struct Split8 {
  bf16x8 h, m, l;
};

// The factors of an operand and of a sum of products.
constexpr float kSplitScale = 65536.f, kSplitUnscale = 1.f / (kSplitScale * kSplitScale);

// Two values: the packed pairs of each part of kSplitScale times them.
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
  a *= kSplitScale;
  b *= kSplitScale;
  h = pack_bf16(a, b);
  const float ra = a - bf16_lo(h), rb = b - bf16_hi(h);
  m = pack_bf16(ra, rb);
  l = pack_bf16(ra - bf16_lo(m), rb - bf16_hi(m));
}

__device__ __forceinline__ Split8 split8(const float (&v)[8]) {
  uintx4 h, m, l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t a, b, c;
    split2(v[2 * i], v[2 * i + 1], a, b, c);
    h[i] = a;
    m[i] = b;
    l[i] = c;
  }
  Split8 s;
  s.h = __builtin_bit_cast(bf16x8, h);
  s.m = __builtin_bit_cast(bf16x8, m);
  s.l = __builtin_bit_cast(bf16x8, l);
  return s;
}

}  // namespace dconv
