// fp32 operands on the bf16 matrix cores (gfx950): an fp32 number is the exact sum of three bf16 numbers, eight
// significand bits each, taken by truncation (splitting into summands of lower precision, as in Dekker's products and Ozaki's
// matrix products).  The second is below 2^-7, the third below 2^-15 of the number, both of its sign.  A product of two such
// sums is the six products of planes i and j with i + j <= 2, each exact in the MFMA's fp32 accumulation; the three left out
// add up to 2^-21 of the product at most, 2^-24.6 on average over random operands, always towards zero.  (Planes by
// rounding: 2^-24 at most, 2^-28 on average and of either sign.  Measured against fp64 over a whole call that changes errors
// of 0.6 to 1.1e-6, which come from the accumulation, by about a tenth, and costs 2 % of the fp32 calls.)  Six 32x32x16
// bf16 MFMAs take 192 cycles where the fp32 MFMA (32x32x2, 64 cycles) takes 512 for the same 32x32x16 product, and three
// suffice where one operand is a bf16 input.  bf16 has fp32's exponent range, so no scaling is needed; what bf16 cannot
// represent is lost, 2^-133 per element: numbers under 2^-109 have fewer than 24 bits here.
#pragma once

#include "fused_common.h"

namespace dark {
namespace sp {
using namespace fz;

typedef unsigned short us;

// Two neighbouring elements -> the packed pairs of the three planes.
__device__ __forceinline__ void split_pair(float a, float b, unsigned& p0, unsigned& p1, unsigned& p2) {
  const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
  p0 = __builtin_amdgcn_perm(ub, ua, 0x07060302u);   // the upper halves of both
  const float a1 = a - __uint_as_float(ua & 0xffff0000u), b1 = b - __uint_as_float(ub & 0xffff0000u);
  const unsigned ua1 = __float_as_uint(a1), ub1 = __float_as_uint(b1);
  p1 = __builtin_amdgcn_perm(ub1, ua1, 0x07060302u);
  const float a2 = a1 - __uint_as_float(ua1 & 0xffff0000u), b2 = b1 - __uint_as_float(ub1 & 0xffff0000u);
  p2 = __builtin_amdgcn_perm(__float_as_uint(b2), __float_as_uint(a2), 0x07060302u);
}
// Eight neighbouring elements (one lane's share of an operand fragment) -> three planes.
__device__ __forceinline__ void split8(const f32x4& lo, const f32x4& hi, u32x4 (&p)[3]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    unsigned a, b, c;
    split_pair(lo[2 * q], lo[2 * q + 1], a, b, c);
    p[0][q] = a; p[1][q] = b; p[2][q] = c;
    split_pair(hi[2 * q], hi[2 * q + 1], a, b, c);
    p[0][2 + q] = a; p[1][2 + q] = b; p[2][2 + q] = c;
  }
}
__device__ __forceinline__ f32x16 mm(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8*>(&a), *reinterpret_cast<bf16x8*>(&b), c, 0, 0, 0);
}
// c += the products of planes below the leading one (the smallest first), and the leading one.
template <int NA, int NB>
__device__ __forceinline__ f32x16 mm_low(const u32x4 (&a)[NA], const u32x4 (&b)[NB], f32x16 c) {
#pragma unroll
  for (int t = 2; t >= 1; --t)
#pragma unroll
    for (int i = 0; i <= t; ++i)
      if (i < NA && t - i < NB) c = mm(a[i], b[t - i], c);
  return c;
}
template <int NA, int NB>
__device__ __forceinline__ f32x16 mm_all(const u32x4 (&a)[NA], const u32x4 (&b)[NB], f32x16 c) {
  return mm(a[0], b[0], mm_low(a, b, c));
}

// Logits of a 32 x 32 block, X (inputs, NX planes) times A' (three planes), either one being the MFMA's first operand.  The leading
// products and the others are summed apart and added at the end: four roundings at the size of the logit instead of
// twenty-four.  Every kernel that forms a logit forms the same bits, whichever way its operands lie (the planes meet in the
// order of X's): what is stored under one rounding of a feature then meets the same rounding of it elsewhere.
struct Logits {
  f32x16 hi, lo;
  __device__ __forceinline__ Logits() : hi{}, lo{} {}
  template <int NX>
  __device__ __forceinline__ void add_xa(const u32x4 (&x)[NX], const u32x4 (&a)[3]) {
#pragma unroll
    for (int t = 2; t >= 1; --t)
#pragma unroll
      for (int i = 0; i <= t; ++i)
        if (i < NX) lo = mm(x[i], a[t - i], lo);
    hi = mm(x[0], a[0], hi);
  }
  template <int NX>
  __device__ __forceinline__ void add_ax(const u32x4 (&a)[3], const u32x4 (&x)[NX]) {
#pragma unroll
    for (int t = 2; t >= 1; --t)
#pragma unroll
      for (int i = 0; i <= t; ++i)
        if (i < NX) lo = mm(a[t - i], x[i], lo);
    hi = mm(a[0], x[0], hi);
  }
  __device__ __forceinline__ f32x16 sum() const { return hi + lo; }
};

// Planes of one operand element group as loaded from an input tensor: 8 elements of type fp32 (NP = 3) or bf16 (NP = 1).
template <int NP>
struct Raw8;
template <>
struct Raw8<3> {
  f32x4 lo, hi;
  __device__ __forceinline__ void load(const void* base, size_t elem) {
    const f32x4* q = reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(base) + elem);
    lo = q[0];
    hi = q[1];
  }
  __device__ __forceinline__ void planes(u32x4 (&p)[3]) const { split8(lo, hi, p); }
};
template <>
struct Raw8<1> {
  u32x4 w;
  __device__ __forceinline__ void load(const void* base, size_t elem) {
    w = *reinterpret_cast<const u32x4*>(reinterpret_cast<const us*>(base) + elem);
  }
  __device__ __forceinline__ void planes(u32x4 (&p)[1]) const { p[0] = w; }
};

// A 32x32 accumulator, packed, is an operand fragment of the next MFMA whose contraction index runs over its rows; a
// lane of half hf then holds rows 16 hh + 4 hf + [0,4) and 16 hh + 8 + 4 hf + [0,4) of step hh.  Matrices that meet
// such a fragment are stored with the rows of every 16 in that order (bits 2 and 3 of the index exchanged), so that
// a lane's eight are one 16-byte read.
__host__ __device__ constexpr int chain_pos(int f) { return (f & ~12) | ((f & 4) << 1) | ((f & 8) >> 1); }

}  // namespace sp
}  // namespace dark
