// fp32 products on the bf16 matrix cores, without loss of precision.
//
// An fp32 value is the sum of three bf16 values: hi = x rounded to bf16, mid =
// (x - hi) rounded to bf16, lo = x - hi - mid (both differences are exact, and
// 3 x 8 significand bits hold the 24 of an fp32 value, so lo is exact too,
// unless it is too small for a bf16 value).  Values are therefore multiplied by
// 2^24 before they are split: a part is then a multiple of 2^-125, since an
// fp32 value is one of 2^-149, and none is subnormal.  Sums of products are
// multiplied by 2^-48 at the end; both factors are exact.  Without them a
// value of 2^-120 keeps 14 of its bits.
//
// A product x w is then the sum of nine bf16 products, each exact in fp32.  Six
// are kept: lo hi', hi lo', mid mid', mid hi', hi mid', hi hi'.  Rounding to
// nearest bounds mid by 2^-8 |x| and lo by 2^-17 |x|, so the three left out
// are below 2^-24 |x w| together (2^-27 in the mean, of either sign), less
// than the rounding of one fp32 product.
//
// A bf16 MFMA (16x16x32, 16 cycles) has 16 times the rate of the fp32 one
// (16x16x4, 32 cycles), so six of them do the same work in 3/8 of the time.
//
// Values of 2^103 (1e31) and more, infinities and NaN have no such sum, and
// results of 2^80 (1.2e24) and more overflow: a kernel that uses it checks its
// accumulators and works out what is not finite once more in plain fp32.
#pragma once

#include "common.h"

namespace oc {

typedef float s3_v4f __attribute__((ext_vector_type(4)));
typedef float s3_v2f __attribute__((ext_vector_type(2)));
typedef uint32_t s3_v2u __attribute__((ext_vector_type(2)));
typedef uint32_t s3_v4u __attribute__((ext_vector_type(4)));
typedef __bf16 s3_v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 s3_v8bf __attribute__((ext_vector_type(8)));

struct Split8 {  // eight values' parts, as operands of one MFMA lane
  s3_v4u p[3];   // hi, mid, lo
};

// Two values rounded to bf16 (nearest, ties to even), the first in the low half.
__device__ __forceinline__ uint32_t s3_round2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((s3_v2f){a, b}, s3_v2bf));
}

// (-1, 0) and (0, -1) as bf16 pairs, in scalar registers: as literals, the
// first would become the inline constant -1.0, which this instruction reads as
// the fp32 value, that is (0, -1).
struct SplitK {
  s3_v2bf lo, hi;
};
__device__ __forceinline__ SplitK s3_consts() {
  uint32_t a = 0x0000bf80u, b = 0xbf800000u;
  asm("" : "+s"(a));
  asm("" : "+s"(b));
  return SplitK{__builtin_bit_cast(s3_v2bf, a), __builtin_bit_cast(s3_v2bf, b)};
}

constexpr float kSplitUp = 0x1p24f;     // factor of a value before it is split
constexpr float kSplitDown = 0x1p-48f;  // factor of a sum of products

// Parts of two scaled values, packed as s3_round2 does.  A difference is one dot
// product of the rounded pair with (-1, 0) or (0, -1), added to the value; it
// equals the fp32 subtraction bit for bit (subnormal results included).
__device__ __forceinline__ void s3_split2(const SplitK& k, float a, float b, uint32_t& h,
                                          uint32_t& m, uint32_t& l) {
  h = s3_round2(a, b);
  const s3_v2bf hb = __builtin_bit_cast(s3_v2bf, h);
  a = __builtin_amdgcn_fdot2_f32_bf16(hb, k.lo, a, false);
  b = __builtin_amdgcn_fdot2_f32_bf16(hb, k.hi, b, false);
  m = s3_round2(a, b);
  const s3_v2bf mb = __builtin_bit_cast(s3_v2bf, m);
  a = __builtin_amdgcn_fdot2_f32_bf16(mb, k.lo, a, false);
  b = __builtin_amdgcn_fdot2_f32_bf16(mb, k.hi, b, false);
  l = s3_round2(a, b);
}

// Four values' parts, scaled by up (kSplitUp or -kSplitUp).
__device__ __forceinline__ void s3_split4(const SplitK& k, const s3_v4f& v, s3_v2u (&p)[3],
                                          float up = kSplitUp) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    uint32_t h, m, l;
    s3_split2(k, v[2 * i] * up, v[2 * i + 1] * up, h, m, l);
    p[0][i] = h, p[1][i] = m, p[2][i] = l;
  }
}

__device__ __forceinline__ Split8 s3_split8(const SplitK& k, const s3_v4f& a, const s3_v4f& b) {
  Split8 r;
  const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t h, m, l;
    s3_split2(k, v[2 * i] * kSplitUp, v[2 * i + 1] * kSplitUp, h, m, l);
    r.p[0][i] = h, r.p[1][i] = m, r.p[2][i] = l;
  }
  return r;
}

__device__ __forceinline__ s3_v4f s3_mfma(const s3_v4u& a, const s3_v4u& b, const s3_v4f& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(s3_v8bf, a),
                                                 __builtin_bit_cast(s3_v8bf, b), c, 0, 0, 0);
}

// Product i = 0..5 of a and b added to c (in units of 2^-48), the smallest first.
__device__ __forceinline__ s3_v4f s3_product(int i, const s3_v4u (&a)[3], const s3_v4u (&b)[3],
                                             const s3_v4f& c) {
  constexpr int ia[6] = {2, 0, 1, 1, 0, 0}, ib[6] = {0, 2, 1, 0, 1, 0};
  return s3_mfma(a[ia[i]], b[ib[i]], c);
}

// True when one of the four values is infinite or NaN.
__device__ __forceinline__ bool s3_bad(const s3_v4f& v) {
  const float t = fmaf(v[0], 0.f, v[1] * 0.f) + fmaf(v[2], 0.f, v[3] * 0.f);
  return !(t == 0.f);
}

}  // namespace oc
