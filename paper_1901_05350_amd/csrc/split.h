// fp32 products on the bf16 matrix cores, without loss: what the fp32 kernels share.
//
// The fp32 matrix instructions of this chip run at 1/16 of the rate of the bf16 ones (157 against 2500 TFLOP/s), so six
// bf16 products per fp32 product still leave 2.7 times the rate.  A float a with 24 significant bits is the exact sum
// hi + mid + lo of three bf16 values (8 bits each): hi = bf16(a), mid = bf16(a - hi), lo = a - hi - mid, both
// differences exact.  A product a b is then the sum of nine products of bf16 values, each exact in fp32; the six of them
// that reach 2^-24 of |a b| are accumulated in fp32 by the matrix cores, and the three that do not (mid lo, lo mid,
// lo lo) are left out: they are below the rounding that every accumulation of an fp32 product makes.  A k-step of the
// bf16 instructions adds 16 products with one rounding, the fp32 ones round after every product, so the sum comes out more accurate:
// against float64, normal operands, relative 2-norm error for K = 128 / 512 / 2048: 1.5e-7 / 3.4e-7 / 6.9e-7 here,
// 2.0e-7 / 4.1e-7 / 8.1e-7 with v_mfma_f32_16x16x4_f32; operands uniform in [0, 1): 1.2e-7 / 2.4e-7 / 3.8e-7 against
// 1.6e-7 / 3.1e-7 / 6.0e-7.  A sum of one or two products, though, has fewer roundings with the fp32 instructions (normal
// operands, K = 1 / 2 / 3 / 4 / 8: 3.5e-8 / 3.4e-8 / 3.3e-8 / 3.3e-8 / 3.1e-8 here, 2.5e-8 / 3.1e-8 / 3.6e-8 / 4.0e-8 / 5.3e-8
// there): contractions of up to kFewProducts take those.
//
// Two kinds of values do not survive the split; what they reach is computed again with the fp32 instructions:
//   - Inf, NaN and magnitudes that round past the largest bf16: a result that they reach is Inf or NaN (so is one that
//     really overflows), which is looked for once, after the loop; the finite results beside it stay;
//   - magnitudes below 2^-110 ("tiny"), whose last bits can lie below the smallest bf16, 2^-133 (conversions, subtractions
//     and matrix instructions of this chip keep subnormals): each loses up to 2^-134.  SplitGuard sees whether any bit was
//     lost.  With operands below 2^20 a sum of K products then misses less than K 2^-113, which no sum of 2^24 times that
//     size (small_limit) notices: only smaller results are computed again, all of them after a larger operand.
//     (8 x 1024^3, 1 value in 1000 at 1e-38: 959 us when every tile with a tiny value was computed again, now as without.)
#ifndef TFX_SPLIT_H_
#define TFX_SPLIT_H_

#include "tfx_internal.h"

namespace tfx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kParts = 3, kFewProducts = 2;

// bf16(a) in the low half, bf16(b) in the high half (round to nearest even, one instruction)
__device__ __forceinline__ unsigned to_bf16_pair(float a, float b) {
  typedef __bf16 pair __attribute__((ext_vector_type(2)));
  typedef float floatx2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, pair));
}

// hi, mid and lo of four floats; `low` collects the bits of the last remainders, whose lower halves are zeros unless the
// split loses something.  (The differences as bf16 dot products with (-1, 0) and (0, -1), one instruction instead
// of two, were slower: that instruction does not overlap with matrix instructions.)
typedef unsigned splitx4 __attribute__((ext_vector_type(2)));  // four bf16
__device__ __forceinline__ void split4(floatx4 v, splitx4 (&part)[kParts], unsigned& low) {
#pragma unroll
  for (int p = 0; p < kParts; ++p)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned pair = to_bf16_pair(v[2 * i], v[2 * i + 1]);
      part[p][i] = pair;
      if (p == kParts - 1) {
        low |= __float_as_uint(v[2 * i]) | __float_as_uint(v[2 * i + 1]);
      } else {
        v[2 * i] -= __uint_as_float(pair << 16);
        v[2 * i + 1] -= __uint_as_float(pair & 0xffff0000u);
      }
    }
}

// acc += A B for one k-step of 16 (32 x 32 tile); smallest products first
__device__ __forceinline__ constexpr int split_pass_a(int s) { return s == 0 ? 1 : s == 1 ? 0 : s == 2 ? 2 : s == 3 ? 1 : 0; }
__device__ __forceinline__ constexpr int split_pass_b(int s) { return s == 0 ? 1 : s == 1 ? 2 : s == 2 ? 0 : s == 3 ? 0 : s == 4 ? 1 : 0; }
constexpr int kSplitPasses = 6;  // (mid, mid), (hi, lo), (lo, hi), (mid, hi), (hi, mid), (hi, hi)

// What a thread saw of the operands that it split: one vector instruction per value.
struct SplitGuard {
  float most = 0.f;  // largest magnitude; NaN is not seen
  unsigned low = 0;
  __device__ __forceinline__ void split(const floatx4& v, splitx4 (&part)[kParts]) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(most) : "v"(v[0]), "v"(v[1]));
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(most) : "v"(v[2]), "v"(v[3]));
    split4(v, part, low);
  }
  __device__ __forceinline__ bool large() const { return !(most < 0x1p20f); }
  __device__ __forceinline__ bool lost() const { return (low & 0xffffu) != 0; }
};
// a sum of K products (plus bias) of at least this magnitude does not depend on what tiny operands lose
__device__ __forceinline__ float small_limit(int products) { return (float)products * 0x1p-89f; }

// nonzero and below 2^-110
__device__ __forceinline__ bool is_tiny(float v) { return (__float_as_uint(v) << 1) - 1u < (17u << 24) - 1u; }
__device__ __forceinline__ bool any_tiny(const floatx4& v) { return is_tiny(v[0]) || is_tiny(v[1]) || is_tiny(v[2]) || is_tiny(v[3]); }

// largest |bits| of accumulators so far; Inf and NaN are the ones with a full exponent
__device__ __forceinline__ void see_result(unsigned& most, float v) { most = max(most, __float_as_uint(v) << 1); }
__device__ __forceinline__ bool overflowed(unsigned most) { return most >= 0xff000000u; }

}  // namespace tfx

#endif  // TFX_SPLIT_H_
