// fp32 products on the binary16 matrix cores, operands split in two: the blocks of block_tile.hip.
//
// (H. Ootomo and R. Yokota, Recovering single precision accuracy from Tensor Cores while surpassing the FP32 theoretical peak
// performance, 2022: two halves, the second times 2^11, with sums of their own.)  a = h + l / 2^11 with h the nearest half and l the
// nearest half of 2^11 times the remainder: 22 bits and the remainder's sign, so the pair misses at most the last bit of a float's 24
// (half of its place where the remainder needs 12 bits, a value in four).  Three or four products of halfs (h h, h l, l h, and l l, 2^-24 of the product
// on average) stand for one of floats, where three bf16 parts (split.h) take six, and two planes for three.  The h h products and
// the others, which are 2^11 times too large, have accumulators of their own: the others lose nothing beside the large ones, and
// these are rounded once for 16 products.
//
// Error of a block against float64: 64 images, three products, 512 -> 512 1.8e-7, 256 -> 256 1.3, 1024 -> 1024 2.3, with three bf16
// parts and one accumulator 3.3, 2.0, 4.7; whole passes' logits, 64 images 2.3 and 4.0, 8 images (four products, the large ones of
// four k-steps summed apart) 1.9 and 2.6, 3/4 width 33 images 2.1 and 2.7.  Where a contraction is short or split, as it is for fewer
// outputs, three parts are the more exact: such blocks stay with them (api.hip).
//
// Binary16 has few exponents, so operands are scaled by powers of two: a depthwise output, 0 ... 6, by 2^13, a column of a filter
// so that its largest value is in [2^14, 2^15).  That holds here, where one operand has bounds and the other a scale a column.  Matrix
// products do not: with a scale a tile, one value of 1000 among normal ones sent 8 x 1024^3 from 78 to 347 us (three bf16 parts 92).
//
// Values that the split does not carry: a scaled value below 2^-14 loses up to 2^-36, one below 2^-60 no more than itself.  With
// operands below 2^16 a sum of K products, n of them with the first, then misses less than n 2^-20 + K 2^-44, which a result of 2^24
// times that does not notice (loss_limit): smaller ones are computed again in fp32 where an operand lost bits.  So are results that
// are Inf or NaN because of the filter, whose other than finite values are NaN here.  (With one bound for both kinds a thousandth of
// the filter at 1e-32, which reaches no result, made a pass of 8 images 1.32 times as long; with n = K the few of a map's values
// that lie within 2^-27 of zero by chance cost 50 us in one pass of three.)
#ifndef TFX_PAIR_H_
#define TFX_PAIR_H_

#include "tfx_internal.h"

namespace tfx {

typedef _Float16 half_t;
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

constexpr int kMapScale = 13;  // depthwise outputs times 2^13
constexpr float kLow = 2048.f;  // second parts times 2^11

// Both parts of a scale and b scale, the first in the low halves.  The remainder is exact before it is rounded.  (In C++ the compiler
// converts twice, once for h and once for the remainder: six instructions a value instead of three and a half.)
__device__ __forceinline__ void split2(float a, float b, float scale, unsigned& h, unsigned& l) {
  const float low = scale * kLow;
  asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(h) : "v"(a * scale), "v"(b * scale));
  asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]\n\tv_fma_mixhi_f16 %0, %1, %2, %4 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
      : "=&v"(l)
      : "v"(h), "s"(-kLow), "v"(a * low), "v"(b * low));
}
typedef unsigned pairx4 __attribute__((ext_vector_type(2)));  // four halfs
__device__ __forceinline__ void split2(const floatx4& v, float scale, pairx4& h, pairx4& l) {
  unsigned h0, h1, l0, l1;
  split2(v[0], v[1], scale, h0, l0);
  split2(v[2], v[3], scale, h1, l1);
  h = pairx4{h0, h1}, l = pairx4{l0, l1};
}

// What operands lose: how many of them up to 2^-36 (kLostMost: more than the 1024 of a contraction), plus kLostTiny where one loses up to 2^-60.
constexpr int kLostMost = 0xffff, kLostTiny = 0x10000;
__device__ __forceinline__ int more_lost(int a, int b) { return min((a & kLostMost) + (b & kLostMost), kLostMost) | ((a | b) & kLostTiny); }

// Depthwise outputs, none of them negative: the least bits of those from 2^-73 on and of all but zeros.
struct MapLoss {
  unsigned from = ~0u, all = ~0u;
  __device__ __forceinline__ void see(float v) {
    from = min(from, __float_as_uint(v) - kFrom);
    all = min(all, __float_as_uint(v) - 1u);
  }
  __device__ __forceinline__ int lost(int seen) const { return (from < kTo - kFrom ? seen : 0) | (all < kFrom - 1u ? kLostTiny : 0); }
  static constexpr unsigned kFrom = (127u - 60 - kMapScale) << 23, kTo = (127u - 14 - kMapScale) << 23;
};

// Exponent of the scale of a column whose largest finite magnitude is `most`.
__device__ __forceinline__ int column_exponent(float most) {
  int e = 15;
  if (most > 0.f) (void)frexpf(most, &e);
  return 15 - e;
}
// both parts of a filter value in a column of exponent e; its losses
__device__ __forceinline__ int split_filter(float w, int e, half_t& h, half_t& l) {
  const float t = ldexpf(w, e);
  const bool finite = __builtin_isfinite(t);
  h = finite ? (half_t)t : (half_t)NAN;
  l = finite ? (half_t)((t - (float)(half_t)t) * kLow) : (half_t)0.f;
  return w == 0.f || !(fabsf(t) < 0x1p-14f) ? 0 : fabsf(t) < 0x1p-60f ? kLostTiny : 1;
}

// The result, of operands scaled by 2^e together, below which lost bits are noticed.
__device__ __forceinline__ float loss_limit(int products, int e, int lost) {
  const int n = min(lost & kLostMost, products);
  return lost == 0 ? 0.f : ldexpf(n != 0 ? (float)n : (float)products, (n != 0 ? 5 : -20) - e);
}

}  // namespace tfx

#endif  // TFX_PAIR_H_
