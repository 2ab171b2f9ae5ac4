// Loads for operands whose rows start at any address and end at any element: what the kernels for sizes that are
// no multiple of a vector load share.
//
// A chunk of 16 bytes (4 floats or 8 halfs) is fetched with one load whatever its alignment (global loads of this
// target need none).  The last chunk of a row is only partly valid; instead of a branch per element, the load is
// unconditional and the elements past the row's end are zeroed when the registers are consumed.  Only at the very end
// of a tensor would such a load leave it: there it starts early enough to end with the tensor, and the registers are
// shifted down by the difference when they are consumed (a wave-wide test skips that almost always).
#ifndef TFX_RAGGED_H_
#define TFX_RAGGED_H_

#include "tfx_internal.h"

namespace tfx {

typedef unsigned ragged_u32x4 __attribute__((ext_vector_type(4)));
typedef ragged_u32x4 ragged_u32x4_any __attribute__((aligned(2)));  // 16 bytes at any half's address

template <typename T>
__device__ __forceinline__ ragged_u32x4 load16(const T* p) {
  return *reinterpret_cast<const ragged_u32x4_any*>(p);
}

// Registers of a chunk that was fetched `s` elements (0 ... elements per chunk) too early: element e <- element e + s.
template <typename T>
__device__ __forceinline__ ragged_u32x4 shift_down(ragged_u32x4 v, unsigned s) {
  const unsigned d = s * sizeof(T) / 2;  // in halfs
  if (d & 8) v = ragged_u32x4{0, 0, 0, 0};
  if (d & 4) v = ragged_u32x4{v[2], v[3], 0, 0};
  if (d & 2) v = ragged_u32x4{v[1], v[2], v[3], 0};
  if constexpr (sizeof(T) == 2)
    if (d & 1)
      v = ragged_u32x4{__builtin_amdgcn_alignbit(v[1], v[0], 16), __builtin_amdgcn_alignbit(v[2], v[1], 16),
                       __builtin_amdgcn_alignbit(v[3], v[2], 16), v[3] >> 16};
  return v;
}

// Mask of the first r elements (r <= 0: none, r >= elements per chunk: all) of a chunk.
template <typename T>
__device__ __forceinline__ ragged_u32x4 first_elements(int r) {
  ragged_u32x4 m;
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int d = 0; d < 4; ++d) m[d] = r > d ? ~0u : 0u;
  } else {
#pragma unroll
    for (int d = 0; d < 4; ++d) m[d] = r >= 2 * d + 2 ? ~0u : (r == 2 * d + 1 ? 0xffffu : 0u);
  }
  return m;
}

// Division of 0 <= n < 2^31 by a constant d >= 1 of the launch: n / d = (n * mul) >> (31 + shift) with the smallest
// shift such that 2^shift >= d and mul = ceil(2^(31 + shift) / d), which fits 32 bits and is exact for such n.
struct FastDiv {
  unsigned mul, shift, d;
};
inline FastDiv fast_div(unsigned d) {
  unsigned s = 0;
  while ((1ull << s) < d) ++s;
  return FastDiv{(unsigned)(((1ull << (31 + s)) + d - 1) / d), s, d};
}
__device__ __forceinline__ unsigned div_by(unsigned n, const FastDiv& f) {
  return (unsigned)(((unsigned long long)n * f.mul) >> (31 + f.shift));
}

}  // namespace tfx

#endif  // TFX_RAGGED_H_
