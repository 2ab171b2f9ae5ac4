// What the tiled fp32 kernels (gemm.hip, gemm_pair.hip) share: which elements of a k-slice a thread loads, how it does so anywhere in
// an operand, and where they go in LDS.
#ifndef TFX_GEMM_SLOTS_H_
#define TFX_GEMM_SLOTS_H_

#include "ragged.h"
#include "tfx_internal.h"

namespace tfx {

// Slots of the tiled kernel: s = tid + it * NT;
//   KC : row s / (BK/4), k = 4 * (s % (BK/4)) .. + 3
//   !KC: a thread's four slots are four consecutive k of the same four rows (block b = tid: rows 4 * (b % (ROWS/4)),
//        k = 4 * (b / (ROWS/4)) + it), so that it can hand each row's four k on together
template <int ROWS, int BK, bool KC, int NT, int NSLOT>
__device__ __forceinline__ int slot_row(int tid, int it) {
  static_assert(KC || (NSLOT == 4 && ROWS * BK == 16 * NT), "one 4 x 4 block per thread");
  return KC ? (tid + it * NT) / (BK / 4) : 4 * (tid % (ROWS / 4));
}
template <int ROWS, int BK, bool KC, int NT>
__device__ __forceinline__ int slot_k(int tid, int it) {
  return KC ? 4 * ((tid + it * NT) % (BK / 4)) : 4 * (tid / (ROWS / 4)) + it;
}
__device__ __forceinline__ float f4_get(const float4& v, int s) {
  return s == 0 ? v.x : (s == 1 ? v.y : (s == 2 ? v.z : v.w));
}

__device__ __forceinline__ float4 load_quad(const float* p) { return __builtin_bit_cast(float4, load16(p)); }

// Loads of any k-slice of an operand of at least 4 elements: the loads of a slice (every one unconditional, from a
// valid place) and, when its registers are consumed, what makes them the slice: quads that would have left the operand
// were fetched a few elements early and are shifted down, elements past K are zeroed.
// CV: the operand is a convolution's filter [taps * Ci, N] seen with the channels of a tap padded to a multiple of 4
// (`by_cp.d`), k_total channels per tap.
struct FilterK {
  FastDiv by_cp;
  int taps;
};
template <int ROWS, int BK, bool KC, bool CV, int NT, int NSLOT>
__device__ __forceinline__ unsigned slot_offset(int ld, int rows_total, int k_total, int row0, int k0, int tid, int it,
                                                unsigned total, const FilterK& fk, unsigned* early, int* valid) {
  int gr = row0 + slot_row<ROWS, BK, KC, NT, NSLOT>(tid, it), gk = k0 + slot_k<ROWS, BK, KC, NT>(tid, it);
  unsigned off;
  if (KC) {
    gr = min(gr, rows_total - 1);
    *valid = k_total - gk;
    off = (unsigned)gr * (unsigned)ld + (unsigned)(*valid > 0 ? gk : 0);
  } else {
    if (gr >= rows_total) gr = 0;
    bool in;
    if constexpr (CV) {
      const int tap = (int)div_by((unsigned)gk, fk.by_cp), c = gk - tap * (int)fk.by_cp.d;
      in = tap < fk.taps && c < k_total;
      gk = tap * k_total + c;
    } else {
      in = gk < k_total;
    }
    *valid = in ? 4 : 0;
    off = (unsigned)(in ? gk : 0) * (unsigned)ld + (unsigned)gr;
  }
  const unsigned at = min(off, total - 4u);
  *early = off - at;
  return at;
}
template <int ROWS, int BK, bool KC, bool CV, int NT, int NSLOT>
__device__ __forceinline__ void load_tile_any(const float* __restrict__ g, int ld, int rows_total, int k_total, int row0, int k0,
                                              int tid, unsigned total, const FilterK& fk, float4 (&reg)[NSLOT]) {
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    unsigned early;
    int valid;
    reg[it] = load_quad(g + slot_offset<ROWS, BK, KC, CV, NT, NSLOT>(ld, rows_total, k_total, row0, k0, tid, it, total, fk, &early, &valid));
  }
}
template <int ROWS, int BK, bool KC, bool CV, int NT, int NSLOT>
__device__ __forceinline__ void settle_tile(int ld, int rows_total, int k_total, int row0, int k0, int tid, unsigned total,
                                            const FilterK& fk, float4 (&reg)[NSLOT]) {
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    unsigned early;
    int valid;
    slot_offset<ROWS, BK, KC, CV, NT, NSLOT>(ld, rows_total, k_total, row0, k0, tid, it, total, fk, &early, &valid);
    ragged_u32x4 v = __builtin_bit_cast(ragged_u32x4, reg[it]);
    if (__builtin_amdgcn_ballot_w64(early != 0) != 0) v = shift_down<float>(v, early);
    reg[it] = __builtin_bit_cast(float4, v & first_elements<float>(valid));
  }
}

// LDS tile of one operand: PARTS planes (the parts of split values) of ROWS rows of 32 k, k contiguous, in
// pieces of 8 k (16 bytes).  Rows of a !KC operand are stored in the order row % 4, row / 4: then the writes of a
// wavefront, one row of every thread's 4 x 4 block at a time, and the fragment reads, 32 consecutive rows, both spread
// over all banks with the piece order rotated as below.
template <int ROWS, bool KC, int PARTS>
struct PlaneTile {
  static constexpr int kPlane = ROWS * 64;  // bytes
  static constexpr int kBytes = PARTS * kPlane;
  static __device__ __forceinline__ int at(int row, int piece) {  // byte offset of a piece in its plane
    const int r = KC ? row : (row % 4) * (ROWS / 4) + row / 4;
    const int turn = KC ? (r / 8) & 3 : ((r / 8) ^ row) & 3;
    return r * 64 + ((piece ^ turn) * 16);
  }
};

}  // namespace tfx

#endif  // TFX_GEMM_SLOTS_H_
