// The order of the pointwise filters of block_tile.hip, which the launch of the stem puts them in, or one behind it (block_rows.hip).
//
// The operands of the contraction's k-step s (rows 16 s ... + 15) and 64 columns from 64 c on, for each lane: 8 rows from
// 8 (lane / 32) on of column 32 j + lane % 32, part p, at piece 64 (4 (steps c + s) + 2 j + p) + lane; behind them for each column
// 2^17 times the exponent of its scale, plus its losses (pair.h).
#ifndef TFX_PACK_H_
#define TFX_PACK_H_

#include "pair.h"

namespace tfx {

constexpr int kMaxLayers = 13;
struct PackList {
  const float* w[kMaxLayers];
  half_t* out[kMaxLayers];
  int* exps[kMaxLayers];
  int c[kMaxLayers], n[kMaxLayers], first[kMaxLayers + 1];  // first: workgroups of the layers before
  int layers = 0;
  // a layer of c x n; `packed`: separable_tile_packed_bytes(c, n)
  void add(const float* filter, void* packed, int channels, int columns) {
    const int i = layers++;
    w[i] = filter, out[i] = static_cast<half_t*>(packed), exps[i] = reinterpret_cast<int*>(out[i] + (size_t)2 * channels * columns);
    c[i] = channels, n[i] = columns;
    if (i == 0) first[0] = 0;
    first[i + 1] = first[i] + columns / 16;
  }
  int groups() const { return layers == 0 ? 0 : first[layers]; }
};

constexpr int kPackScratch = (16 * 16 + 32) * sizeof(float);

// Workgroup `group`, of WAVES wavefronts (0: any number up to 16): 16 columns.  HELD: pairs of k-steps of a wavefront on their way at a time.  scratch:
// kPackScratch bytes of LDS.
template <int HELD, int WAVES = 0>
__device__ __forceinline__ void pack_filters(const PackList& g, int group, float* scratch) {
  float* const wave_most = scratch;  // [wave][16]
  int* const lost = reinterpret_cast<int*>(scratch + 16 * 16);
  int* const tiny = lost + 16;
  int l = 0;
  while (l + 1 < g.layers && group >= g.first[l + 1]) ++l;
  const int waves = WAVES > 0 ? WAVES : (int)blockDim.x / 64, wave = threadIdx.x / 64, lane = threadIdx.x % 64, li = lane % 16, q = lane / 16;
  const int N = g.n[l], steps = g.c[l] / 16;
  int nb = group - g.first[l];
  if (N % 256 == 0 && g.first[l] % 8 == 0) nb = nb / 16 * 16 + nb % 8 * 2 + nb / 8 % 2;  // the two halves of a line on one XCD
  const int n = 16 * nb + li;
  const float* const w = g.w[l] + n;
  // lane (li, q) has rows 8 (q % 2) ... of step q / 2 of a pair; of a wavefront's pairs in excess of HELD all but the last ones are read twice
  const int chunks = 2 * WAVES * HELD >= 64 ? 1 : (steps + 2 * waves * HELD - 1) / (2 * waves * HELD);
  auto fetch = [&](int pair, float (&v)[8]) __attribute__((always_inline)) {
    const int s = min(2 * pair + q / 2, steps - 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = w[(size_t)(16 * s + 8 * (q % 2) + i) * N];
  };
  float most = 0.f;
  auto see = [&](const float (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) most = __builtin_isfinite(v[i]) ? fmaxf(most, fabsf(v[i])) : most;
  };
  float v[HELD][8];
  auto fetch_chunk = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < HELD; ++u) fetch(wave + waves * (HELD * chunk + u), v[u]);
  };
  for (int chunk = 0; chunk < chunks; ++chunk) {
    fetch_chunk(chunk);
#pragma unroll
    for (int u = 0; u < HELD; ++u) see(v[u]);
  }
  most = fmaxf(most, __shfl_xor(most, 32));
  most = fmaxf(most, __shfl_xor(most, 16));
  if (q == 0) wave_most[16 * wave + li] = most;
  if (threadIdx.x < 16) lost[threadIdx.x] = tiny[threadIdx.x] = 0;
  __syncthreads();
  for (int i = 0; i < waves; ++i) most = fmaxf(most, wave_most[16 * i + li]);
  const int e = column_exponent(most);
  int loses = 0;
  auto store = [&](int pair, const float (&v)[8]) __attribute__((always_inline)) {
    const int s = 2 * pair + q / 2;
    if (s >= steps) return;
    h8 part[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      half_t a, b;
      loses = more_lost(loses, split_filter(v[i], e, a, b));
      part[0][i] = a, part[1][i] = b;
    }
    h8* const out = reinterpret_cast<h8*>(g.out[l]) + (size_t)64 * (4 * (steps * (nb / 4) + s) + 2 * (nb / 2 % 2)) + 32 * (q % 2) + 16 * (nb % 2) + li;
    out[0] = part[0];
    out[64] = part[1];
  };
  for (int chunk = chunks - 1; chunk >= 0; --chunk) {
    if (chunk != chunks - 1) fetch_chunk(chunk);
#pragma unroll
    for (int u = 0; u < HELD; ++u) store(wave + waves * (HELD * chunk + u), v[u]);
  }
  if (loses != 0) {
    atomicAdd(&lost[li], loses & kLostMost);
    if ((loses & kLostTiny) != 0) atomicOr(&tiny[li], kLostTiny);
  }
  __syncthreads();
  if (threadIdx.x < 16) g.exps[l][n] = (e << 17) | lost[li] | tiny[li];
}

}  // namespace tfx

#endif  // TFX_PACK_H_
