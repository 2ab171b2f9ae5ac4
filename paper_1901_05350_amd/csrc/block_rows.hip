// The stem (3x3 stride-2 convolution of the image to 8 Q channels) and the first depthwise-separable block (depthwise 3x3 +
// bias + clamp, pointwise 1x1 to 16 Q channels + bias + clamp) of the Section 3.9 network in one launch, fp32: the structure of
// block_rows_f16.hip.  A workgroup walks down a strip of rows of one image, a wavefront for every 16 columns, with four stem
// rows in LDS: three under the depthwise filter and the one it computes for the next step, with one barrier a row.
//
// Contraction of the stem (v_mfma_f32_16x16x4_f32, filters as the first operand, 7 steps): lane (li, q) supplies seven values of
// pixel li's window; for q < 3 the first seven of the nine that lie next to each other in image row q of it, for q = 3 the last
// two of each row.  The depthwise layer: lane (li, q) has channels 16 u + 4 q ... + 3 of pixel li, which are its operands of
// four steps of the pointwise product.
//
// TWO: the second block too, as in block_rows_f16.hip: a wavefront keeps its 16 columns of one row of the first block's output in LDS,
// adds what the row gives to 8 columns of the second depthwise layer, at stride 2, in registers, and multiplies the rows of that two
// at a time by a filter that lies split in LDS.  That takes a CU's LDS for one workgroup, whose seven wavefronts issue on 1.75 SIMDs
// each: 64 images of 224 x 224 at full width 102 us (and 21 for the filters behind, pack.h), bound by issue and latency (a row 3 us), where this launch and
// the second block's took 73 + 62 and moved the 205 MB between them twice; 8 images 24.6 and 32.7.
#include "pack.h"
#include "split.h"

namespace tfx {
namespace {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct RowsArgs {
  const float *x, *st_w, *st_b, *dw_w, *dw_b, *pw_w, *pw_b;
  float* y;
  int IH, IW, OH, OW, pt, pl, strips, rows;  // rows of a strip, of the output
  unsigned image_bytes, x_bytes, y_bytes;
  // the second block, where it comes too
  const float *dw2_w, *dw2_b, *pw2_w, *pw2_b;
  int OH2, OW2, pt2, pl2;
  int strip_groups;  // workgroups with strips
};

// Pixel stride of the ring in 16-byte pieces: the least without bank conflicts when lane (li, q) reads piece q of pixel li.
struct RowsPixel {
  int pieces;
  constexpr int operator()(int li, int q) const { return li * pieces + q; }
};
template <int Q, bool TWO>
constexpr int rows_pixel_pieces() {
  constexpr int G = (8 * Q + 15) / 16;
  if (TWO && Q == 4) return 4 * G + 1;  // (some conflicts, and room for rows of 112 columns)
  for (int p = 4 * G;; ++p)
    if (conflict_free(RowsPixel{p})) return p;
}

// relu6 of four values.  The median of three drops a NaN, so those are looked for on the side.
__device__ __forceinline__ floatx4 relu6(const floatx4& v) {
  floatx4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = __builtin_amdgcn_fmed3f(v[e], 0.f, 6.f);
  if (__builtin_amdgcn_ballot_w64(__builtin_isunordered(v[0], v[1]) | __builtin_isunordered(v[2], v[3])) != 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = v[e] == v[e] ? o[e] : v[e];
  }
  return o;
}

// The second block's part of LDS, of T wavefronts, in floats behind the ring.
template <int Q>
struct SecondLds {
  static constexpr int N = 16 * Q, N2 = 32 * Q, NB2 = 2 * Q, KS = (Q + 1) / 2, PX = N + 4;
  int map, halo, filter, taps, end;  // [T][16][PX], [2][T][N], [KS][NB2][kParts][64] of 16 bytes, [9][N]
  __host__ __device__ explicit constexpr SecondLds(int t)
      : map(0), halo(16 * t * PX), filter(halo + 2 * t * N), taps(filter + KS * NB2 * kParts * 64 * 4), end(taps + 9 * N) {}
};

// Filters: PackList (TWO only: the passes that have some), for workgroups behind the strips' ones to put in order, or NoFilters.
struct NoFilters {};
template <int Q, bool TWO, typename Filters>
__global__ __launch_bounds__(512, 2) void stem_block_rows_kernel(RowsArgs g, Filters filters) {
  using L2 = SecondLds<Q>;
  __shared__ __align__(16) float dw2_bias[TWO ? L2::N : 4], pw2_bias[TWO ? L2::N2 : 4];
  __shared__ int odd_filter2;  // bit 0: bits lost, bit 1: a large value
  constexpr int C = 8 * Q, N = 16 * Q, NB = Q, G = (C + 15) / 16, PX = 4 * rows_pixel_pieces<Q, TWO>();
  extern __shared__ __align__(16) float ring[];  // [4][16 T + 2][PX]: stem row r in slot r % 4, column c at c + 1
  if constexpr (std::is_same_v<Filters, PackList>)
    if ((int)blockIdx.x >= g.strip_groups) return pack_filters<5>(filters, (int)blockIdx.x - g.strip_groups, ring);
  // what a step reads once or twice stays in LDS
  __shared__ __align__(16) float stem_w[7][64][G], stem_bias[16 * G], dw_bias[16 * G], pw_bias[N];
  const int lane = threadIdx.x % 64, li = lane % 16, q = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int cols = (int)blockDim.x / 4 + 2, slot = cols * PX;
  // rows [r0, r1) of the first block's output, under rows [i0, i1) of the second's
  const int n = blockIdx.x / g.strips, i0 = (blockIdx.x - n * g.strips) * g.rows, i1 = min(i0 + g.rows, TWO ? g.OH2 : g.OH);
  const int r0 = TWO ? max(2 * i0 - g.pt2, 0) : i0, r1 = TWO ? min(2 * i1 + 1 - g.pt2, g.OH) : i1;
  const int ow = 16 * wave + li;

  // Byte offsets of this lane's stem operands in the image's row 0: three pairs and a single value.  What lies outside the
  // image's columns has an offset past the end of the buffer, from where loads return 0.  (SAME padding of a 3-wide filter at
  // stride 2 leaves at most one column of a window outside.)
  constexpr unsigned kNone = 0x80000000u;
  const int iw0 = 2 * ow - g.pl, row_bytes = 12 * g.IW;
  const bool left = iw0 < 0, right = iw0 + 2 >= g.IW, in = ow < g.OW;
  unsigned at[4];
  if (q < 3) {
    const unsigned base = (unsigned)(q * row_bytes + 12 * iw0);
    at[0] = in && !left ? base : kNone;
    at[1] = in ? base + (left ? 12 : 8) : kNone;  // (left: value 3 comes first)
    at[2] = in ? base + 16 : kNone;
    at[3] = in && !right ? base + 24 : kNone;
  } else {
#pragma unroll
    for (int t = 0; t < 3; ++t) at[t] = in && !right ? (unsigned)(t * row_bytes + 12 * iw0 + 28) : kNone;
    at[3] = kNone;
  }
  const unsigned start = (unsigned)n * g.image_bytes;
  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.x) + start / 4, 0, (int)(g.x_bytes - start), 0x00020000);
  const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(g.y, 0, (int)g.y_bytes, 0x00020000);

  // Pointwise filter, split (split.h): block j has output channels 16 j + li, k slot (q, e) channel 16 (e / 4) + 4 q + e % 4, as
  // the depthwise layer's result comes.
  bf16x8 pw[NB][kParts];
  SplitGuard filter;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    splitx4 part[2][kParts] = {};
#pragma unroll
    for (int u = 0; u < G; ++u) {
      floatx4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = 16 * u + 4 * q + e;
        v[e] = g.pw_w[(k < C ? k : 0) * N + 16 * j + li];
        if (k >= C) v[e] = 0.f;
        filter.most = fabsf(v[e]) < 0x1p20f ? filter.most : INFINITY;  // (NaN too)
      }
      filter.split(v, part[u]);
    }
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
      const u32x4 both = {part[0][p][0], part[0][p][1], part[1][p][0], part[1][p][1]};
      pw[j][p] = __builtin_bit_cast(bf16x8, both);
    }
  }
  const bool filter_large = __builtin_amdgcn_ballot_w64(filter.large()) != 0, filter_lost = __builtin_amdgcn_ballot_w64(filter.lost()) != 0;
  for (int i = threadIdx.x; i < 7 * 64 * G; i += (int)blockDim.x) {
    const int j = i % G, l = i / G % 64, s = i / G / 64;
    const int row = l / 16 < 3 ? 9 * (l / 16) + s : 9 * (s / 2) + 7 + s % 2, ch = 16 * j + l % 16;
    stem_w[s][l][j] = ch < C && (l / 16 < 3 || s < 6) ? g.st_w[row * C + ch] : 0.f;
  }
  // (TWO, for registers: in LDS)
  constexpr bool kTapsInLds = TWO && Q >= 3;
  __shared__ __align__(16) float dw_taps[kTapsInLds ? 9 : 1][16 * G];
  floatx4 dww[kTapsInLds ? 1 : 9][G];
  if constexpr (kTapsInLds) {
    for (int i = threadIdx.x; i < 9 * 16 * G; i += (int)blockDim.x) {
      const int k = i % (16 * G);
      dw_taps[i / (16 * G)][k] = k < C ? g.dw_w[i / (16 * G) * C + k] : 0.f;
    }
  } else {
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int u = 0; u < G; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = 16 * u + 4 * q + e;
          const float v = g.dw_w[t * C + (k < C ? k : 0)];
          dww[kTapsInLds ? 0 : t][u][e] = k < C ? v : 0.f;
        }
  }
  for (int i = threadIdx.x; i < 16 * G; i += (int)blockDim.x) {
    stem_bias[i] = i < C ? g.st_b[i] : 0.f;
    dw_bias[i] = i < C ? g.dw_b[i] : 0.f;
  }
  for (int i = threadIdx.x; i < N; i += (int)blockDim.x) pw_bias[i] = g.pw_b[i];
  for (int i = threadIdx.x; i < 4 * 2 * 4 * G; i += (int)blockDim.x) {  // zeros left and right of the map
    const int s = i / (8 * G), side = i / (4 * G) % 2, piece = i % (4 * G);
    *reinterpret_cast<floatx4*>(ring + s * slot + (side ? cols - 1 : 0) * PX + 4 * piece) = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  // ---- the second block: depthwise 3x3, stride 2, and the pointwise layer ----
  // Lane (li, q) has column 8 wave + li % 8 of its rows, depthwise channels ch2 ... + 3 and ch2 + 16 ... + 19.
  const L2 at2((int)blockDim.x / 64);
  float* const second = ring + 4 * slot;
  float* const map = second + at2.map + wave * 16 * L2::PX;  // this wavefront's 16 columns of the first block's row
  const int ch2 = 4 * q + (Q > 2 && li >= 8 ? 32 : 0);
  const bool have2[2] = {ch2 < N, ch2 + 16 < N};
  int at_map[3];  // where the three columns under the filter are; one of the 17 comes from the wavefront beside, and lies in `halo`
  int halo_step = 0;
  floatx4 acc2[2] = {}, first_row[2] = {};
  const bool beside_left = TWO && g.pl2 != 0;  // which of the three columns that is
  if constexpr (TWO) {
    const int waves = (int)blockDim.x / 64;
    if (threadIdx.x == 0) odd_filter2 = 0;
    __syncthreads();
    SplitGuard guard;
    for (int i = threadIdx.x; i < L2::KS * L2::NB2 * 64; i += (int)blockDim.x) {
      const int l = i % 64, j = i / 64 % L2::NB2, ks = i / 64 / L2::NB2;
      splitx4 part[2][kParts];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        floatx4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = 32 * ks + 16 * u + 4 * (l / 16) + e;
          const float w = g.pw2_w[(k < N ? k : 0) * L2::N2 + 16 * j + l % 16];
          v[e] = k < N ? w : 0.f;
          guard.most = fabsf(v[e]) < 0x1p20f ? guard.most : INFINITY;  // (NaN too)
        }
        guard.split(v, part[u]);
      }
#pragma unroll
      for (int p = 0; p < kParts; ++p)
        *reinterpret_cast<u32x4*>(second + at2.filter + 4 * ((((ks * L2::NB2 + j) * kParts) + p) * 64 + l)) =
            u32x4{part[0][p][0], part[0][p][1], part[1][p][0], part[1][p][1]};
    }
    if (guard.lost() || guard.large()) atomicOr(&odd_filter2, (guard.lost() ? 1 : 0) | (guard.large() ? 2 : 0));
    for (int i = threadIdx.x; i < 9 * N; i += (int)blockDim.x) second[at2.taps + i] = g.dw2_w[i];
    for (int i = threadIdx.x; i < 2 * waves * N; i += (int)blockDim.x) second[at2.halo + i] = 0.f;
    for (int i = threadIdx.x; i < N; i += (int)blockDim.x) dw2_bias[i] = g.dw2_b[i];
    for (int i = threadIdx.x; i < L2::N2; i += (int)blockDim.x) pw2_bias[i] = g.pw2_b[i];
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) {
      const int c = 2 * (li % 8) - g.pl2 + kw;
      const bool beside = c < 0 || c > 15;
      at_map[kw] = beside ? at2.halo + wave * N : at2.map + (wave * 16 + c) * L2::PX;
      if (beside) halo_step = waves * N;
    }
  }
  bool filter2_large = false, filter2_lost = false;
  auto channel = [&](int u) __attribute__((always_inline)) { return have2[u] ? ch2 + 16 * u : 0; };
  auto start_row = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2; ++u) acc2[u] = *reinterpret_cast<const floatx4*>(dw2_bias + channel(u));
  };
  // row i of the second block's depthwise layer is complete: rows are multiplied two at a time
  auto finish_row = [&](int i) __attribute__((always_inline)) {
    floatx4 row[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      row[u] = relu6(acc2[u]);
      if (!have2[u]) row[u] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const bool odd = ((i - i0) & 1) != 0;
    if (!odd) first_row[0] = row[0], first_row[1] = row[1];
    if (!odd && i + 1 < i1) return;
    floatx4 b[L2::KS][2];  // lanes li < 8: pixels of the first row, the others: of the second
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float low = first_row[u][e], high = odd ? row[u][e] : 0.f, low_moved = swap8(low), high_moved = swap8(high);
        b[0][u][e] = li < 8 ? low : high_moved;
        if constexpr (L2::KS == 2) b[L2::KS - 1][u][e] = li < 8 ? low_moved : high;
      }
    bf16x8 a[L2::KS][kParts];
    unsigned lost = 0;
#pragma unroll
    for (int ks = 0; ks < L2::KS; ++ks) {
      splitx4 part[2][kParts];
#pragma unroll
      for (int u = 0; u < 2; ++u) split4(b[ks][u], part[u], lost);
#pragma unroll
      for (int p = 0; p < kParts; ++p) {
        const u32x4 both = {part[0][p][0], part[0][p][1], part[1][p][0], part[1][p][1]};
        a[ks][p] = __builtin_bit_cast(bf16x8, both);
      }
    }
    const bool again = filter2_large || filter2_lost || __builtin_amdgcn_ballot_w64((lost & 0xffffu) != 0) != 0;
    const float limit = filter2_large ? INFINITY : small_limit(N);
    const int col = 8 * wave + li % 8, line = i - (odd ? 1 : 0) + li / 8;
    const unsigned to = col < g.OW2 && line <= i ? 4u * ((unsigned)((n * g.OH2 + line) * g.OW2 + col) * L2::N2) : kNone;
    const float* const filter = second + at2.filter + 4 * lane;
#pragma unroll
    for (int j = 0; j < L2::NB2; ++j) {
      floatx4 out = *reinterpret_cast<const floatx4*>(pw2_bias + 16 * j + 4 * q);
      bf16x8 w[L2::KS][kParts];
#pragma unroll
      for (int ks = 0; ks < L2::KS; ++ks)
#pragma unroll
        for (int p = 0; p < kParts; ++p)
          w[ks][p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(filter + (((ks * L2::NB2 + j) * kParts) + p) * 256));
      // (smallest products first, of both halves of the contraction)
#pragma unroll
      for (int s = 0; s < kSplitPasses; ++s)
#pragma unroll
        for (int ks = 0; ks < L2::KS; ++ks)
          out = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][split_pass_b(s)], a[ks][split_pass_a(s)], out, 0, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, relu6(out)), yr, to + 64 * j + 16 * q, 0, 0);
      if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    if (!again) return;
    // small results (with a large filter: all) again with the fp32 instructions, over the first ones
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.pw2_w), 0, 4 * N * L2::N2, 0x00020000);
#pragma unroll 1
    for (int j = 0; j < L2::NB2; ++j) {
      floatx4 exact = *reinterpret_cast<const floatx4*>(pw2_bias + 16 * j + 4 * q);
#pragma unroll
      for (int ks = 0; ks < L2::KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (32 * ks + 16 * (e / 4) < N)
            exact = __builtin_amdgcn_mfma_f32_16x16x4f32(
                __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wr, 4 * (4 * q * L2::N2 + 16 * j + li), 4 * (32 * ks + 16 * (e / 4) + e % 4) * L2::N2, 0)),
                b[ks][e / 4][e % 4], exact, 0, 0, 0);
      const floatx4 o = relu6(exact);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[e]), yr, filter2_large || fabsf(exact[e]) < limit ? (int)(to + 64 * j + 16 * q + 4 * e) : (int)kNone, 0, 0);
    }
  };
  auto second_depthwise = [&](int r) __attribute__((always_inline)) {  // what row r of the first block's output adds
    const int t = r + g.pt2, parity = (r & 1) * halo_step;
    floatx4 v[3][2];
#pragma unroll
    for (int kw = 0; kw < 3; ++kw)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        v[kw][u] = *reinterpret_cast<const floatx4*>(second + at_map[kw] + (kw == 0 ? (beside_left ? parity : 0) : kw == 2 ? (beside_left ? 0 : parity) : 0) + channel(u));
    auto add = [&](int kh) __attribute__((always_inline)) {
#pragma unroll
      for (int kw = 0; kw < 3; ++kw)
#pragma unroll
        for (int u = 0; u < 2; ++u)
          acc2[u] += v[kw][u] * *reinterpret_cast<const floatx4*>(second + at2.taps + (3 * kh + kw) * N + channel(u));
    };
    if (t & 1) {
      add(1);
    } else {
      if (t / 2 > i0) {
        add(2);
        finish_row(t / 2 - 1);
      }
      start_row();
      add(0);
    }
  };
  // the first block's output at this lane's column of row r, channels ch ... + 3: for the wavefront itself and, of its first or
  // last column, for the one beside
  auto put = [&](int r, int ch, const floatx4& v) __attribute__((always_inline)) {
    *reinterpret_cast<floatx4*>(map + li * L2::PX + ch) = v;
    const int to = beside_left ? wave + 1 : wave - 1;
    if (li == (beside_left ? 15 : 0) && to >= 0 && to < (int)blockDim.x / 64)
      *reinterpret_cast<floatx4*>(second + at2.halo + (r & 1) * ((int)blockDim.x / 64) * N + to * N + ch) = v;
  };

  struct Window {
    u32x2 pair[3];
    unsigned single;
  };
  auto fetch = [&](int r, Window& w) __attribute__((always_inline)) {  // of stem row r; image rows outside: anything
    const unsigned row = (unsigned)((2 * r - g.pt) * row_bytes);
#pragma unroll
    for (int t = 0; t < 3; ++t) w.pair[t] = __builtin_amdgcn_raw_buffer_load_b64(xr, at[t] + row, 0, 0);
    w.single = __builtin_amdgcn_raw_buffer_load_b32(xr, at[3] + row, 0, 0);
  };
  auto stem = [&](int r, const Window& w) __attribute__((always_inline)) {
    float* const to = ring + (r & 3) * slot + (ow + 1) * PX + 4 * q;
    if (r < 0 || r >= g.OH) {
#pragma unroll
      for (int j = 0; j < G; ++j) *reinterpret_cast<floatx4*>(to + 16 * j) = floatx4{0.f, 0.f, 0.f, 0.f};
      return;
    }
    unsigned v[7] = {w.pair[0][0], w.pair[0][1], w.pair[1][0], w.pair[1][1], w.pair[2][0], w.pair[2][1], w.single};
    if (wave == 0 && g.pl > 0) {
      v[3] = left && q < 3 ? v[2] : v[3];
      v[2] = left && q < 3 ? 0u : v[2];
    }
    const int ih0 = 2 * r - g.pt;
    if (ih0 < 0 || ih0 + 3 > g.IH) {  // a row outside the image
#pragma unroll
      for (int s = 0; s < 7; ++s) {
        const int ih = ih0 + (q < 3 ? q : s / 2);
        v[s] = ih >= 0 && ih < g.IH ? v[s] : 0u;
      }
    }
    floatx4 acc[G];
#pragma unroll
    for (int j = 0; j < G; ++j) acc[j] = *reinterpret_cast<const floatx4*>(stem_bias + 16 * j + 4 * q);
#pragma unroll
    for (int s = 0; s < 7; ++s)
#pragma unroll
      for (int j = 0; j < G; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(stem_w[s][lane][j], __uint_as_float(v[s]), acc[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < G; ++j) {
      floatx4 o = relu6(acc[j]);
      if (!in || 16 * j + 4 * q >= C) o = floatx4{0.f, 0.f, 0.f, 0.f};  // (no such channel: not 0 x Inf)
      *reinterpret_cast<floatx4*>(to + 16 * j) = o;
    }
  };

  // Loads and stores are counted in one order: the window of the next step is requested before this step's stores, so that
  // waiting for it waits for no store but those of the step before.
  Window w[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) fetch(r0 - 1 + i, w[i]);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) stem(r0 - 1 + i, w[i]);
  Window& next = w[0];
  if (r0 + 1 < r1) fetch(r0 + 2, next);
  __syncthreads();
  if constexpr (TWO) {
    filter2_lost = (odd_filter2 & 1) != 0, filter2_large = (odd_filter2 & 2) != 0;
    start_row();
  }
  unsigned out = in ? 4u * ((unsigned)((n * g.OH + r0) * g.OW + ow) * N) : kNone;  // past the end: not stored
  for (int r = r0; r < r1; ++r, out += 4u * g.OW * N) {
    if (r + 1 < r1) stem(r + 2, next);
    if (r + 2 < r1) fetch(r + 3, next);
    if constexpr (TWO) {
      __builtin_amdgcn_sched_barrier(0);
      if (r > r0) second_depthwise(r - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    floatx4 d[G];
#pragma unroll
    for (int u = 0; u < G; ++u) d[u] = *reinterpret_cast<const floatx4*>(dw_bias + 16 * u + 4 * q);
#pragma unroll
    for (int kh = 0; kh < 3; ++kh) {
      const float* const row = ring + ((r + kh + 3) & 3) * slot + ow * PX + 4 * q;
#pragma unroll
      for (int kw = 0; kw < 3; ++kw)
#pragma unroll
        for (int u = 0; u < G; ++u)
          d[u] += *reinterpret_cast<const floatx4*>(row + kw * PX + 16 * u) *
                  (kTapsInLds ? *reinterpret_cast<const floatx4*>(dw_taps[kTapsInLds ? 3 * kh + kw : 0] + 16 * u + 4 * q) : dww[kTapsInLds ? 0 : 3 * kh + kw][u]);
      __builtin_amdgcn_sched_barrier(0);  // three taps at a time in registers
    }
#pragma unroll
    for (int u = 0; u < G; ++u) d[u] = relu6(d[u]);
    // A depthwise output is at most 6 or NaN, which stays one: with a filter below 2^20 no product overflows, and only bits lost
    // to tiny values are looked for.
    bf16x8 a[kParts];
    unsigned low = 0;
    {
      splitx4 part[2][kParts] = {};
#pragma unroll
      for (int u = 0; u < G; ++u) split4(d[u], part[u], low);
#pragma unroll
      for (int p = 0; p < kParts; ++p) {
        const u32x4 both = {part[0][p][0], part[0][p][1], part[1][p][0], part[1][p][1]};
        a[p] = __builtin_bit_cast(bf16x8, both);
      }
    }
    floatx4 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = *reinterpret_cast<const floatx4*>(pw_bias + 16 * j + 4 * q);
#pragma unroll
    for (int s = 0; s < kSplitPasses; ++s)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pw[j][split_pass_b(s)], a[split_pass_a(s)], acc[j], 0, 0, 0);
    if (filter_large || filter_lost || __builtin_amdgcn_ballot_w64((low & 0xffffu) != 0) != 0) {
      // small results (with a large filter: all) again with the fp32 instructions
      const float limit = filter_large ? INFINITY : small_limit(C);
      bool any = filter_large;
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) any = any || fabsf(acc[j][e]) < limit;
      if (__builtin_amdgcn_ballot_w64(any) != 0) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          floatx4 exact = *reinterpret_cast<const floatx4*>(pw_bias + 16 * j + 4 * q);
#pragma unroll
          for (int s = 0; s < 4 * G; ++s) {
            const int k = 16 * (s / 4) + 4 * q + s % 4;
            const float v = g.pw_w[(k < C ? k : 0) * N + 16 * j + li];
            exact = __builtin_amdgcn_mfma_f32_16x16x4f32(k < C ? v : 0.f, d[s / 4][s % 4], exact, 0, 0, 0);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[j][e] = filter_large || fabsf(acc[j][e]) < limit ? exact[e] : acc[j][e];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const floatx4 o = relu6(acc[j]);
      if constexpr (TWO) put(r, 16 * j + 4 * q, in ? o : floatx4{0.f, 0.f, 0.f, 0.f});
      else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), yr, out + 64 * j + 16 * q, 0, 0);
    }
    __syncthreads();
  }
  if constexpr (TWO) {
    second_depthwise(r1 - 1);
    if (((r1 - 1 + g.pt2) & 1) != 0) finish_row(i1 - 1);  // (its last row lies outside the map)
  }
}

__global__ __launch_bounds__(1024) void pack_filters_kernel(PackList filters) {
  __shared__ float scratch[kPackScratch / sizeof(float)];
  pack_filters<2, 16>(filters, (int)blockIdx.x, scratch);
}

constexpr int kRowsMaxWidth = 128;  // columns of the map: 8 wavefronts of 16

template <int Q, bool TWO>
constexpr size_t rows_lds_bytes(int tiles) {
  return (size_t)4 * (4 * (16 * tiles + 2) * 4 * rows_pixel_pieces<Q, TWO>() + (TWO ? SecondLds<Q>(tiles).end : 0));
}
constexpr int kStaticLds = 7 * 1024;  // bytes beside, at most
// (what all call with: the narrower maps of the second block, whose filter takes LDS, and the widest one)
template <int Q, bool TWO>
constexpr int rows_max_tiles() {
  int t = kRowsMaxWidth / 16;
  while (rows_lds_bytes<Q, TWO>(t) + kStaticLds > 160 * 1024) --t;
  return t;
}

template <int Q, bool TWO, typename Filters>
int launch_rows_kernel(const RowsArgs& g, int groups, const Filters& filters, hipStream_t stream) {
  auto kern = stem_block_rows_kernel<Q, TWO, Filters>;
  const int tiles = (g.OW + 15) / 16;
  // The kernel is allowed once what its widest rows need: a later call may be wider than the first.
  static std::atomic<uint64_t> lds_allowed{0};
  constexpr size_t most = rows_lds_bytes<Q, TWO>(rows_max_tiles<Q, TWO>());
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), most, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  static_assert(!TWO || rows_lds_bytes<Q, TWO>(1) >= kPackScratch, "room to order the filters");
  hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(64u * tiles), (rows_lds_bytes<Q, TWO>(tiles)), stream, g, filters);
  return check_launch();
}

// filters: null, or what workgroups of this launch put in order
template <int Q>
int launch_rows(const RowsArgs& g, bool two, const PackList* filters, hipStream_t stream) {
  if (!two) return launch_rows_kernel<Q, false>(g, g.strip_groups, NoFilters(), stream);
  if (filters == nullptr) return launch_rows_kernel<Q, true>(g, g.strip_groups, NoFilters(), stream);
  return launch_rows_kernel<Q, true>(g, g.strip_groups + filters->groups(), *filters, stream);
}

}  // namespace

bool stem_two_blocks_supported(int ow, int q) {
  const int most[4] = {rows_max_tiles<1, true>(), rows_max_tiles<2, true>(), rows_max_tiles<3, true>(), rows_max_tiles<4, true>()};
  return q >= 1 && q <= 4 && (ow + 15) / 16 <= most[q - 1];
}

int launch_stem_block_rows(const float* image, const float* st_w, const float* st_b, const float* dw_w, const float* dw_b, const float* pw_w,
                           const float* pw_b, float* y, int batch, int ih, int iw, int oh, int ow, int pt, int pl, int q,
                           hipStream_t stream, const SecondBlock<float>* second, const PackList& filters) {
  const int out_rows = second ? second->oh : oh;
  const long long in = (long long)ih * iw * 3, out = second ? (long long)second->oh * second->ow * 32 * q : (long long)oh * ow * 16 * q;  // floats of an image
  if (ow > kRowsMaxWidth || iw < 3 || ih < 3 || reinterpret_cast<uintptr_t>(y) % 16 != 0) return TFX_ERR_UNSUPPORTED;
  const int tiles = (ow + 15) / 16;
  int per_cu = (q <= 2 ? 16 : 8) / tiles > 0 ? (q <= 2 ? 16 : 8) / tiles : 1;
  if (second) {
    if (!stem_two_blocks_supported(ow, q)) return TFX_ERR_UNSUPPORTED;
    per_cu = 8 / tiles;
    const int fit = 160 * 1024 / (kStaticLds + (int)(q == 1 ? rows_lds_bytes<1, true>(tiles) : q == 2 ? rows_lds_bytes<2, true>(tiles)
                                                     : q == 3 ? rows_lds_bytes<3, true>(tiles) : rows_lds_bytes<4, true>(tiles)));
    if (fit < per_cu) per_cu = fit;
  }
  const int slots = 256 * per_cu;
  // byte offsets of a launch stay below 2^31
  const long long most = ((1ll << 29) - 1) / (in > out ? in : out);
  for (long long first = 0; first < batch; first += most) {
    const int images = (int)(batch - first < most ? batch - first : most);
    // Strips of an image: rounds of resident workgroups (their registers leave 8 wavefronts to a CU, of the narrow networks 16)
    // times their rows, and five more for the two rows computed twice and for start and end.  224 x 224, 2 images: 112 strips
    // 10.1 us, 56 11.5; 16: 16 24.6, 28 30.5, 8 36.1; 64: 4 74, 8 81, 16 90.
    int strips = 1;
    double best = 1e30;
    for (int s = 1; s <= out_rows; ++s) {
      const int rows = (out_rows + s - 1) / s;
      if ((out_rows + rows - 1) / rows != s) continue;
      const double cost = (double)(((long long)images * s + slots - 1) / slots) * (second ? 2 * rows + 7 : rows + 5);
      if (cost < best) best = cost, strips = s;
    }
    RowsArgs g{image + first * in, st_w, st_b, dw_w, dw_b, pw_w, pw_b, y + first * out, ih, iw, oh, ow, pt, pl, strips,
               (out_rows + strips - 1) / strips, (unsigned)(4 * in), (unsigned)(4 * images * in), (unsigned)(4 * images * out),
               nullptr, nullptr, nullptr, nullptr, 0, 0, 0, 0, images * strips};
    if (second) {
      g.dw2_w = second->dw_w, g.dw2_b = second->dw_b, g.pw2_w = second->pw_w, g.pw2_b = second->pw_b;
      g.OH2 = second->oh, g.OW2 = second->ow, g.pt2 = second->pt, g.pl2 = second->pl;
    }
    // The tile blocks' filters: workgroups of this launch where it leaves CUs idle, and with 7 wavefronts and more, which hold a column of
    // 1024 rows in one go; else a launch of its own.  us a pass, so and in this launch: full width 224 x 224 4 images 150.6 / 146.2, 8 187.0 /
    // 186.3, 16 242.2 / 239.3, 192 x 192 12 images 200.1 / 192.7, 160 x 160 8 images 160.2 / 154.6.  Without idle CUs they come behind the
    // strips, one to a CU: 224 x 224 48 images 445 / 442, 64 517.5 / 516.5, 24 294 / 295, 32 325.5 / 326, 3/4 width 64 398.5 / 399, of which
    // 5 us and less are the difference of two runs; with fewer wavefronts 160 x 160 48 images 311 / 315, 96 x 96 64 images 242 / 249.
    const bool with = first == 0 && second && filters.groups() > 0 && (tiles >= 7 || images * strips <= slots / 8 * 7);
    const PackList* const list = with ? &filters : nullptr;
    int rc = TFX_ERR_UNSUPPORTED;
    if (q == 1) rc = launch_rows<1>(g, second != nullptr, list, stream);
    if (q == 2) rc = launch_rows<2>(g, second != nullptr, list, stream);
    if (q == 3) rc = launch_rows<3>(g, second != nullptr, list, stream);
    if (q == 4) rc = launch_rows<4>(g, second != nullptr, list, stream);
    if (rc) return rc;
    if (first == 0 && filters.groups() > 0 && !with) {
      hipLaunchKernelGGL(pack_filters_kernel, dim3((unsigned)filters.groups()), dim3(1024), 0, stream, filters);
      if (const int bad = check_launch()) return bad;
    }
  }
  return TFX_OK;
}

}  // namespace tfx
