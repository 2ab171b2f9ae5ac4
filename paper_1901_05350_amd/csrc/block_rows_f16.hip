// The stem (3x3 stride-2 convolution of the image to 8 Q channels) and the first depthwise-separable block (depthwise 3x3 +
// bias + clamp, pointwise 1x1 to 16 Q channels + bias + clamp) on binary16 storage in one launch (Section 4.1 storage format,
// the Section 3.9 network).
//
// The stem's output is the largest map but one of the network; written and read again it costs as much as the block's own
// output.  Here a workgroup walks down a strip of rows of one image, a wavefront for every 16 columns, and keeps the four stem
// rows that it works on in LDS: three under the depthwise filter and the one it computes for the next step, with one barrier
// a row.  Stem rows are rounded to binary16 as the separate kernel rounds them, and only the two rows above and below a strip
// are computed twice.
//
// Contraction of the stem (v_mfma_f32_16x16x32_f16, filters as the first operand): lane (li, q) supplies 8 values of pixel
// li's window, for q < 3 the first 8 of the 9 that lie next to each other in image row q of it -- one load of 16 bytes at
// whatever address --, for q = 3 the ninth of each row.
//
// The depthwise layer runs on the matrix cores too, as products with diagonal matrices: two taps x 16 channels are the 32 of a
// contraction, of which each channel's row of the filter operand has but its own two weights.  15/16 of the multiplications are
// with zero, and still ten such instructions (16 cycles each) replace 72 mixed-precision multiply-adds (4.4 cycles each,
// measured); the result comes as the pointwise product's operand.  A zero times a NaN is a NaN in 15 other channels, but all
// channels of the pixel meet in every output of the pointwise layer, so the same outputs are NaN; the map itself, behind a
// relu6, has no infinities.
//
// 64 images of 224 x 224, full width: 28 us (31 under the profiler), where the stem and the block's kernel took 52 (23 + 30); the
// image's and the output's 122 MB take 24 at the rate of a large copy.  With the depthwise layer on the vector units 33.  One
// image: 6.4 us, two launches 8.6.
//
// TWO: the second block too, whose depthwise layer walks down the rows at stride 2.  The first block's output, the largest map of the
// network, then never leaves the CU: a wavefront keeps its 16 columns of one row in LDS (the seventeenth comes from the wavefront
// beside), adds what the row gives to 8 columns of the second depthwise layer in registers, and multiplies the rows of that two at a
// time.  LDS bounds it (38 reads of 16 bytes a lane and row, 70 % of the cycles) beside the vector units; two workgroups of seven
// wavefronts need 128 registers a lane and 80 KB, so part of the filters is in LDS and part of the diagonal operands is made in each
// step; 1 register (3/4 width 7) that still does not fit is spilled.  64 images 46.8 us, the two launches 27 + 29; with all filters in
// registers and one workgroup on a CU 49.8, windows requested two steps ahead made no difference.
#include "ragged.h"
#include "stream_f16.h"

namespace tfx {
namespace {

using namespace f16s;

struct RowsArgs {
  const half_t *x, *st_w, *st_b, *dw_w, *dw_b, *pw_w, *pw_b;
  half_t* y;
  int IH, IW, OH, OW, pt, pl, strips, rows;  // rows of a strip, of the output
  long long image_halfs, total_halfs;  // of one image, of all
  unsigned y_bytes;
  // the second block, where it comes too
  const half_t *dw2_w, *dw2_b, *pw2_w, *pw2_b;
  int OH2, OW2, pt2, pl2;
  ChainClear clear;  // optional, by workgroups behind the first `strip_groups`
  int strip_groups;
};

struct RowsPixel {
  int pieces;
  constexpr int operator()(int li, int q) const { return li * pieces + q; }
};
template <int Q, bool TWO>
constexpr int rows_pixel_pieces() {
  if (TWO && Q == 4) return 5;  // (some conflicts; with 6 pieces a CU has room for one workgroup only)
  for (int p = Q;; ++p)
    if (conflict_free(RowsPixel{p})) return p;
}

// The second block's part of LDS, of T wavefronts, in halfs behind the ring.
template <int Q>
struct SecondLds {
  static constexpr int N = 16 * Q, N2 = 32 * Q, NB2 = 2 * Q, KS = (Q + 1) / 2, PX = 8 * (2 * Q + 1);
  int map, halo, filter, taps, end;  // [T][16][PX], [2][T][N], [KS][NB2][64][8], [9][N]
  __host__ __device__ explicit constexpr SecondLds(int t)
      : map(0), halo(16 * t * PX), filter(halo + 2 * t * N), taps(filter + KS * NB2 * 64 * 8), end(taps + 9 * N) {}
};

__device__ __forceinline__ h8 other_half(const h8& v) {  // of lane (li + 8) % 16
  u32x4 o = __builtin_bit_cast(u32x4, v);
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = (unsigned)__builtin_amdgcn_update_dpp(0, (int)o[i], 0x128, 0xf, 0xf, false);
  return __builtin_bit_cast(h8, o);
}

template <int Q, bool TWO>
__global__ __launch_bounds__(512, 4) void stem_block_rows_f16_kernel(RowsArgs g) {
  if ((int)blockIdx.x >= g.strip_groups)
    return clear_for_chain(g.clear, (blockIdx.x - g.strip_groups) * blockDim.x + threadIdx.x, (gridDim.x - g.strip_groups) * blockDim.x);
  constexpr int C = 8 * Q, N = 16 * Q, NB = Q, G = (C + 15) / 16, PX = 8 * rows_pixel_pieces<Q, TWO>();
  using L2 = SecondLds<Q>;
  extern __shared__ __align__(16) half_t ring[];  // [4][16 T + 2][PX]: stem row r in slot r % 4, column c at c + 1
  __shared__ __align__(16) float dw2_bias[TWO ? N : 4], pw2_bias[TWO ? L2::N2 : 4];
  // what a step reads once or twice stays in LDS: 128 registers for each of the 16 wavefronts of a CU
  __shared__ __align__(16) float stem_bias[16 * G], dw_bias[16 * G], pw_bias[N];
  __shared__ __align__(16) h8 stem_w[G][64];
  const int lane = threadIdx.x % 64, li = lane % 16, q = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int cols = (int)blockDim.x / 4 + 2, slot = cols * PX;
  // rows [r0, r1) of the first block's output, under rows [i0, i1) of the second's
  const int n = blockIdx.x / g.strips, i0 = (blockIdx.x - n * g.strips) * g.rows, i1 = min(i0 + g.rows, TWO ? g.OH2 : g.OH);
  const int r0 = TWO ? max(2 * i0 - g.pt2, 0) : i0, r1 = TWO ? min(2 * i1 + 1 - g.pt2, g.OH) : i1;
  const int ow = 16 * wave + li;

  // The stem's operand.  Byte offsets of this lane's values in the image's row 0, past the end of the buffer (from where loads
  // return 0) for a lane without any.
  constexpr unsigned kNone = 0x80000000u;
  const int iw0 = 2 * ow - g.pl, row_bytes = 6 * g.IW;
  const bool left = iw0 < 0;            // (by one column) loaded from the row's start and moved up by a pixel
  const int inside = 3 * (g.IW - iw0);  // values of a window row up to the image's end (9 or more: all)
  const unsigned at8 = q < 3 && ow < g.OW ? (unsigned)(6 * max(iw0, 0) + q * row_bytes) : kNone;
  const unsigned at9 = q == 3 && ow < g.OW && inside >= 9 ? (unsigned)(6 * iw0 + 16) : kNone;
  const bool edge = (wave == 0 && g.pl > 0) || 2 * (16 * wave + 15) - g.pl + 3 > g.IW;  // of the wavefront's columns
  const long long start = n * g.image_halfs;
  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(g.x + start), 0, (int)(2 * (g.total_halfs - start)), 0x00020000);
  const unsigned last = (unsigned)(2 * (g.total_halfs - start) - 16);  // offset at which 16 bytes can be loaded
  if (wave == 0) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      h8 sw;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int row = q < 3 ? 9 * q + t : 9 * (t < 3 ? t : 2) + 8, ch = 16 * j + li;
        const half_t v = g.st_w[row * C + (ch < C ? ch : 0)];
        sw[t] = ch < C && (q < 3 || t < 3) ? v : (half_t)0.f;
      }
      stem_w[j][lane] = sw;
    }
  }
  // The depthwise layer as a product with diagonal matrices: k = (tap, channel) of two taps and 16 channels, row = channel.
  // Lane (li, q) supplies tap 2 i + q / 2, channels 8 (q % 2) ... + 7 of the group to both operands; of the filter all but
  // channel li is zero.
  // (TWO, for registers: the last pair of taps lies in LDS, kMade of the others are one word a lane and made an operand in each step.)
  constexpr int kMade = TWO ? 3 : 0;
  constexpr int kKept = (TWO ? 4 : 5) - kMade;
  h8 dww[kKept][G];
  __shared__ __align__(16) h8 dw_lds[TWO ? G : 1][64];
  unsigned short dwv[5][G];
  unsigned dwm[kMade + 1][G];
  auto spread = [&](unsigned word) __attribute__((always_inline)) {
    u32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = li % 8 / 2 == e ? word : 0u;
    return __builtin_bit_cast(h8, v);
  };
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int t = min(2 * i + q / 2, 8), ch = 16 * u + li;
      dwv[i][u] = reinterpret_cast<const unsigned short*>(g.dw_w)[t * C + (ch < C ? ch : 0)];
    }
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const bool mine = li / 8 == q % 2 && 2 * i + q / 2 < 9 && 16 * u + li < C;
      const unsigned word = mine ? (unsigned)dwv[i][u] << 16 * (li % 2) : 0u;
      if (i < kKept) dww[i < kKept ? i : 0][u] = spread(word);
      else if (TWO && i == 4) dw_lds[TWO ? u : 0][lane] = spread(word);  // (every wavefront's are the same)
      else dwm[i < kKept || i == 4 ? 0 : i - kKept][u] = word;
    }
  // block j of the output's channels: pairs in rho order (16-byte stores), a last single one as it comes
  h8 pw[TWO ? 1 : NB];  // (TWO: in LDS, for registers)
  __shared__ __align__(16) h8 pw_lds[TWO ? NB : 1][64];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if (TWO && wave != j % ((int)blockDim.x / 64)) continue;
    h8 v;
    const int c = j + (j % 2 == 0) < NB ? 32 * (j / 2) + 8 * (li / 4) + 4 * (j % 2) + li % 4 : 16 * j + li;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 16 * (i / 4) + 4 * q + i % 4;  // as the depthwise layer's result comes
      const half_t w = g.pw_w[(k < C ? k : 0) * N + c];
      v[i] = k < C ? w : (half_t)0.f;
    }
    if constexpr (TWO) pw_lds[j][lane] = v;
    else pw[j] = v;
  }
  // the biases in the accumulators' order, and zeros left and right of the map
  for (int i = threadIdx.x; i < 16 * G; i += (int)blockDim.x) {
    stem_bias[i] = i < C ? (float)g.st_b[i] : 0.f;
    dw_bias[i] = i < C ? (float)g.dw_b[i] : 0.f;
  }
  for (int i = threadIdx.x; i < N; i += (int)blockDim.x) {
    const int j = i / 16, e = i % 16;
    pw_bias[i] = (float)g.pw_b[j + (j % 2 == 0) < NB ? 32 * (j / 2) + 8 * (e / 4) + 4 * (j % 2) + e % 4 : i];
  }
  for (int i = threadIdx.x; i < 4 * 2 * Q; i += (int)blockDim.x) {
    const int s = i / (2 * Q), side = i / Q % 2, piece = i % Q;
    *reinterpret_cast<u32x4*>(ring + s * slot + (side ? cols - 1 : 0) * PX + 8 * piece) = u32x4{0, 0, 0, 0};
  }
  const ActClamp clamp = make_act(TFX_ACT_RELU6);

  // ---- the second block: depthwise 3x3, stride 2, and the pointwise layer ----
  // Lane (li, q) has column 8 wave + li % 8 of its rows, depthwise channels 8 oct ... + 7.
  const L2 at2((int)blockDim.x / 64);
  half_t* const second = ring + 4 * slot;
  half_t* const map = second + at2.map + wave * 16 * L2::PX;  // this wavefront's 16 columns of the first block's row
  const int oct_of = q + (Q > 2 && li >= 8 ? 4 : 0), oct = oct_of < 2 * Q ? oct_of : 0;
  int at_map[3];  // where the three columns under the filter are; one of the 17 comes from the wavefront beside, and lies in `halo`
  int halo_step = 0;
  float acc2[8];
  h8 first_row = {0, 0, 0, 0, 0, 0, 0, 0};
  if constexpr (TWO) {
    const int waves = (int)blockDim.x / 64;
    for (int i = threadIdx.x; i < L2::KS * L2::NB2 * 64; i += (int)blockDim.x) {
      const int l = i % 64, j = i / 64 % L2::NB2, ks = i / 64 / L2::NB2;
      const int c = 32 * (j / 2) + 8 * (l % 16 / 4) + 4 * (j % 2) + l % 4;
      h8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 32 * ks + 8 * (l / 16) + e;
        const half_t w = g.pw2_w[(k < N ? k : 0) * L2::N2 + c];
        v[e] = k < N ? w : (half_t)0.f;
      }
      *reinterpret_cast<h8*>(second + at2.filter + 8 * i) = v;
    }
    for (int i = threadIdx.x; i < 9 * N; i += (int)blockDim.x) second[at2.taps + i] = g.dw2_w[i];
    for (int i = threadIdx.x; i < 2 * waves * N; i += (int)blockDim.x) second[at2.halo + i] = (half_t)0.f;
    for (int i = threadIdx.x; i < N; i += (int)blockDim.x) dw2_bias[i] = (float)g.dw2_b[i];
    for (int i = threadIdx.x; i < L2::N2; i += (int)blockDim.x) {
      const int j = i / 16, e = i % 16;
      pw2_bias[i] = (float)g.pw2_b[32 * (j / 2) + 8 * (e / 4) + 4 * (j % 2) + e % 4];
    }
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) {
      const int c = 2 * (li % 8) - g.pl2 + kw;
      const bool beside = c < 0 || c > 15;
      at_map[kw] = beside ? at2.halo + wave * N + 8 * oct : at2.map + (wave * 16 + c) * L2::PX + 8 * oct;
      if (beside) halo_step = waves * N;
    }
  }
  const bool beside_left = TWO && g.pl2 != 0;  // which of the three columns that is
  auto start_row = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) acc2[e] = dw2_bias[8 * oct + e];
  };
  // row i of the second block's depthwise layer is complete: rows are multiplied two at a time
  auto finish_row = [&](int i) __attribute__((always_inline)) {
    h8 row[1];
    const f32x4 v[2] = {{acc2[0], acc2[1], acc2[2], acc2[3]}, {acc2[4], acc2[5], acc2[6], acc2[7]}};
    activate_and_pack(v, clamp, row);
    const h8 none = {0, 0, 0, 0, 0, 0, 0, 0};
    if (oct_of >= 2 * Q) row[0] = none;
    const bool odd = ((i - i0) & 1) != 0;
    if (!odd) first_row = row[0];
    if (!odd && i + 1 < i1) return;
    const h8 low = first_row, high = odd ? row[0] : none;
    const h8 low_moved = other_half(low), high_moved = other_half(high);  // (by all lanes)
    h8 b[2];  // lanes li < 8: pixels of the first row, the others: of the second
    b[0] = li < 8 ? low : high_moved;
    b[1] = li < 8 ? low_moved : high;
    const int col = 8 * wave + li % 8, line = i - (odd ? 1 : 0) + li / 8;
    const unsigned to = col < g.OW2 && line <= i ? 2u * ((unsigned)((n * g.OH2 + line) * g.OW2 + col) * L2::N2) : kNone;
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(g.y, 0, (int)g.y_bytes, 0x00020000);
    const half_t* const filter = second + at2.filter + 8 * lane;
    constexpr int STEP = 2;
#pragma unroll
    for (int j0 = 0; j0 < L2::NB2; j0 += STEP) {
      f32x4 out[STEP];
      h8 o[STEP / 2];
#pragma unroll
      for (int j = 0; j < STEP; ++j) out[j] = *reinterpret_cast<const f32x4*>(pw2_bias + 16 * (j0 + j) + 4 * q);
#pragma unroll
      for (int ks = 0; ks < L2::KS; ++ks)
#pragma unroll
        for (int j = 0; j < STEP; ++j)
          out[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const h8*>(filter + (ks * L2::NB2 + j0 + j) * 512), b[ks], out[j], 0, 0, 0);
      activate_and_pack(out, clamp, o);
#pragma unroll
      for (int m = 0; m < STEP / 2; ++m)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o[m]), yr, to + 32 * j0 + 64 * m + 16 * q, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto second_depthwise = [&](int r) __attribute__((always_inline)) {  // what row r of the first block's output adds
    const int t = r + g.pt2, parity = (r & 1) * halo_step;
    h8 v[3];
    v[0] = *reinterpret_cast<const h8*>(second + at_map[0] + (beside_left ? parity : 0));
    v[1] = *reinterpret_cast<const h8*>(second + at_map[1]);
    v[2] = *reinterpret_cast<const h8*>(second + at_map[2] + (beside_left ? 0 : parity));
    auto add = [&](int kh) __attribute__((always_inline)) {
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const h8 w = *reinterpret_cast<const h8*>(second + at2.taps + (3 * kh + kw) * N + 8 * oct);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc2[e] = fmaf((float)v[kw][e], (float)w[e], acc2[e]);
      }
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

  auto operand = [&](int i, int u) __attribute__((always_inline)) {
    return i < kKept ? dww[i < kKept ? i : 0][u] : TWO && i == 4 ? dw_lds[TWO ? u : 0][lane] : spread(dwm[i < kKept || i == 4 ? 0 : i - kKept][u]);
  };

  struct Window {
    u32x4 v;
    unsigned short n[3];
  };
  auto fetch = [&](int r, Window& w) __attribute__((always_inline)) {  // of stem row r; image rows outside: anything
    const unsigned row = (unsigned)((2 * r - g.pt) * row_bytes);
    // 16 bytes from before the end of the last image where the window's 8 values would pass it (back in place in `stem`)
    const unsigned at = at8 + row;
    w.v = __builtin_amdgcn_raw_buffer_load_b128(xr, at8 != kNone && (int)at > (int)last ? last : at, 0, 0);
#pragma unroll
    for (int t = 0; t < 3; ++t) w.n[t] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(xr, at9 + row + t * row_bytes, 0, 0);
  };
  auto stem = [&](int r, const Window& w) __attribute__((always_inline)) {
    half_t* const to = ring + (r & 3) * slot + (ow + 1) * PX + 4 * q;
    if (r < 0 || r >= g.OH) {
#pragma unroll
      for (int j = 0; j < G; ++j)
        if (16 * j + 4 * q < C) *reinterpret_cast<h4*>(to + 16 * j) = h4{0, 0, 0, 0};
      return;
    }
    const int ih0 = 2 * r - g.pt;
    u32x4 v = w.v, ninth = {(unsigned)w.n[0] | (unsigned)w.n[1] << 16, w.n[2], 0, 0};
    if (edge) {
      const unsigned at = at8 + (unsigned)(ih0 * row_bytes);
      if (at8 != kNone && (int)at > (int)last) v = shift_down<half_t>(v, min((at - last) / 2, 8u));
      const u32x4 moved = {0, v[0] << 16, __builtin_amdgcn_alignbit(v[1], v[0], 16), __builtin_amdgcn_alignbit(v[2], v[1], 16)};
      v = left ? moved : v & first_elements<half_t>(inside);
    }
    if (ih0 < 0 || ih0 + 3 > g.IH) {  // a row outside the image
      if (ih0 + q < 0 || ih0 + q >= g.IH) v = u32x4{0, 0, 0, 0};
      if (ih0 < 0) ninth[0] &= 0xffff0000u;
      if (ih0 + 2 >= g.IH) ninth[1] = 0;
      if (ih0 + 1 >= g.IH) ninth[0] &= 0xffffu;
    }
    const h8 xv = __builtin_bit_cast(h8, q == 3 ? ninth : v);
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int j = 0; j < G; ++j)
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(stem_w[j][lane], xv, *reinterpret_cast<const f32x4*>(stem_bias + 16 * j + 4 * q), 0, 0, 0);
    h8 o[1];
    activate_and_pack(acc, clamp, o);
    if (ow >= g.OW) o[0] = h8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < G; ++j)
      if (16 * j + 4 * q < C) *reinterpret_cast<h4*>(to + 16 * j) = h4{o[0][4 * j], o[0][4 * j + 1], o[0][4 * j + 2], o[0][4 * j + 3]};
  };

  // the first block's output at this lane's column of row r, channels ch ...: for the wavefront itself and, of its first or last
  // column, for the one beside
  auto put = [&](int r, int ch, const auto& v) __attribute__((always_inline)) {
    typedef std::remove_cv_t<std::remove_reference_t<decltype(v)>> V;
    *reinterpret_cast<V*>(map + li * L2::PX + ch) = v;
    const int to = beside_left ? wave + 1 : wave - 1;
    if (li == (beside_left ? 15 : 0) && to >= 0 && to < (int)blockDim.x / 64)
      *reinterpret_cast<V*>(second + at2.halo + (r & 1) * ((int)blockDim.x / 64) * N + to * N + ch) = v;
  };

  // Loads and stores are counted in one order: the window of the next step is requested before this step's stores, so that
  // waiting for it waits for no store but those of the step before.
  Window w[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) fetch(r0 - 1 + i, w[i]);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    stem(r0 - 1 + i, w[i]);
    if constexpr (TWO) __builtin_amdgcn_sched_barrier(0);
  }
  Window& next = w[0];
  if (r0 + 1 < r1) fetch(r0 + 2, next);
  __syncthreads();
  if constexpr (TWO) start_row();
  const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(g.y, 0, (int)g.y_bytes, 0x00020000);
  unsigned out = ow < g.OW ? 2u * ((unsigned)((n * g.OH + r0) * g.OW + ow) * N) : kNone;  // past the end: not stored
  for (int r = r0; r < r1; ++r, out += 2u * g.OW * N) {
    if (r + 1 < r1) stem(r + 2, next);
    if (r + 2 < r1) fetch(r + 3, next);
    if constexpr (TWO) {
      __builtin_amdgcn_sched_barrier(0);  // (as everywhere here: one phase's values in registers at a time)
      if (r > r0) second_depthwise(r - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < kMade; ++i)
#pragma unroll
      for (int u = 0; u < G; ++u) asm volatile("" : "+v"(dwm[i][u]));  // (else they are made in front of the loop, and kept)
    f32x4 d[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int u = 0; u < G; ++u) d[u] = *reinterpret_cast<const f32x4*>(dw_bias + 16 * u + 4 * q);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      // taps 2 i and 2 i + 1 (of the ninth, whose partner has zeros: itself)
      const int t0 = 2 * i, t1 = i < 4 ? t0 + 1 : t0;
      const int at0 = ((r + t0 / 3 + 3) & 3) * slot + t0 % 3 * PX, at1 = ((r + t1 / 3 + 3) & 3) * slot + t1 % 3 * PX;
      const half_t* const tap = ring + (ow * PX + 8 * (q % 2)) + (q < 2 ? at0 : at1);
#pragma unroll
      for (int u = 0; u < G; ++u)
        d[u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(operand(i, u),
                                                      *reinterpret_cast<const h8*>(tap + (2 * u + 1 < Q ? 16 * u : 16 * u - 8 * (q % 2))), d[u], 0, 0, 0);
    }
    h8 a[1];
    activate_and_pack(d, clamp, a);
    if constexpr (TWO) __builtin_amdgcn_sched_barrier(0);
    f32x4 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(TWO ? pw_lds[TWO ? j : 0][lane] : pw[TWO ? 0 : j], a[0], *reinterpret_cast<const f32x4*>(pw_bias + 16 * j + 4 * q), 0, 0, 0);
    if constexpr (NB >= 2) {
      constexpr int PAIRS = NB / 2;
      f32x4 pairs[2 * PAIRS];
#pragma unroll
      for (int j = 0; j < 2 * PAIRS; ++j) pairs[j] = acc[j];
      h8 o[PAIRS];
      activate_and_pack(pairs, clamp, o);
#pragma unroll
      for (int m = 0; m < PAIRS; ++m) {
        if constexpr (TWO) put(r, 32 * m + 8 * q, ow < g.OW ? o[m] : h8{0, 0, 0, 0, 0, 0, 0, 0});
        else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o[m]), yr, out + 64 * m + 16 * q, 0, 0);
      }
    }
    if constexpr (NB % 2 == 1) {
      typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
      h4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (half_t)apply_act(acc[NB - 1][e], clamp);
      if constexpr (TWO) put(r, 16 * (NB - 1) + 4 * q, ow < g.OW ? o : h4{0, 0, 0, 0});
      else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, o), yr, out + 32 * (NB - 1) + 8 * q, 0, 0);
    }
    __syncthreads();
  }
  if constexpr (TWO) {
    second_depthwise(r1 - 1);
    if (((r1 - 1 + g.pt2) & 1) != 0) finish_row(i1 - 1);  // (its last row lies outside the map)
  }
}

// (the largest: 128 columns of full width)
template <int Q, bool TWO>
constexpr size_t rows_lds_bytes(int tiles) {
  return ((size_t)4 * (16 * tiles + 2) * 8 * rows_pixel_pieces<Q, TWO>() + (TWO ? SecondLds<Q>(tiles).end : 0)) * sizeof(half_t);
}
template <int Q, bool TWO>
int launch_rows(const RowsArgs& args, hipStream_t stream) {
  const int tiles = (args.OW + 15) / 16;
  auto kern = stem_block_rows_f16_kernel<Q, TWO>;
  static std::atomic<uint64_t> lds_allowed{0};
  if (TWO && allow_dynamic_lds(reinterpret_cast<const void*>(kern), rows_lds_bytes<Q, TWO>(8), lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  const unsigned clearing = (args.clear.fill_pieces / 4 + (unsigned)args.clear.zero_count + 64 * tiles - 1) / (64 * tiles);
  hipLaunchKernelGGL(kern, dim3((unsigned)args.strip_groups + clearing), dim3(64u * tiles), (rows_lds_bytes<Q, TWO>(tiles)), stream, args);
  return check_launch();
}

}  // namespace

int launch_stem_block_rows_f16(const uint16_t* image, const uint16_t* st_w, const uint16_t* st_b, const uint16_t* dw_w,
                               const uint16_t* dw_b, const uint16_t* pw_w, const uint16_t* pw_b, uint16_t* y, int batch, int ih, int iw,
                               int oh, int ow, int pt, int pl, int q, hipStream_t stream, const SecondBlock<uint16_t>* second, const ChainClear& clear) {
  auto p = [](const uint16_t* v) { return reinterpret_cast<const half_t*>(v); };
  const int out_rows = second ? second->oh : oh;
  const long long in = (long long)ih * iw * 3, out = second ? (long long)second->oh * second->ow * 32 * q : (long long)oh * ow * 16 * q;  // halfs of an image
  if (ow > 128 || iw < 3 || ih < 3 || reinterpret_cast<uintptr_t>(y) % 16 != 0) return TFX_ERR_UNSUPPORTED;
  const int tiles = (ow + 15) / 16;
  int per_cu = 16 / tiles;
  if (second) {
    constexpr int kStatic = 9472;  // bytes of LDS beside the dynamic ones
    const int fit = 163840 / (kStatic + (int)(q == 3 ? rows_lds_bytes<3, true>(tiles) : rows_lds_bytes<4, true>(tiles)));
    if (fit < per_cu) per_cu = fit;
  }
  const int slots = 256 * per_cu;
  // byte offsets of a launch stay below 2^31
  const long long most = ((1ll << 30) - 1) / (in > out ? in : out);
  for (long long first = 0; first < batch; first += most) {
    const int images = (int)(batch - first < most ? batch - first : most);
    // Strips of an image: rounds of resident workgroups (16 wavefronts a CU) times their rows, and five more for the two rows
    // computed twice and for start and end.  224 x 224, one image: 112 strips 6.4 us, 56 7.5; 8: 28 or 56 11.4, 16 14.1; 16: 28 or
    // 16 15.7, 56 19.0; 64: 8 31.1, 16 34.7, 4 37.7.  (With the second block: twice its rows, and one.)
    int strips = 1;
    double best = 1e30;
    for (int s = 1; s <= out_rows; ++s) {
      const int rows = (out_rows + s - 1) / s;
      if ((out_rows + rows - 1) / rows != s) continue;
      const double cost = (double)(((long long)images * s + slots - 1) / slots) * (second ? 2 * rows + 7 : rows + 5);
      if (cost < best) best = cost, strips = s;
    }
    RowsArgs g{p(image) + first * in, p(st_w), p(st_b), p(dw_w), p(dw_b), p(pw_w), p(pw_b), reinterpret_cast<half_t*>(y) + first * out,
               ih, iw, oh, ow, pt, pl, strips, (out_rows + strips - 1) / strips, in, images * in, (unsigned)(2 * images * out),
               nullptr, nullptr, nullptr, nullptr, 0, 0, 0, 0, first == 0 ? clear : ChainClear(), images * strips};
    if (second) {
      g.dw2_w = p(second->dw_w), g.dw2_b = p(second->dw_b), g.pw2_w = p(second->pw_w), g.pw2_b = p(second->pw_b);
      g.OH2 = second->oh, g.OW2 = second->ow, g.pt2 = second->pt, g.pl2 = second->pl;
    }
    int rc = TFX_ERR_UNSUPPORTED;
    if (q == 1 && !second) rc = launch_rows<1, false>(g, stream);
    if (q == 2 && !second) rc = launch_rows<2, false>(g, stream);
    if (q == 3) rc = second ? launch_rows<3, true>(g, stream) : launch_rows<3, false>(g, stream);
    if (q == 4) rc = second ? launch_rows<4, true>(g, stream) : launch_rows<4, false>(g, stream);
    if (rc) return rc;
  }
  return TFX_OK;
}

}  // namespace tfx
