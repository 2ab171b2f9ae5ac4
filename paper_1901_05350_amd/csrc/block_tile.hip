// A depthwise-separable block (depthwise 3x3 + bias + relu6, pointwise 1x1 + bias + clamp, fp32) in one launch, for the layers
// whose pointwise filter does not fit a workgroup's LDS: the fp32 form of block_tile_f16.hip.
//
// The pointwise layer is a product on the binary16 matrix cores with operands split in two (pair.h).  A workgroup owns a tile of 32 TM
// output pixels, as patches of 4 x 2, and 64 columns for each of its groups of wavefronts; all its threads compute the depthwise
// output of the tile into LDS, split, and each wavefront multiplies the tile by its 64 columns of the filter, whose operands it loads
// straight from L2 in the order of pack_filters (pack.h).
//
// 64 x 14 x 14 x 512 -> 512, one layer: 33.6 us, of which 5.4 are the start and the launch, 9.5 the depthwise layer, 14.3 the contraction
// (a megabyte of the filter for each CU through the path from L2, 73 GB/s to each; the matrix cores would take 8), 4.4 the stores; the
// depthwise kernel and the product of bf16 parts that stood here took 66.  64 x 28 x 28 x 256 -> 256 83 -> 45, 256 -> 512 at stride 2
// 45 -> 27, 7 x 7 x 1024 -> 1024 64 -> 39; the pass of 64 images 760 -> 565, of 16 271 -> 246, of 8 203 -> 189.
//
// 96 channels, an odd number of k-step pairs, take two blocks of 32 pixels (96 -> 192 of the 3/4 width: 20 images 28.1 us as two launches,
// 13.0 so).
//
// Results that the split does not carry (pair.h) are computed again over the first ones, unless the pixel's depthwise output is NaN.
#include "pair.h"

namespace tfx {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kXcds = 8;

struct TileArgs {
  const float *x, *dw_w, *dw_b, *pw_w, *pw_b;
  const half_t* packed;
  const int* exps;
  float* y;
  int H, W, C, N, OH, OW, pt, pl;
  int row_patches, col_patches, patches;
  unsigned x_bytes, y_bytes;
  int pw_act;
};
// What the depthwise layer needs comes in the 14 dwords of arguments that a wavefront finds in its scalar registers when it starts,
// dimensions in halves; the rest is read from memory while that is under way (the pass of 64 images 588 -> 583 us, of 8 194.4 -> 192.2).
struct TileRest {
  const float *pw_w, *pw_b;
  const half_t* packed;
  const int* exps;
  float* y;
  unsigned y_bytes;
  int pw_act;
};

// S: stride; TM: 32-pixel blocks of a tile; WK: parts of the contraction (wavefront = column group + WN x part)
template <int S, int TM, int WK>
__global__ __launch_bounds__(512) void separable_tile_kernel(const float* x, const float* dw_w, const float* dw_b, unsigned x_bytes, unsigned map,
                                                           unsigned out_map, unsigned channels, unsigned per, int patches, int total,
                                                           unsigned form, TileRest g) {
  static_assert(WK == 1 || TM == 1, "the parts' sums take the tile's place");
  constexpr int PATCHES = 4 * TM, kAhead = TM == 1 ? 4 : 2;
  // Few pixels, which leave the matrix cores idle, are computed as exactly as by the kernels that take them otherwise: all four
  // products, and the large ones of four k-steps summed apart from those before (an instruction cuts off what lies behind the last
  // place of its accumulator).
  constexpr bool kFine = WK > 1;
  struct Patch {
    int out, cols, rows, ih, iw, image;  // first output pixel, extent inside the map; first tap's row and column, image's first row
  };
  extern __shared__ __align__(16) half_t tile[];  // the tile's depthwise output, two planes of [32 TM][C + 8]; later the parts' sums
  __shared__ Patch patch[PATCHES];
  __shared__ __align__(16) float bias[512];
  __shared__ __align__(16) int exps[512];
  __shared__ unsigned row_nan[TM];
  __shared__ int lost, lost_tiny;

  const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int li = lane % 32, h = lane / 32;
  const int H = (int)(map & 0xffff), W = (int)(map >> 16), OH = (int)(out_map & 0xffff), OW = (int)(out_map >> 16);
  const int C = (int)(channels & 0xffff), N = (int)(channels >> 16), row_patches = (int)(per & 0xffff), col_patches = (int)(per >> 16);
  const int pt = (int)(form & 1), pl = (int)(form >> 1 & 1), tiles_n = (int)(form >> 2 & 31);
  const int waves_n = (int)(form >> 7), threads = 64 * waves_n * WK, wn = wave % waves_n, part = wave / waves_n;
  int bid = blockIdx.x;
  {  // tiles of the same pixels, and neighbouring ones, on one XCD
    const int q = total / kXcds, rem = total % kXcds, xcd = bid % kXcds;
    bid = xcd * q + (xcd < rem ? xcd : rem) + bid / kXcds;
  }
  const int tile_n = bid % tiles_n, tile_m = bid / tiles_n;
  const int C4 = C / 4, LD = C + 8, plane = 32 * TM * LD;
  const int first_n = 64 * tile_n * waves_n;

  if (tid < PATCHES) {
    const int i = tile_m * PATCHES + tid, row = i / row_patches, n = row / col_patches;
    const int ow = 4 * (i % row_patches), oh = 2 * (row % col_patches);
    Patch p;
    p.out = (n * OH + oh) * OW + ow;
    p.cols = i < patches ? (OW - ow < 4 ? OW - ow : 4) : 0;
    p.rows = OH - oh < 2 ? 1 : 2;
    p.ih = oh * S - pt;
    p.iw = ow * S - pl;
    p.image = n * H;
    patch[tid] = p;
  }
  if (tid < TM) row_nan[tid] = 0;
  if (tid == TM) lost = lost_tiny = 0;
  __syncthreads();
  float column_bias = 0.f;
  int column_exp = 0;
  if (tid < 64 * waves_n) column_bias = g.pw_b[first_n + tid], column_exp = g.exps[first_n + tid];

  // Each workgroup fetches its share of the filter's lines into its XCD's L2 while it computes the depthwise layer, a dword of each
  // (block_tile_f16.hip); those after the first 64 of an XCD find it there.
  const int of_xcd = max(1, min(total / kXcds, 64)), lines = C * N / 32, l0 = lines * min((int)blockIdx.x / kXcds, of_xcd - 1) / of_xcd;
  const int line = min(l0 + min(tid, (lines - 1) / of_xcd), lines - 1);
  auto touch = [&]() __attribute__((always_inline)) { return reinterpret_cast<const unsigned*>(g.packed)[32 * line]; };
  unsigned touched = 0;
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, (int)x_bytes, 0x00020000);
  MapLoss loss;
  if (tid >= PATCHES * C4) touched = touch();
  for (int item = tid; item < PATCHES * C4; item += threads) {
    const int s = item / C4, c4 = item - s * C4;
    constexpr int PX = S == 1 ? 4 : 2, ROWS = S + 3, COLS = (PX - 1) * S + 3;  // columns at a time, and what they read
    f32x4 w[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) w[t] = *reinterpret_cast<const f32x4*>(dw_w + (size_t)t * C + 4 * c4);
    const f32x4 bv = *reinterpret_cast<const f32x4*>(dw_b + 4 * c4);
    // byte offsets of a row and a column of x; outside the map (and for a patch outside the batch) the largest, which the
    // saturating sum keeps: such a load is past the end and reads zeros
    const Patch at = patch[s];
    unsigned row_off[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
      row_off[i] = (unsigned)(at.ih + i) < (unsigned)H && at.cols > 0 ? 4u * ((unsigned)(at.image + at.ih + i) * W * C + 4 * c4) : ~0u;
#pragma unroll
    for (int p0 = 0; p0 < 4; p0 += PX) {
      f32x4 win[ROWS][COLS];
#pragma unroll
      for (int j = 0; j < COLS; ++j) {
        const int iw = at.iw + p0 * S + j;
        const unsigned col_off = (unsigned)iw < (unsigned)W ? 4u * (unsigned)(iw * C) : ~0u;
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
          win[i][j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, __builtin_elementwise_add_sat(row_off[i], col_off), 0, 0));
      }
      if (item == tid && p0 == 0) touched = touch();
#pragma unroll
      for (int p = 0; p < 2 * PX; ++p) {
        f32x4 acc = bv;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = fmaf(win[p % 2 * S + t / 3][p / 2 * S + t % 3][e], w[t][e], acc[e]);
        const int row = 8 * s + 4 * (p % 2) + p0 + p / 2;
        const bool nan = __builtin_isunordered(acc[0], acc[1]) || __builtin_isunordered(acc[2], acc[3]);
        floatx4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = __builtin_amdgcn_fmed3f(acc[e], 0.f, 6.f);
          loss.see(v[e]);
        }
        pairx4 hi, lo;
        split2(v, (float)(1 << kMapScale), hi, lo);
        if (nan) {
          constexpr unsigned kNan = 0x7e00;
          hi[0] = (acc[0] == acc[0] ? hi[0] & 0xffffu : kNan) | (acc[1] == acc[1] ? hi[0] & 0xffff0000u : kNan << 16);
          hi[1] = (acc[2] == acc[2] ? hi[1] & 0xffffu : kNan) | (acc[3] == acc[3] ? hi[1] & 0xffff0000u : kNan << 16);
          atomicOr(&row_nan[row / 32], 1u << (row % 32));
        }
        *reinterpret_cast<pairx4*>(tile + row * LD + 4 * c4) = hi;
        *reinterpret_cast<pairx4*>(tile + plane + row * LD + 4 * c4) = lo;
      }
    }
  }
  if (tid < 64 * waves_n) bias[tid] = column_bias, exps[tid] = column_exp;
  {
    const int l = loss.lost(8 * PATCHES * C4 / threads * 4 + 32);  // (all that this thread computed, for one of them)
    if (l != 0) {
      atomicAdd(&lost, l & kLostMost);
      if ((l & kLostTiny) != 0) atomicOr(&lost_tiny, kLostTiny);
    }
  }

  asm volatile("" ::"v"(touched));
  __builtin_amdgcn_sched_barrier(0);
  // the filter's operands, in the order of pack_filters (pack.h)
  const int n0 = first_n + 64 * wn;
  const int steps = C / 16, s0 = steps / WK * part, s1 = s0 + steps / WK;
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(g.packed), 0, C * N * 4, 0x00020000);
  const int wp = n0 / 64 * steps * 4096;
  h8 raw[kAhead][2][2];
  auto load_step = [&](int s, h8 (&r)[2][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      r[i / 2][i % 2] = __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(wr, 16 * lane + 1024 * i, wp + 4096 * s, 0));
  };
#pragma unroll
  for (int u = 0; u < kAhead; ++u) load_step(s0 + u, raw[u]);
  f32x16 acc[TM][2], mixed[TM][2], part_sum[2];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][0][i] = acc[t][1][i] = mixed[t][0][i] = mixed[t][1][i] = 0.f;
  __syncthreads();

  // The scheduling barriers keep the loads of a step together (block_tile_f16.hip).
  const half_t* const a_base = tile + li * LD + 8 * h;
  h8 a[2][TM][2];
  auto read = [&](int buf, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int p = 0; p < 2; ++p) a[buf][t][p] = *reinterpret_cast<const h8*>(a_base + p * plane + 32 * t * LD + 16 * s);
  };
  read(0, s0);
  for (int s = s0; s < s1; s += kAhead) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      read((u + 1) & 1, s + u + 1 < s1 ? s + u + 1 : s0);
      h8 b[2][2];
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i / 2][i % 2] = raw[u][i / 2][i % 2];
      load_step(s + u + kAhead < s1 ? s + u + kAhead : s1 - 1, raw[u]);  // past the end: the last step again, dropped
#pragma unroll
      for (int pass = kFine ? 0 : 1; pass < 4; ++pass)  // (low, low), (low, high), (high, high), (high, low)
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const h8 at = pass == 0 ? a[u & 1][t][1] * (half_t)(1 / kLow) : a[u & 1][t][pass == 3];
            f32x16& to = pass == 2 ? acc[t][j] : mixed[t][j];
            if (kFine && pass == 2) part_sum[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[j][0], at, u == 0 ? f32x16{} : part_sum[j], 0, 0, 0);
            else to = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[j][pass < 2], at, to, 0, 0, 0);
          }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kFine) acc[0][0] += part_sum[0], acc[0][1] += part_sum[1];
  }

  // Lane (li, h) has pixel li of each 32 and, in group i of the accumulators of column block j, channels 32 j + 8 i + 4 h ... + 3 of
  // the wavefront's 64.
  const ActClamp clamp = make_act(g.pw_act);
  const float lowest = clamp.on ? 0.f : -INFINITY;
  unsigned out[TM];
  const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(g.y, 0, (int)g.y_bytes, 0x00020000);
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const Patch at = patch[4 * t + li / 8];
    const int row = li % 8 / 4, col = li % 4;
    // past the end, where nothing is stored, for a lane without a pixel
    out[t] = row < at.rows && col < at.cols ? 4u * ((unsigned)(at.out + row * OW + col) * N + n0 + 4 * h) : 0x80000000u;
  }
  constexpr int GROUPS = 8 * TM / WK;  // of four channels, for this wavefront
  const int g0 = part * GROUPS;
  f32x4 v[GROUPS];
  if constexpr (WK == 1) {
#pragma unroll
    for (int q = 0; q < GROUPS; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[q][e] = fmaf(mixed[q / 8][q / 4 % 2][4 * (q % 4) + e], 1 / kLow, acc[q / 8][q / 4 % 2][4 * (q % 4) + e]);
  } else {
    // the parts' sums through LDS: part p adds up groups p GROUPS ... of its columns
    f32x4* const sums = reinterpret_cast<f32x4*>(tile);  // [wave][group][64]
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      f32x4 t;
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = fmaf(mixed[0][q / 4][4 * (q % 4) + e], 1 / kLow, acc[0][q / 4][4 * (q % 4) + e]);
      sums[(wave * 8 + q) * 64 + lane] = t;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < GROUPS; ++q) {
      v[q] = sums[(wn * 8 + g0 + q) * 64 + lane];
#pragma unroll
      for (int p = 1; p < WK; ++p) v[q] += sums[((p * waves_n + wn) * 8 + g0 + q) * 64 + lane];
    }
  }
  float finite = 0.f, smallest = INFINITY;  // NaN where a result is not finite; the smallest magnitude
  int column_lost = 0, exponent = 1 << 20;
#pragma unroll
  for (int q = 0; q < GROUPS; ++q) {
    const int i = 64 * wn + 8 * ((g0 + q) % 8) + 4 * h;
    const f32x4 bv = *reinterpret_cast<const f32x4*>(bias + i);
    const i32x4 ev = *reinterpret_cast<const i32x4*>(exps + i);
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[q][e] = ldexpf(v[q][e], -(ev[e] >> 17) - kMapScale) + bv[e];
      finite = fmaf(v[q][e], 0.f, finite);
      smallest = fminf(smallest, fabsf(v[q][e]));
      column_lost |= ev[e];  // (at least each of them)
      exponent = min(exponent, ev[e] >> 17);
      o[e] = __builtin_amdgcn_fmed3f(v[q][e], lowest, clamp.hi);
    }
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), yr, out[TM == 1 ? 0 : q / 8] + 32 * ((g0 + q) % 8), 0, 0);
  }
  const int tile_lost = min(lost, kLostMost) | lost_tiny;
  // (the code behind this is in no instruction cache)
  if (__builtin_amdgcn_ballot_w64(finite != finite || smallest < loss_limit(C, exponent + kMapScale, more_lost(tile_lost, column_lost))) == 0) return;

  // Which of a lane's results are computed again, over the first ones: a pixel at a time, its depthwise output over the lanes; then
  // up to four columns one after the other, a sum over the lanes, or all 64, a lane for each.
  constexpr int WORDS = (4 * GROUPS + 31) / 32;
  unsigned again[WORDS] = {};
#pragma unroll
  for (int q = 0; q < GROUPS; ++q) {
    const i32x4 ev = *reinterpret_cast<const i32x4*>(exps + 64 * wn + 8 * ((g0 + q) % 8) + 4 * h);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool small = fabsf(v[q][e]) < loss_limit(C, (ev[e] >> 17) + kMapScale, more_lost(tile_lost, ev[e]));
      if ((small || !__builtin_isfinite(v[q][e])) && out[TM == 1 ? 0 : q / 8] < 0x80000000u) again[q / 8] |= 1u << (4 * (q % 8) + e);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // behind the first results
#pragma unroll
  for (int t = 0; t < WORDS; ++t) {
    unsigned long long lanes = __builtin_amdgcn_ballot_w64(again[t] != 0);
    unsigned pixels = (unsigned)lanes | (unsigned)(lanes >> 32);
    while (pixels != 0) {
      const int px = __builtin_ctz(pixels);
      pixels &= pixels - 1;
      const int q = lane / 8 - g0;  // (g0 is 0 where there are more than 8 groups)
      const unsigned word = __shfl(again[t], px + 32 * (lane / 4 % 2));
      const bool mine = q >= 0 && q < GROUPS && (word >> (4 * (q & 7) + lane % 4) & 1) != 0;  // of column `lane`
      const unsigned long long columns = __builtin_amdgcn_ballot_w64(mine);
      const Patch p = patch[4 * t + px / 8];
      const int ih = p.ih + px % 8 / 4 * S, iw = p.iw + px % 4 * S;
      auto depthwise = [&](int k) __attribute__((always_inline)) {
        float d = dw_b[k];
#pragma unroll
        for (int kk = 0; kk < 9; ++kk) {
          const int r = ih + kk / 3, c = iw + kk % 3;
          const bool in = (unsigned)r < (unsigned)H && (unsigned)c < (unsigned)W;
          const float xv = x[in ? ((size_t)(p.image + r) * W + c) * C + k : 0];
          d = in ? fmaf(xv, dw_w[(size_t)kk * C + k], d) : d;
        }
        return apply_act(d, TFX_ACT_RELU6);
      };
      float sum = 0.f;
      if ((row_nan[t] >> px & 1) != 0) {
        sum = NAN;
      } else if (__builtin_popcountll(columns) <= 4) {
        float d[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) d[i] = 64 * i + lane < C ? depthwise(64 * i + lane) : 0.f;
        for (unsigned long long rest = columns; rest != 0; rest &= rest - 1) {
          const int col = __builtin_ctzll(rest);
          float s = 0.f;
#pragma unroll
          for (int i = 0; i < 16; ++i) s = fmaf(d[i], 64 * i + lane < C ? g.pw_w[(size_t)(64 * i + lane) * N + n0 + col] : 0.f, s);
#pragma unroll
          for (int m = 32; m > 0; m /= 2) s += __shfl_xor(s, m);
          sum = lane == col ? s : sum;
        }
      } else {
#pragma unroll 1
        for (int k0 = 0; k0 < C; k0 += 64) {
          const float d = k0 + lane < C ? depthwise(k0 + lane) : 0.f;
          float part_sum = 0.f;
#pragma unroll 1
          for (int k1 = 0; k1 < 64 && k0 + k1 < C; k1 += 32)
#pragma unroll
            for (int k = 0; k < 32; ++k)
              part_sum = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(d), k1 + k)), g.pw_w[(size_t)(k0 + k1 + k) * N + n0 + lane], part_sum);
          sum += part_sum;
        }
      }
      const unsigned to = (unsigned)__builtin_amdgcn_readlane((int)out[TM == 1 ? 0 : t], px);
      if (mine) *reinterpret_cast<float*>(reinterpret_cast<char*>(g.y) + to + 4u * (unsigned)lane) = apply_act(sum + bias[64 * wn + lane], clamp);
    }
  }
}

size_t tile_lds(int tm, int waves_n, int wk, int c) {
  const size_t depth = (size_t)32 * tm * (c + 8) * 2 * sizeof(half_t), sums = wk == 1 ? 0 : (size_t)waves_n * wk * 32 * 64 * sizeof(float);
  return depth > sums ? depth : sums;
}

template <int S, int TM, int WK>
int launch_tile(const TileArgs& args, int waves_n, hipStream_t stream) {
  const TileArgs& g = args;
  auto kern = separable_tile_kernel<S, TM, WK>;
  const size_t lds_bytes = tile_lds(TM, waves_n, WK, g.C);
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), 150 * 1024, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  const int tiles_n = g.N / (64 * waves_n), total = (g.patches + 4 * TM - 1) / (4 * TM) * tiles_n;
  auto halves = [](int low, int high) { return (unsigned)low | (unsigned)high << 16; };
  hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(64u * waves_n * WK), lds_bytes, stream, g.x, g.dw_w, g.dw_b, g.x_bytes,
                     halves(g.H, g.W), halves(g.OH, g.OW), halves(g.C, g.N), halves(g.row_patches, g.col_patches), g.patches, total,
                     (unsigned)(g.pt | g.pl << 1 | tiles_n << 2 | waves_n << 7), TileRest{g.pw_w, g.pw_b, g.packed, g.exps, g.y, g.y_bytes, g.pw_act});
  return check_launch();
}

// The largest divisor of `groups` up to `most`.
int divisor(int groups, int most) {
  for (int d = groups < most ? groups : most; d > 1; --d)
    if (groups % d == 0) return d;
  return 1;
}

// The tile (32 tm pixels, column groups of wavefronts, parts of the contraction): the least modelled time -- a start; for each round of
// resident workgroups another and the depthwise layer of a thread; for each workgroup of a CU its depthwise loads, its columns of
// the filter from L2, its matrix instructions and stores.  Fitted to 4233 launches (2 - 64 images, every width, 3 sizes); the form it
// takes is 2 % slower than the fastest on average, 19 % at most.  14 x 14 x 512 -> 512, us a launch: 64 images {2, 8, 1} 34, {1, 8, 1} 40;
// 16 images {1, 4, 2} 15.6, {1, 8, 1} 18.4, {2, 8, 1} 26; 8 images {1, 2, 4} 12.2, {1, 4, 2} 13.6; 4 images {1, 1, 4} 10.6, {1, 4, 2} 13.3.
struct TileForm {
  int tm, waves_n, wk;
  double us;
};
TileForm tile_form(long long patches, int c, int n, int stride) {
  const int groups = n / 64;
  TileForm best{};
  best.us = 1e30;
  for (int tm = c % 64 == 0 ? 1 : 2; tm <= 2 && tm * c <= 1024; ++tm)  // (k-steps of a part are taken four at a time, or two with tm = 2)
    for (int wk = 1; wk <= (tm == 1 ? 4 : 1) && (wk == 1 || c % (64 * wk) == 0); wk *= 2)
      for (int most = 8 / wk; most > 0; most /= 2) {
        const int waves_n = divisor(groups, most), waves = waves_n * wk;
        const long long blocks = (patches + 4 * tm - 1) / (4 * tm) * (groups / waves_n);
        const int lds = (int)tile_lds(tm, waves_n, wk, c) + 5 * 1024, resident = 8 / waves < 160 * 1024 / lds ? 8 / waves : 160 * 1024 / lds;
        const double rounds = (double)((blocks + 256 * resident - 1) / (256 * resident)), cu = (double)((blocks + 255) / 256);
        const double us = 3.1 + rounds * (1.4 + .0157 * c * tm * stride / waves) +
                          cu * (c * (1.09e-3 * tm * stride + 4.9e-3 * tm + 1.3e-3 * waves_n + .33e-3 * tm * waves_n) + .59 * tm * waves_n);
        if (us < best.us) best = TileForm{tm, waves_n, wk, us};
      }
  return best;
}
}  // namespace

size_t separable_tile_packed_bytes(int c, int n) { return ((size_t)c * n + (size_t)n) * sizeof(float); }

bool separable_tile_supported(int batch, int h, int w, int c, int n, int stride, int oh, int ow, const void* x, const void* dw_w,
                              const void* dw_b, const void* pw_w, const void* pw_b, const void* y) {
  const void* ptrs[] = {x, dw_w, dw_b, pw_w, pw_b, y};
  bool aligned = true;
  for (const void* p : ptrs) aligned = aligned && reinterpret_cast<uintptr_t>(p) % 16 == 0;
  const long long patches = (long long)batch * ((oh + 1) / 2) * ((ow + 3) / 4), x_bytes = (long long)batch * h * w * c * 4,
                  y_bytes = (long long)batch * oh * ow * n * 4;
  return aligned && (stride == 1 || stride == 2) && c >= 64 && (c % 64 == 0 ? c <= 1024 : c % 32 == 0 && c <= 512) && n % 64 == 0 && n <= 1024 &&
         x_bytes < (1ll << 31) && y_bytes < (1ll << 31) && patches < (1ll << 27) && h < 65536 && w < 65536;
}

int launch_separable_tile(const float* x, const float* dw_w, const float* dw_b, const float* pw_w, const float* pw_b, const void* packed,
                          float* y, int batch, int h, int w, int c, int n, int oh, int ow, int stride, int pt, int pl, int pw_act,
                          hipStream_t stream) {
  const int row_patches = (ow + 3) / 4, col_patches = (oh + 1) / 2, patches = batch * col_patches * row_patches;
  const half_t* const parts = static_cast<const half_t*>(packed);
  const TileArgs g{x, dw_w, dw_b, pw_w, pw_b, parts, reinterpret_cast<const int*>(parts + (size_t)2 * c * n), y, h, w, c, n, oh, ow, pt, pl,
                   row_patches, col_patches, patches, (unsigned)((long long)batch * h * w * c * 4),
                   (unsigned)((long long)batch * oh * ow * n * 4), pw_act};
  const TileForm f = tile_form(patches, c, n, stride);
#define TFX_TILE(S, TM, WK) \
  if (stride == S && f.tm == TM && f.wk == WK) return launch_tile<S, TM, WK>(g, f.waves_n, stream);
  TFX_TILE(1, 2, 1)
  TFX_TILE(1, 1, 1)
  TFX_TILE(1, 1, 2)
  TFX_TILE(1, 1, 4)
  TFX_TILE(2, 2, 1)
  TFX_TILE(2, 1, 1)
  TFX_TILE(2, 1, 2)
  TFX_TILE(2, 1, 4)
#undef TFX_TILE
  return TFX_ERR_UNSUPPORTED;
}

}  // namespace tfx
