// A depthwise-separable block (depthwise 3x3 + bias + clamp, pointwise 1x1 + bias + clamp) on binary16 storage in one
// launch, for the layers whose pointwise filter does not fit a workgroup's LDS (Section 4.1 storage format, the 28 x 28 ...
// 7 x 7 blocks of the Section 3.9 network).
//
// A workgroup owns a tile of 32 TM output pixels, as patches of 4 x 2, and 64 columns for each of its groups of wavefronts.
// First all its threads compute the depthwise output of the tile -- the whole depth of the contraction, up to 132 KB -- into
// LDS, rounded to binary16 as the separate kernel rounds it (the same bits): an item is 8 channels of a patch, whose 24
// 16-byte pieces (stride 2: 25 for each half) are all loaded before the first multiply.  Then each wavefront multiplies the
// tile by its 64 columns of the filter (v_mfma_f32_32x32x16_f16), whose operands it loads straight from L2, four k-steps
// ahead.  The depthwise output so never goes to memory and back, one launch of two is left, and no barrier stands in the
// contraction.
//
// The filter comes in the order of the operands, 16 bytes for a lane; pack_filters_kernel puts the filters of all such
// layers of a pass into it, in one launch of 4 us (loaded as it is stored, two columns of a k-row at a time, the
// contraction took 11 us instead of 7, and more in all layers together than that launch).
//
// The first rows of the filter were late for every workgroup of an XCD at once, in its L2 for the first time and all waiting for
// the same k-step: so each fetches its share of the filter's lines there while it computes the depthwise layer.  And the filter is
// the first operand, so that a lane has 8 consecutive channels of a pixel to store (two of them, 32 stores of 4 bytes, kept the
// memory busy after the contraction: 2.7 us, now 1.6).
//
// 64 x 14 x 14 x 512 -> 512, one layer: 17.2 us (18.5 without the last two), of which 1.2 are the start and the launch, 6 the
// depthwise layer (the map's 13 MB from memory, then its arithmetic), 5.5 the contraction, 2 the stores; the two separate kernels
// take 26 back to back and 32 in the network.  64 x 28 x 28 x 256 -> 256 33 -> 26, 64 x 28 x 28 x 256 -> 512 at stride 2 20 -> 16,
// 64 x 7 x 7 x 1024 -> 1024 23 -> 21 (its contraction 9 - 11: a megabyte of the filter for each CU).  The whole pass of 64 images
// 287 -> 277 us, 16 images 168 -> 164.
#include "stream_f16.h"

namespace tfx {
namespace {

using namespace f16s;

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kXcds = 8, kAhead = 4, kMaxLayers = 13;

struct TileBlockArgs {
  const half_t *x, *dw_w, *dw_b, *pw_w, *pw_b;
  half_t* y;
  int H, W, C, N, OH, OW, pt, pl;
  int row_patches, col_patches, patches;
  unsigned x_bytes, y_bytes;
  int dw_act, pw_act;
};
// What the depthwise layer needs comes in the 14 dwords of arguments that a wavefront finds in its scalar registers when it starts,
// dimensions in halves; the rest is read from memory while that is under way, as the fp32 form's (passes of 8 - 64 images: .99 of the time on one GPU, the same on another).
struct TileRest {
  const half_t *pw_w, *pw_b;
  half_t* y;
  unsigned y_bytes;
  int dw_act, pw_act;
};

// S: stride; TM: 32-pixel blocks of a tile; WK: parts of the contraction (wavefront = column group + WN x part)
template <int S, int TM, int WK>
__global__ __launch_bounds__(512) void separable_tile_f16_kernel(const half_t* x, const half_t* dw_w, const half_t* dw_b, unsigned x_bytes, unsigned map,
                                                               unsigned out_map, unsigned channels, unsigned per, int patches, int total,
                                                               unsigned form, TileRest g) {
  constexpr int PATCHES = 4 * TM;
  struct Patch {
    int out, cols, rows, ih, iw, image;  // first output pixel, extent inside the map; first tap's row and column, image's first row
  };
  extern __shared__ __align__(16) half_t tile[];  // the tile's depthwise output, [32 TM][C + 8]; later the parts' sums
  __shared__ Patch patch[PATCHES];

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
  const int C8 = C / 8, LD = C + 8;

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
  __syncthreads();

  // The filter is in no L2 yet, and all workgroups of an XCD walk through it in the same order: each fetches its share of the lines
  // while the depthwise layer is computed, a dword of each, instead of all waiting for every k-step in turn.
  // (Those after the first 64 of an XCD find it there.)
  const int of_xcd = max(1, min(total / kXcds, 64)), lines = C * N / 64, l0 = lines * min((int)blockIdx.x / kXcds, of_xcd - 1) / of_xcd;
  const int line = min(l0 + min(tid, (lines - 1) / of_xcd), lines - 1);
  auto touch = [&]() __attribute__((always_inline)) { return reinterpret_cast<const unsigned*>(g.pw_w)[32 * line]; };
  unsigned touched = 0;
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(x), 0, (int)x_bytes, 0x00020000);
  const ActClamp dw_clamp = make_act(g.dw_act);
  if (tid >= PATCHES * C8) touched = touch();
  for (int item = tid; item < PATCHES * C8; item += threads) {
    const int s = item / C8, c8 = item - s * C8;
    constexpr int PX = S == 1 ? 4 : 2, ROWS = S + 3, COLS = (PX - 1) * S + 3;  // columns at a time, and what they read
    u32x4 wraw[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) wraw[t] = *reinterpret_cast<const u32x4*>(dw_w + (size_t)t * C + 8 * c8);
    const h8 bv = *reinterpret_cast<const h8*>(dw_b + 8 * c8);
    // byte offsets of a row and a column of x; outside the map (and for a patch outside the batch) the largest, which the
    // saturating sum keeps: such a load is past the end and reads zeros
    const Patch at = patch[s];
    unsigned row_off[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
      row_off[i] = (unsigned)(at.ih + i) < (unsigned)H && at.cols > 0 ? 2u * ((unsigned)(at.image + at.ih + i) * W * C + 8 * c8) : ~0u;
#pragma unroll
    for (int p0 = 0; p0 < 4; p0 += PX) {
      u32x4 win[ROWS][COLS];
#pragma unroll
      for (int j = 0; j < COLS; ++j) {
        const int iw = at.iw + p0 * S + j;
        const unsigned col_off = (unsigned)iw < (unsigned)W ? 2u * (unsigned)(iw * C) : ~0u;
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
          win[i][j] = __builtin_amdgcn_raw_buffer_load_b128(xr, __builtin_elementwise_add_sat(row_off[i], col_off), 0, 0);
      }
      if (item == tid && p0 == 0) touched = touch();
#pragma unroll
      for (int p = 0; p < 2 * PX; ++p) {
        f32x4 acc[2];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e / 4][e % 4] = (float)bv[e];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
          // the filter stays packed: without the empty asm its conversions to fp32 are hoisted into 72 more registers
          asm volatile("" : "+v"(wraw[t]));
          const h8 wt = __builtin_bit_cast(h8, wraw[t]), xt = __builtin_bit_cast(h8, win[p % 2 * S + t / 3][p / 2 * S + t % 3]);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e / 4][e % 4] = fmaf((float)xt[e], (float)wt[e], acc[e / 4][e % 4]);
        }
        h8 out[1];
        activate_and_pack(acc, dw_clamp, out);
        *reinterpret_cast<h8*>(tile + (8 * s + 4 * (p % 2) + p0 + p / 2) * LD + 8 * c8) = out[0];
      }
    }
  }

  asm volatile("" ::"v"(touched));
  __builtin_amdgcn_sched_barrier(0);
  // the filter's operands, in the order of pack_filters_kernel
  const int n0 = 64 * (tile_n * waves_n + wn);
  const int steps = C / 16, s0 = steps / WK * part, s1 = s0 + steps / WK;
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(g.pw_w), 0, C * N * 2, 0x00020000);
  const int wp = n0 / 64 * steps * 2048;
  h8 raw[kAhead][2];
  auto load_step = [&](int s, h8 (&r)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      r[i] = __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(wr, 16 * lane + 1024 * i, wp + 2048 * s, 0));
  };

#pragma unroll
  for (int u = 0; u < kAhead; ++u) load_step(s0 + u, raw[u]);
  // before the stores, which loads after them would wait for: the bias of this part's groups
  constexpr int QP = 4 * TM / WK, BIASES = QP < 4 ? QP : 4;
  static_assert(QP >= 1 && (WK == 1 || TM == 1), "a group for every part");
  h8 bias[BIASES];
#pragma unroll
  for (int i = 0; i < BIASES; ++i) bias[i] = *reinterpret_cast<const h8*>(g.pw_b + n0 + 8 * h + 16 * (part * BIASES + i));
  f32x16 acc[TM][2];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][0][i] = acc[t][1][i] = 0.f;
  __syncthreads();

  // The scheduling barriers keep the loads of a step together: left to itself the compiler mixes those of several steps, and
  // the first step then waits for all of them.
  const half_t* const a_base = tile + li * LD + 8 * h;
  h8 a[2][TM];
#pragma unroll
  for (int t = 0; t < TM; ++t) a[0][t] = *reinterpret_cast<const h8*>(a_base + 32 * t * LD + 16 * s0);
  for (int s = s0; s < s1; s += kAhead) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int next = s + u + 1 < s1 ? s + u + 1 : s0;
#pragma unroll
      for (int t = 0; t < TM; ++t) a[(u + 1) & 1][t] = *reinterpret_cast<const h8*>(a_base + 32 * t * LD + 16 * next);
      const h8 b0 = raw[u][0], b1 = raw[u][1];
      load_step(s + u + kAhead < s1 ? s + u + kAhead : s1 - 1, raw[u]);  // past the end: the last step again, dropped
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        acc[t][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b0, a[u & 1][t], acc[t][0], 0, 0, 0);
        acc[t][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b1, a[u & 1][t], acc[t][1], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // Lane (li, h) has pixel li of each 32; group i of its accumulators is channels 16 i + 8 h ... + 7 of the wavefront's 64, the even
  // ones in the first.
  const ActClamp pw_clamp = make_act(g.pw_act);
  unsigned out[TM];
  const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(g.y, 0, (int)g.y_bytes, 0x00020000);
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const Patch at = patch[4 * t + li / 8];
    const int row = li % 8 / 4, col = li % 4;
    // past the end, where nothing is stored, for a lane without a pixel
    out[t] = row < at.rows && col < at.cols ? 2u * ((unsigned)(at.out + row * OW + col) * N + n0 + 8 * h) : 0x80000000u;
  }
  auto emit = [&](int q, h8 bv, const float (&v0)[4], const float (&v1)[4]) __attribute__((always_inline)) {
    f32x4 v[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e / 2][2 * (e % 2)] = v0[e] + (float)bv[2 * e], v[e / 2][2 * (e % 2) + 1] = v1[e] + (float)bv[2 * e + 1];
    h8 o[1];
    activate_and_pack(v, pw_clamp, o);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o[0]), yr, out[TM == 1 ? 0 : q / 4] + 32 * (q % 4), 0, 0);
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int q = 0; q < 4 * TM; ++q) {
      float v0[4], v1[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v0[r] = acc[q / 4][0][4 * (q % 4) + r], v1[r] = acc[q / 4][1][4 * (q % 4) + r];
      emit(q, bias[q % 4], v0, v1);
    }
  } else {
    // the parts' sums through LDS: part p adds up groups p QP ... of its columns
    float* const sums = reinterpret_cast<float*>(tile);  // [wave][group][8][64]
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4 * TM; ++q)
#pragma unroll
      for (int r = 0; r < 8; ++r)
        sums[((wave * 4 * TM + q) * 8 + r) * 64 + lane] = acc[q / 4][r / 4][4 * (q % 4) + r % 4];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < QP; ++i) {
      const int q = part * QP + i;
      float v[2][4];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        float t = 0.f;
#pragma unroll
        for (int p = 0; p < WK; ++p) t += sums[(((p * waves_n + wn) * 4 * TM + q) * 8 + r) * 64 + lane];
        v[r / 4][r % 4] = t;
      }
      emit(q, bias[i], v[0], v[1]);
    }
  }
}

// The operands of the contraction's k-step s (rows 16 s ... + 15) and 64 columns from 64 c on, for each lane: 8 rows from
// 8 (lane / 32) on of column 2 (lane % 32), then of the next column, at piece 128 (steps c + s) + lane (+ 64).
struct PackArgs {
  const half_t* w[kMaxLayers];
  h8* out[kMaxLayers];
  int c[kMaxLayers], n[kMaxLayers], first[kMaxLayers + 1];  // first: workgroups of the layers before
  int layers;
};
__global__ __launch_bounds__(256) void pack_filters_kernel(PackArgs g) {
  int l = 0;
  while (l + 1 < g.layers && (int)blockIdx.x >= g.first[l + 1]) ++l;
  const int u = ((int)blockIdx.x - g.first[l]) * 4 + (int)threadIdx.x / 64, lane = threadIdx.x % 64;
  const int N = g.n[l], groups = N / 64, steps = g.c[l] / 16;
  if (u >= groups * steps) return;
  const int c = u % groups, s = u / groups;
  const half_t* const w = g.w[l] + (size_t)(16 * s + 8 * (lane / 32)) * N + 64 * c + 2 * (lane % 32);
  unsigned raw[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) raw[i] = *reinterpret_cast<const unsigned*>(w + (size_t)i * N);
  u32x4 b0, b1;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    b0[j] = __builtin_amdgcn_perm(raw[2 * j + 1], raw[2 * j], 0x05040100u);
    b1[j] = __builtin_amdgcn_perm(raw[2 * j + 1], raw[2 * j], 0x07060302u);
  }
  h8* const out = g.out[l] + (size_t)128 * (steps * c + s) + lane;
  out[0] = __builtin_bit_cast(h8, b0);
  out[64] = __builtin_bit_cast(h8, b1);
}

template <int S, int TM, int WK>
int launch_tile(const TileBlockArgs& args, int waves_n, hipStream_t stream) {
  const TileBlockArgs& g = args;
  auto kern = separable_tile_f16_kernel<S, TM, WK>;
  const size_t depth = (size_t)32 * TM * (g.C + 8) * sizeof(half_t), sums = WK == 1 ? 0 : (size_t)waves_n * WK * TM * 32 * 64 * sizeof(float);
  const size_t lds_bytes = depth > sums ? depth : sums;
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), 160 * 1024 - 1024, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  const int tiles_n = g.N / (64 * waves_n), total = (g.patches + 4 * TM - 1) / (4 * TM) * tiles_n;
  auto halves = [](int low, int high) { return (unsigned)low | (unsigned)high << 16; };
  hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(64u * waves_n * WK), lds_bytes, stream, g.x, g.dw_w, g.dw_b, g.x_bytes,
                     halves(g.H, g.W), halves(g.OH, g.OW), halves(g.C, g.N), halves(g.row_patches, g.col_patches), g.patches, total,
                     (unsigned)(g.pt | g.pl << 1 | tiles_n << 2 | waves_n << 7), TileRest{g.pw_w, g.pw_b, g.y, g.y_bytes, g.dw_act, g.pw_act});
  return check_launch();
}

// The largest divisor of `groups` up to `most`.
int divisor(int groups, int most) {
  for (int d = groups < most ? groups : most; d > 1; --d)
    if (groups % d == 0) return d;
  return 1;
}

// The tile (32 tm pixels, column groups of wavefronts, parts of the contraction): the least modelled time -- a start for each round
// of resident workgroups (8 wavefronts a CU), and for each workgroup of a CU its depthwise layer, which all workgroups of a tile
// compute, and its columns of the filter from L2.  With the largest tile of at least 160 workgroups instead, 280 of them were two
// rounds: 10 images 188 us, now 155; 20 219 and 182; 40 276 and 241; 20 at half width 159 and 131.  14 x 14 x 512 -> 512, us a launch: 64 images {2, 8, 1} 17.3, {1, 8, 1} 27;
// 16 images {1, 4, 2} 9.9, {1, 8, 1} 11.7, {2, 8, 1} 16; 8 images {1, 2, 4} 8.2, {1, 8, 1} 11.2.
struct TileForm {
  int tm, waves_n, wk;
};
TileForm tile_form(long long patches, int c, int n, int stride) {
  const int groups = n / 64;
  TileForm best{};
  double least = 1e30;
  for (const TileForm f : {TileForm{2, divisor(groups, 8), 1}, TileForm{1, divisor(groups, 8), 1}, TileForm{1, divisor(groups, 4), 2},
                           TileForm{1, divisor(groups, 2), 4}}) {
    if (c % (64 * f.wk) != 0) continue;
    const long long blocks = (patches + 4 * f.tm - 1) / (4 * f.tm) * (groups / f.waves_n), slots = 256 * (8 / (f.waves_n * f.wk));
    const double us = 2.3 * (double)((blocks + slots - 1) / slots) + (double)((blocks + 255) / 256) * c * (.011 * stride * f.tm + .93e-3 * f.waves_n);
    if (us < least) best = f, least = us;
  }
  return best;
}

}  // namespace

bool separable_tile_f16_supported(int batch, int h, int w, int c, int n, int stride, int oh, int ow, const void* x,
                                  const void* dw_w, const void* dw_b, const void* pw_w, const void* pw_b, const void* y) {
  const void* ptrs[] = {x, dw_w, dw_b, pw_w, pw_b, y};
  bool aligned = true;
  for (const void* p : ptrs) aligned = aligned && reinterpret_cast<uintptr_t>(p) % 16 == 0;
  const long long patches = (long long)batch * ((oh + 1) / 2) * ((ow + 3) / 4), x_bytes = (long long)batch * h * w * c * 2,
                  y_bytes = (long long)batch * oh * ow * n * 2;
  // output pixels (with the patches' padding) from which it is the faster: every workgroup of a tile's columns computes the
  // depthwise layer again, so few pixels of a deep layer are not worth it (8 x 7 x 7 x 1024 10.7 us, 4 x 10.4; 7 apart)
  const long long least = c <= 256 ? 1024 : c <= 512 ? 700 : 850;
  return aligned && (stride == 1 || stride == 2) && c % 64 == 0 && c <= 1024 && n % 64 == 0 && n <= 1024 &&
         x_bytes < (1ll << 31) && y_bytes < (1ll << 31) && patches < (1ll << 27) && h < 65536 && w < 65536 && 8 * patches >= least;
}

int launch_separable_tile_f16(const uint16_t* x, const uint16_t* dw_w, const uint16_t* dw_b, const uint16_t* packed,
                              const uint16_t* pw_b, uint16_t* y, int batch, int h, int w, int c, int n, int oh, int ow,
                              int stride, int pt, int pl, int dw_act, int pw_act, hipStream_t stream) {
  auto p = [](const uint16_t* q) { return reinterpret_cast<const half_t*>(q); };
  const int row_patches = (ow + 3) / 4, col_patches = (oh + 1) / 2, patches = batch * col_patches * row_patches;
  const TileBlockArgs g{p(x), p(dw_w), p(dw_b), p(packed), p(pw_b), reinterpret_cast<half_t*>(y), h, w, c, n, oh, ow, pt, pl,
                        row_patches, col_patches, patches, (unsigned)((long long)batch * h * w * c * 2),
                        (unsigned)((long long)batch * oh * ow * n * 2), dw_act, pw_act};
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

int launch_pack_filters_f16(int layers, const uint16_t* const* w, uint16_t* const* packed, const int* c, const int* n,
                            hipStream_t stream) {
  PackArgs g{};
  if (layers > kMaxLayers) return TFX_ERR_UNSUPPORTED;
  for (int i = 0; i < layers; ++i) {
    g.w[i] = reinterpret_cast<const half_t*>(w[i]);
    g.out[i] = reinterpret_cast<h8*>(packed[i]);
    g.c[i] = c[i], g.n[i] = n[i];
    g.first[i + 1] = g.first[i] + (c[i] / 16 * (n[i] / 64) + 3) / 4;
  }
  g.layers = layers;
  hipLaunchKernelGGL(pack_filters_kernel, dim3((unsigned)g.first[layers]), dim3(256), 0, stream, g);
  return check_launch();
}

}  // namespace tfx
