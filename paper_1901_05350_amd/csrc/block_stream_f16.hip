// A depthwise-separable block of the Section 3.9 network at large batch in one launch, on 16-bit float storage
// (Section 4.1):  y = half(relu6(pointwise(half(relu6(depthwise3x3(x) + dw_b))) + pw_b)),  stride 1 or 2, SAME.
// The fp32 kernel of block_stream.hip with the operand layout of pointwise_f16.hip: the pointwise filter is the stationary
// operand in LDS (stream_f16.h), a unit is a patch of 2 or 4 x 8 output pixels of one image = one or two
// v_mfma_f32_16x16x32_f16 slabs of 2 x 8 pixels, and the wavefront copies the patch's input window, 32 or 64 channels at a
// time, into its own piece of LDS.  The next channels of the window (and, before the pointwise layer, the first ones of the
// next unit) are on their way from memory into registers meanwhile.
//
// The depthwise layer runs on the matrix cores, as products with diagonal matrices: two taps x 16 channels are the 32 of a
// contraction, lane (li, q) supplying channels 8 (q % 2) ... + 7 of tap q / 2 of the pair at slab pixel (li / 8, li % 8); of the
// filter, the other operand, each row has but its own two weights, a dword a lane in LDS.  It is accumulated in fp32, clamped and
// rounded to binary16 as the depthwise kernel rounds what it stores, and comes as the pointwise product's operand: lane (li, q)
// holds channels 4 q ... + 3 of the two groups of a k-step, in which order the filter is put into LDS.  A zero times a NaN is a
// NaN in 15 other channels, but all channels of the pixel meet in every output of the pointwise layer, so the same outputs are
// NaN; the map itself, behind a relu6, has no infinities.
//
// Bound by LDS and issue, with two or three wavefronts a SIMD: on the vector units a slab and 32 channels took 72 mixed multiply-
// adds of 4.3 cycles and 18 reads of LDS, as products they take 10 of 16 cycles and 9 or 10 reads (and 10 dwords for all slabs).
// 64 images: 56 x 56 x 128 -> 128 33.0 us -> 26.0 (102 MB, 20 us at the rate of a large copy), 112 x 112 x 64 -> 128 at stride 2
// 37.3 -> 29.5 (154 MB, 30), 56 x 56 x 128 -> 256 at stride 2 21.7 -> 20.6 (77 MB, 15).
#include "stream_f16.h"

namespace tfx {
namespace {

using namespace f16s;

constexpr int kPatchW = 8;  // a unit is PH x 8 output pixels: PH / 2 slabs of 2 x 8

// The layers' units and workgroups: as many wavefronts as their windows leave room for in LDS and three or four a SIMD in the
// registers.  Measured, 64 images (us): 128 -> 128: {4, 32, 768, 64} 26.0, with 128 columns a pass 26.5, of 64 channels and 512
// threads 27.5, {4, 32, 1024, 32} 26.8.  64 -> 128: {2, 64, 640} 29.5, 512 threads 29.9, {2, 32, 512} 32.1, {4, 32, 512} 36.7.
// 128 -> 256: {2, 32, 704} 20.6, 512 threads 22.3.  96 -> 96: {4, 32, 1024, 96} 19.5, 768 threads 20.2 (two launches 51).
// 96 -> 192: {2, 32, 768} 16.9, 512 threads 17.9 (33).  32 -> 64: {4, 32, 768} 16.1, {2, 32, 768} 17.5 (25).
struct WindowForm16 {
  int rows, channels, threads, columns;  // of a unit; of a chunk of its window; of a workgroup; of a pass over the operands
};
template <int K, int N>
constexpr WindowForm16 window_form() {
  if (K == 128) return N == 128 ? WindowForm16{4, 32, 768, 64} : WindowForm16{2, 32, 704, 128};
  if (K == 96) return N == 96 ? WindowForm16{4, 32, 1024, 96} : WindowForm16{2, 32, 768, 96};
  if (K == 64) return WindowForm16{2, 64, 640, 128};
  return WindowForm16{4, 32, 768, 64};
}

struct WindowBlockGeom16 {
  int H, W, OH, OW, pt, pl;
  int tiles_c, tiles_r;  // patches per output row and column
  unsigned x_bytes;
};

// LDS layout of a window chunk of CC channels in 16-byte pieces (8 channels each): pixel stride PS >= CC / 8 and
// row stride RS >= WW * PS, the least ones for which the tap read of a wavefront (pixel (li / 8, li % 8) * S plus a
// constant, piece q) has no bank conflict.
template <int S, int CC, int PH>
struct WindowLayout16 {
  static constexpr int WH = (PH - 1) * S + 3, WW = (kPatchW - 1) * S + 3, QC = CC / 8;
  struct Piece {
    int ps, rs;
    constexpr int operator()(int li, int q) const { return (li / 8) * S * rs + (li % 8) * S * ps + q; }
  };
  static constexpr int pixel_stride() {
    for (int ps = QC;; ++ps)
      for (int rs = WW * ps; rs < WW * ps + 32; ++rs)
        if (conflict_free(Piece{ps, rs})) return ps;
  }
  static constexpr int PS = pixel_stride();
  static constexpr int row_stride() {
    for (int rs = WW * PS;; ++rs)
      if (conflict_free(Piece{PS, rs})) return rs;
  }
  static constexpr int RS = row_stride();
  static constexpr int kHalfs = WH * RS * 8;
  static constexpr int kPieces = WH * WW * QC, kLoads = (kPieces + 63) / 64;
};

// The nine taps (row-major) in pairs: columns 0 and 1 of each row, column 2 of rows 0 and 1, the ninth alone.
constexpr int kTapPairs = 5;
__device__ __forceinline__ int tap_of(int pair, int second) {
  return pair < 3 ? 3 * pair + second : pair == 3 ? 2 + 3 * second : 8;
}

template <int K, int N, int S>
__global__ __launch_bounds__((window_form<K, N>().threads)) void separable_window_f16_kernel(const half_t* __restrict__ x,
                                                                        const half_t* __restrict__ dw_w,
                                                                        const half_t* __restrict__ dw_b,
                                                                        const half_t* __restrict__ pw_w,
                                                                        const half_t* __restrict__ pw_b,
                                                                        half_t* __restrict__ y, WindowBlockGeom16 g,
                                                                        int units, int dw_act, int pw_act) {
  constexpr WindowForm16 F = window_form<K, N>();
  constexpr int kThreads = F.threads, kWaves = kThreads / 64, CC = F.channels, PH = F.rows, SL = PH / 2;  // slabs per unit
  using WL = WindowLayout16<S, CC, PH>;
  using Stage = FilterStage<K, N, kThreads>;
  constexpr int KS = K / 32, NB = N / 16, LD = Stage::LD, CH = K / CC, SPC = CC / 32;  // k-steps, blocks, chunks, steps per chunk
  constexpr int PS = WL::PS, RS = WL::RS, WW = WL::WW, LI = WL::kLoads, QC = WL::QC;
  constexpr int NBP = F.columns / 16, PASSES = NB / NBP;  // 16-channel blocks per pass over the unit's operands
  static_assert(K % CC == 0 && N % 32 == 0 && NB % NBP == 0 && NBP % 2 == 0 && N <= kThreads && K <= kThreads, "shape");
  // pointwise filter [N][LD] halfs, its bias (N floats, in the filter's row order), depthwise filter [tap pair][K / 16][lane]
  // (a half in its half of a dword), its bias (K floats), then one window per wavefront
  extern __shared__ __align__(16) half_t wl[];
  float* const pwb_l = reinterpret_cast<float*>(wl + N * LD);
  unsigned* const dww_l = reinterpret_cast<unsigned*>(pwb_l + N);
  float* const dwb_l = reinterpret_cast<float*>(dww_l + kTapPairs * K * 4);
  half_t* const win = reinterpret_cast<half_t*>(dwb_l + K) + (threadIdx.x / 64) * WL::kHalfs;
  __shared__ int next_unit;

  const int tid = threadIdx.x;
  const int lane = tid % 64, li = lane % 16, q = lane / 16;
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(x), 0, (int)g.x_bytes, 0x00020000);
  const int u0 = (int)((long long)units * blockIdx.x / gridDim.x);
  const int u1 = (int)((long long)units * (blockIdx.x + 1) / gridDim.x);

  // This lane's pieces of a window chunk: piece e = lane + 64 i is 8 channels (cq) of window pixel (wr, wc).
  int wrc[LI], goff[LI], loff[LI];
#pragma unroll
  for (int i = 0; i < LI; ++i) {
    const int e = lane + 64 * i, p = e / QC, cq = e % QC, wr = p / WW, wc = p % WW;
    wrc[i] = wr | wc << 8 | (e < WL::kPieces ? 1 << 16 : 0);  // bit 16: the piece exists
    goff[i] = ((wr * g.W + wc) * K + 8 * cq) * 2;
    loff[i] = (wr * RS + wc * PS + cq) * 8;
  }
  // a unit's place: image, patch, and the byte offset of window pixel (0, 0), channel 0 (may lie outside x)
  struct Place {
    int n, tr, tc, ih0, iw0, base;
  };
  auto place_of = [&](int unit) {
    Place p;
    p.tc = unit % g.tiles_c;
    const int t1 = unit / g.tiles_c;
    p.tr = t1 % g.tiles_r;
    p.n = t1 / g.tiles_r;
    p.ih0 = PH * p.tr * S - g.pt;
    p.iw0 = kPatchW * p.tc * S - g.pl;
    p.base = ((p.n * g.H + p.ih0) * g.W + p.iw0) * K * 2;
    return p;
  };
  // byte offsets of this lane's window pieces, channel 0; a piece outside the image (or of no unit) gets an offset
  // past the end of the buffer, from where the hardware returns 0
  struct Offsets {
    unsigned v[LI];
  };
  auto offsets_of = [&](const Place& p, bool live) {
    Offsets o;
#pragma unroll
    for (int i = 0; i < LI; ++i) {
      const int ih = p.ih0 + (wrc[i] & 0xff), iw = p.iw0 + ((wrc[i] >> 8) & 0xff);
      const bool in = live & (wrc[i] >> 16 != 0) & ((unsigned)ih < (unsigned)g.H) & ((unsigned)iw < (unsigned)g.W);
      o.v[i] = in ? (unsigned)(p.base + goff[i]) : 0x80000000u;
    }
    return o;
  };
  u32x4 wreg[LI];  // window pieces of one chunk
  auto load_chunk = [&](const Offsets& o, int ch) {
#pragma unroll
    for (int i = 0; i < LI; ++i) wreg[i] = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)o.v[i], CC * 2 * ch, 0);
  };

  // The filters' loads first, then the first chunk of the wavefront's first unit (fixed; the rest are handed out
  // by the counter): all in flight while the pointwise filter is transposed.
  Stage stage;
  stage.fetch(pw_w, tid);
  constexpr int DW = kTapPairs * K * 4, DWI = (DW + kThreads - 1) / kThreads;
  unsigned short dwv[DWI];
#pragma unroll
  for (int i = 0; i < DWI; ++i) {
    const int e = tid + i * kThreads < DW ? tid + i * kThreads : 0, eq = e % 64 / 16;
    dwv[i] = reinterpret_cast<const unsigned short*>(dw_w)[tap_of(e / (4 * K), eq / 2) * K + e / 64 % (K / 16) * 16 + e % 16];
  }
  const half_t pwb = (pw_b ? pw_b : pw_w)[tid < N ? tid : 0];
  const half_t dwb = (dw_b ? dw_b : pw_w)[tid < K ? tid : 0];
  if (tid == 0) next_unit = kWaves;
  int cur = u0 + __builtin_amdgcn_readfirstlane(tid / 64);
  Place pc = place_of(cur < u1 ? cur : u0);
  Offsets oc = offsets_of(pc, cur < u1);
  load_chunk(oc, 0);
  stage.template store<true>(wl, tid);
#pragma unroll
  for (int i = 0; i < DWI; ++i) {
    const int e = tid + i * kThreads, eli = e % 16, eq = e % 64 / 16, pair = e / (4 * K);
    const bool mine = eli / 8 == eq % 2 && (pair < kTapPairs - 1 || eq < 2);
    if (e < DW) dww_l[e] = mine ? (unsigned)dwv[i] << 16 * (eli % 2) : 0u;
  }
  if (tid < N) pwb_l[rho(tid)] = pw_b ? (float)pwb : 0.f;
  if (tid < K) dwb_l[tid] = dw_b ? (float)dwb : 0.f;
  __syncthreads();

  const ActClamp dw_clamp = make_act(dw_act), pw_clamp = make_act(pw_act);
  // where this lane's taps start in a window: pixel (li / 8, li % 8) * S of slab 0, piece q % 2; the second of a pair of taps is
  // the next column's, the next row's, or (the ninth tap has no
  // partner) the same, so that a NaN outside a pixel's window meets none of its zeros
  const half_t* const tap0 = win + ((li / 8) * S * RS + (li % 8) * S * PS + q % 2) * 8;
  const half_t* const tap_col = tap0 + (q / 2) * PS * 8;
  const half_t* const tap_row = tap0 + ((q / 2) * RS + 2 * PS) * 8;
  unsigned own[4];  // the dword of an operand that holds channel li
#pragma unroll
  for (int e = 0; e < 4; ++e) own[e] = li % 8 / 2 == e ? ~0u : 0u;
  const half_t* const w_base = wl + li * LD + 8 * q;

  while (cur < u1) {
    int ticket = 0;
    if (lane == 0) ticket = atomicAdd(&next_unit, 1);
    // depthwise layer, chunk by chunk: the chunk in the registers goes to LDS, the next one is requested, and the operands of the
    // chunk's k-steps are formed for all slabs
    h8 a[SL][KS];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
#pragma unroll
      for (int i = 0; i < LI; ++i)
        if (LI * 64 == WL::kPieces || i + 1 < LI || lane + 64 * i < WL::kPieces)
          *reinterpret_cast<u32x4*>(win + loff[i]) = wreg[i];
      if (ch + 1 < CH) load_chunk(oc, ch + 1);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int sc = 0; sc < SPC; ++sc) {
        const int s = SPC * ch + sc;  // k-step: channels 32 s ... + 31, as two groups of 16
        f32x4 d[SL][2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x4 b = *reinterpret_cast<const f32x4*>(dwb_l + 32 * s + 16 * u + 4 * q);
#pragma unroll
          for (int sl = 0; sl < SL; ++sl) d[sl][u] = b;
#pragma unroll
          for (int i = 0; i < kTapPairs; ++i) {
            const unsigned wv = dww_l[(i * (K / 16) + 2 * s + u) * 64 + lane];
            const u32x4 diagonal = {wv & own[0], wv & own[1], wv & own[2], wv & own[3]};
#pragma unroll
            for (int sl = 0; sl < SL; ++sl) {
              const half_t* const at = i < 3 ? tap_col + i * RS * 8 : i == 3 ? tap_row : tap0 + (2 * RS + 2 * PS) * 8;
              const h8 xv = *reinterpret_cast<const h8*>(at + (2 * sl * S * RS + 4 * sc + 2 * u) * 8);
              d[sl][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, diagonal), xv, d[sl][u], 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int sl = 0; sl < SL; ++sl) {
          h8 o[1];
          activate_and_pack(d[sl], dw_clamp, o);
          a[sl][s] = o[0];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }

    // the first chunk of the next unit's window is requested before the MFMAs of this one
    const int nxt = u0 + __builtin_amdgcn_readfirstlane(ticket);
    const Place pn = place_of(nxt < u1 ? nxt : cur);
    const Offsets on = offsets_of(pn, nxt < u1);
    load_chunk(on, 0);

    // pointwise layer, F.columns output channels per pass over the operands and one k-step's filter fragments at a time
    // (the scheduling barriers keep the compiler from gathering all the reads in front, which does not fit the
    // registers); the accumulators start from the bias
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      f32x4 acc[SL][NBP];
#pragma unroll
      for (int j = 0; j < NBP; ++j) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(pwb_l + 16 * (NBP * p + j) + 4 * q);
#pragma unroll
        for (int sl = 0; sl < SL; ++sl) acc[sl][j] = b;
      }
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        h8 fw[NBP];
#pragma unroll
        for (int j = 0; j < NBP; ++j) fw[j] = *reinterpret_cast<const h8*>(w_base + 16 * (NBP * p + j) * LD + 32 * s);
#pragma unroll
        for (int j = 0; j < NBP; ++j)
#pragma unroll
          for (int sl = 0; sl < SL; ++sl)
            acc[sl][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fw[j], a[sl][s], acc[sl][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      // epilogue: activation, and one 16-byte store per lane, slab and 32 channels
      auto emit = [&](const f32x4 (&acc)[NBP], int slab) {
        const int oh = PH * pc.tr + 2 * slab + li / 8, ow = kPatchW * pc.tc + li % 8;
        half_t* const yp = y + ((size_t)(pc.n * g.OH + oh) * g.OW + ow) * N + 16 * NBP * p + 8 * q;
        h8 o[NBP / 2];
        activate_and_pack(acc, pw_clamp, o);
        if (oh < g.OH && ow < g.OW) {
#pragma unroll
          for (int m = 0; m < NBP / 2; ++m) *reinterpret_cast<h8*>(yp + 32 * m) = o[m];
        }
      };
#pragma unroll
      for (int sl = 0; sl < SL; ++sl) emit(acc[sl], sl);
    }
    cur = nxt;
    pc = pn;
    oc = on;
  }
}

template <int K, int N, int S>
int launch_cfg(const half_t* x, const half_t* dw_w, const half_t* dw_b, const half_t* pw_w, const half_t* pw_b, half_t* y, int batch,
               int h, int w, int oh, int ow, int pt, int pl, int dw_act, int pw_act, hipStream_t stream) {
  constexpr WindowForm16 F = window_form<K, N>();
  constexpr int kThreads = F.threads, kWaves = kThreads / 64;
  using WL = WindowLayout16<S, F.channels, F.rows>;
  const WindowBlockGeom16 g{h, w, oh, ow, pt, pl, (ow + kPatchW - 1) / kPatchW, (oh + F.rows - 1) / F.rows,
                            (unsigned)((long long)batch * h * w * K * 2)};
  const long long all = (long long)batch * g.tiles_c * g.tiles_r;
  if (all > 0x3fffffffLL) return TFX_ERR_UNSUPPORTED;
  const int units = (int)all;
  constexpr size_t lds_bytes = (size_t)N * filter_row_halfs(K) * 2 + N * 4 + kTapPairs * K * 16 + K * 4 + (size_t)kWaves * WL::kHalfs * 2;
  static_assert(lds_bytes + 64 <= 160 * 1024, "LDS budget per workgroup");
  auto kern = separable_window_f16_kernel<K, N, S>;
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds_bytes, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  // as many workgroups as are resident at once: each stages the filters once; fewer for less than 4 units each (16 images,
  // 56 x 56 x 128 -> 128: 131 of 12 units 15.0 us, 256 of 6 13.0)
  static std::atomic<int> resident{0};
  int per_cu = resident.load(std::memory_order_relaxed);
  if (per_cu == 0) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kThreads, lds_bytes) != hipSuccess || per_cu < 1)
      per_cu = 1;
    if (per_cu > 2) per_cu = 2;
    resident.store(per_cu, std::memory_order_relaxed);
  }
  int blocks = 256 * per_cu;
  if (blocks > (units + 3) / 4) blocks = (units + 3) / 4;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(kThreads), lds_bytes, stream, x, dw_w, dw_b, pw_w, pw_b, y, g, units,
                     dw_act, pw_act);
  return check_launch();
}

}  // namespace

// Blocks 2 - 4 (channels -> filters, stride) of the full-width network, 3 and 4 at 3/4 and 2, 4 and 6 at half width, many output pixels,
// 16-byte aligned operands, an input below 2^31 bytes.
bool separable_stream_f16_supported(int batch, int h, int w, int c, int n, int stride, int oh, int ow, const void* x,
                                    const void* dw_w, const void* dw_b, const void* pw_w, const void* pw_b,
                                    const void* y) {
  const bool shape = stride == 1 ? c == n && (c == 96 || c == 128) : n == 2 * c && (c == 32 || c == 64 || c == 96 || c == 128);
  const void* ptrs[] = {x, dw_w, dw_b, pw_w, pw_b, y};
  bool aligned = true;
  for (const void* p : ptrs) aligned = aligned && reinterpret_cast<uintptr_t>(p) % 16 == 0;
  const long long m = (long long)batch * oh * ow, x_bytes = (long long)batch * h * w * c * 2;
  // least output pixels from which the one launch beats the two kernels (measured on the network, per block)
  const long long least = n > 128 ? 6272 : 16384;
  return shape && aligned && m >= least && m <= 0x3fffffffLL && x_bytes < (1ll << 31);
}

int launch_separable_stream_f16(const uint16_t* x16, const uint16_t* dw_w16, const uint16_t* dw_b16, const uint16_t* pw_w16,
                                const uint16_t* pw_b16, uint16_t* y16, int batch, int h, int w, int c, int n, int oh,
                                int ow, int stride, int pt, int pl, int dw_act, int pw_act, hipStream_t stream) {
  const half_t* x = reinterpret_cast<const half_t*>(x16);
  const half_t* dw_w = reinterpret_cast<const half_t*>(dw_w16);
  const half_t* dw_b = reinterpret_cast<const half_t*>(dw_b16);
  const half_t* pw_w = reinterpret_cast<const half_t*>(pw_w16);
  const half_t* pw_b = reinterpret_cast<const half_t*>(pw_b16);
  half_t* y = reinterpret_cast<half_t*>(y16);
#define TFX_WINDOW_BLOCK16(C, NN, SS) \
  if (c == C && n == NN && stride == SS) \
    return launch_cfg<C, NN, SS>(x, dw_w, dw_b, pw_w, pw_b, y, batch, h, w, oh, ow, pt, pl, dw_act, pw_act, stream);
  TFX_WINDOW_BLOCK16(128, 128, 1)
  TFX_WINDOW_BLOCK16(64, 128, 2)
  TFX_WINDOW_BLOCK16(128, 256, 2)
  TFX_WINDOW_BLOCK16(96, 96, 1)
  TFX_WINDOW_BLOCK16(96, 192, 2)
  TFX_WINDOW_BLOCK16(32, 64, 2)
#undef TFX_WINDOW_BLOCK16
  return TFX_ERR_UNSUPPORTED;
}

}  // namespace tfx
