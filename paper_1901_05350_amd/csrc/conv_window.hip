// conv2d in fp32 with a filter of 3 or 5 columns on the bf16 matrix cores, operands split three ways (split.h), for outputs of
// many tiles: the input under a tile is split once, not once per filter tap.
//
// A workgroup computes 128 TM consecutive output pixels (of all images, row after row) x 64 columns.  It works through the
// channels 16 at a time.  The input rows under its pixels, with zeros where they leave the image, lie in LDS as the planes hi,
// mid, lo (32 bytes each and 16 of padding a pixel); every tap of the filter reads its operands from them at a constant
// distance.  The filter is split too: per step -- 16 channels of one filter row -- its operands are written to one of two LDS
// buffers, in their order, while the step before is multiplied.  Raw values of the next step (filter) and of the next channels
// (window) wait in registers.
//
// Precision: a matrix instruction rounds its whole accumulator, so a step starts from zero and is added to the sum at its end, and
// in it the small passes of a tap come before the hi hi pass of the tap before, while the accumulator is shorter: about
// sqrt(4 + steps / 2) roundings (3 columns) instead of sqrt(3 K / 16).  Error against float64, normal operands, 3 x 3, K = 144 / 1944:
// 0.72 / 1.43e-7; one chain of all steps 1.72 / 6.8e-7, gemm_direct.hip, which such shapes took before, 0.90 / 2.4e-7.  It costs 2 - 3 %
// (39 drawn shapes: 0.786 of the time without this kernel, one chain 0.769; 8 x 73 x 73 x 80 -> 192 65.9 -> 67.9 us).
#include "kernel_cost.h"
#include "split.h"
#include "ragged.h"

#include <type_traits>

namespace tfx {
namespace {

constexpr int kXcds = 8, kThreads = 512, kChannels = 16, kPixelBytes = 112, kWindowItems = 8;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct WindowConv {
  const float *x, *w, *bias;
  float* y;
  int N, H, W, Ci, fh, Co, OH, OW, sh, sw, pt, pl, act;
  int M, tiles_n, total, cols, half, slots;  // columns of the window (half: where the odd ones begin if sw is 2), its most pixels
  unsigned x_bytes, w_bytes;
  FastDiv by_ow, by_oh, by_cols, by_rows;  // rows: of a whole image's window
};

// (fh rows per output row; LDS: window, then two filter buffers)
template <int TM, int FW, bool DOUBLE>
__global__ __launch_bounds__(kThreads, 2) void conv_window_kernel(WindowConv g) {
  constexpr int BM = 128 * TM, BN = 64, FITEMS = (FW * 128 + kThreads - 1) / kThreads, kFilter = FW * 6 * 1024;
  extern __shared__ __align__(16) char lds[];
  const int window_bytes = g.slots * kPixelBytes;
  char* const filter = lds + (DOUBLE ? 2 : 1) * window_bytes;

  const int bid = blockIdx.x;
  const int q8 = g.total / kXcds, rem = g.total % kXcds, xcd = bid % kXcds;
  const int vid = xcd * q8 + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int m0 = vid / g.tiles_n * BM, n0 = vid % g.tiles_n * BN;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, li = lane % 32, h = lane / 32;
  const int wm0 = wave / 2 * 32 * TM, wn = wave % 2;

  // window rows: those of the first image from its first output row here on, then whole images'
  const int g0 = (int)div_by((unsigned)m0, g.by_ow), first = (int)div_by((unsigned)g0, g.by_oh), oh0 = g0 - first * g.OH;
  const int rows0 = (g.OH - 1 - oh0) * g.sh + g.fh, rows = (int)g.by_rows.d;
  const int last = (int)div_by((unsigned)(min(m0 + BM, g.M) - 1), g.by_ow), last_image = (int)div_by((unsigned)last, g.by_oh);
  auto window_row = [&](int image, int oh) {
    return image == first ? (oh - oh0) * g.sh : rows0 + (image - first - 1) * rows + oh * g.sh;
  };
  const int used = (window_row(last_image, last - last_image * g.OH) + g.fh) * g.cols;

  // this lane's pixels
  int at[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = min(m0 + wm0 + 32 * i + li, g.M - 1), out = (int)div_by((unsigned)row, g.by_ow), ow = row - out * g.OW;
    const int image = (int)div_by((unsigned)out, g.by_oh);
    at[i] = (window_row(image, out - image * g.OH) * g.cols + (g.sw == 2 ? ow : ow * g.sw)) * kPixelBytes + 16 * h;
  }
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.x), 0, (int)g.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.w), 0, (int)g.w_bytes, 0x00020000);

  // This thread's pieces of the window: 4 channels of a pixel each, byte offset in x at channel 0, or past the end (zeros).
  constexpr unsigned kNone = 0x80000000u;
  unsigned from[kWindowItems];
#pragma unroll
  for (int i = 0; i < kWindowItems; ++i) {
    const int e = tid + i * kThreads, slot = e / 4, row = (int)div_by((unsigned)slot, g.by_cols), c = slot - row * g.cols;
    int image = first, ih = oh0 * g.sh - g.pt + row;
    if (row >= rows0) {
      const int image_after = (int)div_by((unsigned)(row - rows0), g.by_rows);
      image = first + 1 + image_after;
      ih = row - rows0 - image_after * rows - g.pt;
    }
    const int iw = (g.sw == 2 ? (c < g.half ? 2 * c : 2 * (c - g.half) + 1) : c) - g.pl;
    const bool ok = slot < used && image < g.N && ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
    from[i] = ok ? 4u * (((unsigned)(image * g.H + ih) * g.W + iw) * g.Ci + 4 * (e % 4)) : kNone;
  }
  char* const to = lds + tid / 4 * kPixelBytes + 8 * (tid % 4);  // piece i: 128 i pixels on
  floatx4 raw[kWindowItems];
  auto load_window = [&](int c0) __attribute__((always_inline)) {
    const unsigned none = c0 + 4 * (tid % 4) < g.Ci ? 0u : kNone;  // (Ci is a multiple of 4; the last 16 channels may be fewer)
#pragma unroll
    for (int i = 0; i < kWindowItems; ++i)
      if (i * kThreads < 4 * used) raw[i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(xr, from[i] | none, 4 * c0, 0));
  };
  SplitGuard guard;
  auto store_window = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kWindowItems; ++i)
      if (tid + i * kThreads < 4 * used) {
        splitx4 part[kParts];
        guard.split(raw[i], part);
#pragma unroll
        for (int p = 0; p < kParts; ++p)
          *reinterpret_cast<splitx4*>(to + buf * window_bytes + i * (kThreads / 4) * kPixelBytes + 32 * p) = part[p];
      }
  };
  // the filter's operands of a step: item (tap, column block, lane) has 8 channels of a column
  floatx4 wraw[FITEMS][2];
  unsigned wfrom[FITEMS];
#pragma unroll
  for (int f = 0; f < FITEMS; ++f) {
    const int item = tid + f * kThreads, kw = item / 128, col = n0 + item % 128 / 64 * 32 + li;
    wfrom[f] = item < FW * 128 && col < g.Co ? 4u * ((unsigned)(kw * g.Ci + 8 * h) * g.Co + col) : kNone;
  }
  auto load_filter = [&](int kh, int c0) __attribute__((always_inline)) {
    const unsigned step = 4u * ((unsigned)(kh * FW * g.Ci + c0) * g.Co);
    const bool whole = c0 + kChannels <= g.Ci;
#pragma unroll
    for (int f = 0; f < FITEMS; ++f)
      if (f * kThreads + 64 * wave < FW * 128) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const unsigned none = whole || c0 + 8 * h + e < g.Ci ? 0u : kNone;
          wraw[f][e / 4][e % 4] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wr, wfrom[f] | none, step + 4u * e * g.Co, 0));
        }
      }
  };
  auto store_filter = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < FITEMS; ++f)
      if (f * kThreads + 64 * wave < FW * 128) {
        const int item = tid + f * kThreads;
        splitx4 part[2][kParts];
        guard.split(wraw[f][0], part[0]);
        guard.split(wraw[f][1], part[1]);
#pragma unroll
        for (int p = 0; p < kParts; ++p)
          *reinterpret_cast<u32x4*>(filter + buf * kFilter + (item / 64 * kParts + p) * 1024 + lane * 16) =
              u32x4{part[0][p][0], part[0][p][1], part[1][p][0], part[1][p][1]};
      }
  };

  floatx16 sum[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[i][v] = 0.f;
  const int col = n0 + 32 * wn + li;
  const float bv = g.bias != nullptr && col < g.Co ? g.bias[col] : 0.f;

  const int chunks = (g.Ci + kChannels - 1) / kChannels, steps = chunks * g.fh;
  load_window(0);
  load_filter(0, 0);
  store_window(0);
  store_filter(0);
  if (chunks > 1) load_window(kChannels);
  if (steps > 1) load_filter(g.fh > 1 ? 1 : 0, g.fh > 1 ? 0 : kChannels);
  __syncthreads();

  bf16x8 fa[2][TM][kParts], fb[2][kParts];
  // parts [p0, p1) of a tap's operands
  auto read_a = [&](const char* window, int kh, int kw, int set, int p0, int p1) __attribute__((always_inline)) {
    const char* const tap = window + (kh * g.cols + (g.sw == 2 ? kw / 2 + (kw % 2 ? g.half : 0) : kw)) * kPixelBytes;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int p = p0; p < p1; ++p) fa[set][i][p] = *reinterpret_cast<const bf16x8*>(tap + at[i] + 32 * p);
  };
  auto read_b = [&](int buf, int kw, int set, int p0, int p1) __attribute__((always_inline)) {
    const char* const fbuf = filter + buf * kFilter + wn * kParts * 1024 + lane * 16;
#pragma unroll
    for (int p = p0; p < p1; ++p) fb[set][p] = *reinterpret_cast<const bf16x8*>(fbuf + (2 * kw * kParts + p) * 1024);
  };
  read_a(lds, 0, 0, 0, 0, kParts);
  read_b(0, 0, 0, 0, kParts);
  // One step; PAR: set of operand registers that its first tap has (FW is odd, so they alternate).  A step's first operands
  // from the window are read ahead of the barrier before it (with one window buffer not the first step's of a chunk).
  int kh = 0, c0 = 0;
  auto multiply = [&](int s, auto par) __attribute__((always_inline)) {
    constexpr int PAR = decltype(par)::value;
    const int wbuf = DOUBLE ? c0 / kChannels & 1 : 0;
    const char* const window = lds + wbuf * window_bytes;
    int kh1 = kh + 1, c1 = c0;  // the next step
    if (kh1 == g.fh) kh1 = 0, c1 += kChannels;
    int kh2 = kh1 + 1, c2 = c1;  // and the one after it
    if (kh2 == g.fh) kh2 = 0, c2 += kChannels;
    const bool more = s + 1 < steps, turn = more && kh1 == 0;  // the next step is one of the next channels
    floatx16 acc[TM];  // of this step
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    // Of the next tap's operands: the parts that are read ahead of this tap's products.  With 64 rows and 5 columns there are no
    // registers for three high parts, and it is read behind them.
    constexpr int kFirst = TM == 2 && FW == 5 ? 1 : 0;
    bf16x8 ha[TM], hb;  // high parts of the tap before
    auto high = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ha[i], hb, acc[i], 0, 0, 0);
    };
#pragma unroll
    for (int kw = 0; kw < FW; ++kw) {
      const int set = (PAR + kw) & 1;
      auto ahead = [&](int p0, int p1) __attribute__((always_inline)) {
        if (kw + 1 < FW) {
          read_a(window, kh, kw + 1, set ^ 1, p0, p1);
          read_b(s & 1, kw + 1, set ^ 1, p0, p1);
        } else if (more && (DOUBLE || !turn)) {
          read_a(turn ? lds + (wbuf ^ 1) * window_bytes : window, kh1, 0, set ^ 1, p0, p1);
        }
      };
      ahead(kFirst, kParts);
      if (kw == FW / 2 && more) {
        store_filter((s + 1) & 1);
        if (s + 2 < steps) load_filter(kh2, c2);
      }
      if (DOUBLE && kw == 0 && kh == 0 && c0 + kChannels < g.Ci) {  // (fh > 1: a barrier lies before the next channels' first read)
        store_window(wbuf ^ 1);
        if (c0 + 2 * kChannels < g.Ci) load_window(c0 + 2 * kChannels);
      }
#pragma unroll
      for (int x = 0; x < kSplitPasses - 1; ++x)
#pragma unroll
        for (int i = 0; i < TM; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i][split_pass_a(x)], fb[set][split_pass_b(x)], acc[i], 0, 0, 0);
      if (kw > 0) high();
      ahead(0, kFirst);
#pragma unroll
      for (int i = 0; i < TM; ++i) ha[i] = fa[set][i][0];
      hb = fb[set][0];
      if (kw + 1 == FW) high();
    }
    __syncthreads();
    if (!DOUBLE && turn) {
      store_window(0);
      if (c1 + kChannels < g.Ci) load_window(c1 + kChannels);
      __syncthreads();
      read_a(window, 0, 0, PAR ^ 1, 0, kParts);
    }
    if (more) read_b((s + 1) & 1, 0, PAR ^ 1, 0, kParts);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[i][v] += acc[i][v];
    kh = kh1, c0 = c1;
  };
  for (int s = 0; s < steps; s += 2) {
    multiply(s, std::integral_constant<int, 0>{});
    if (s + 1 < steps) multiply(s + 1, std::integral_constant<int, 1>{});
  }

  // (here and not in the conditional stores, each of which would wait for the bias and so for the store before it)
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[i][v] += bv;
  const ActClamp clamp = make_act(g.act);
  if (col < g.Co) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = m0 + wm0 + 32 * i + 8 * (v / 4) + 4 * h + v % 4;
        if (row < g.M) g.y[(size_t)row * g.Co + col] = apply_act(sum[i][v], clamp);
      }
  }
  // Values that the split does not carry (split.h): results that are Inf or NaN, and small ones if it lost bits of an operand
  // of this workgroup, once more with the fp32 instructions, over what was stored.
  unsigned most = 0;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) see_result(most, sum[i][v]);
  bool again = overflowed(most);
  float limit = 0.f;
  if (__syncthreads_or(guard.lost())) {
    limit = __syncthreads_or(guard.large()) ? INFINITY : small_limit(g.Ci * g.fh * FW);
    float least = INFINITY;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) least = fminf(least, fabsf(sum[i][v]));
    again = again || least < limit;
  }
  auto wanted = [&](float r) __attribute__((always_inline)) { return !__builtin_isfinite(r) || fabsf(r) < limit; };
  if (__builtin_amdgcn_ballot_w64(again) != 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      bool any = false;
#pragma unroll
      for (int v = 0; v < 16; ++v) any = any || wanted(sum[i][v]);
      if (__builtin_amdgcn_ballot_w64(any) == 0) continue;
      const int row = min(m0 + wm0 + 32 * i + li, g.M - 1), t = row / g.OW, image = t / g.OH;
      const int ih0 = (t - image * g.OH) * g.sh - g.pt, iw0 = (row - t * g.OW) * g.sw - g.pl, wc = min(col, g.Co - 1);
      floatx16 exact;
#pragma unroll
      for (int v = 0; v < 16; ++v) exact[v] = 0.f;
#pragma unroll 1
      for (int tap = 0; tap < g.fh * FW; ++tap) {
        const int ih = ih0 + tap / FW, iw = iw0 + tap % FW;
        const bool inside = ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
        const float* const xp = g.x + (inside ? (((size_t)image * g.H + ih) * g.W + iw) * g.Ci : 0);
        const float* const wp = g.w + (size_t)tap * g.Ci * g.Co + wc;
#pragma unroll 1
        for (int c = 2 * h; c - 2 * h < g.Ci; c += 4)  // (Ci is a multiple of 4)
#pragma unroll
          for (int e = 0; e < 2; ++e)
            exact = __builtin_amdgcn_mfma_f32_32x32x2f32(inside ? xp[c + e] : 0.f, wp[(size_t)(c + e) * g.Co], exact, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int out = m0 + wm0 + 32 * i + 8 * (v / 4) + 4 * h + v % 4;
        if (wanted(sum[i][v]) && out < g.M && col < g.Co) g.y[(size_t)out * g.Co + col] = apply_act(exact[v] + bv, clamp);
      }
    }
  }
}

constexpr int kLdsBytes = 159 * 1024;
int window_lds(int slots, int fw, bool twice) { return (twice ? 2 : 1) * slots * kPixelBytes + 2 * fw * 6 * 1024; }

template <int TM, int FW, bool DOUBLE>
int launch_window(const WindowConv& args, hipStream_t stream) {
  WindowConv g = args;
  auto kern = conv_window_kernel<TM, FW, DOUBLE>;
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), kLdsBytes, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  g.tiles_n = (g.Co + 63) / 64;
  g.total = (g.M + 128 * TM - 1) / (128 * TM) * g.tiles_n;
  hipLaunchKernelGGL(kern, dim3((unsigned)g.total), dim3(kThreads), (size_t)window_lds(g.slots, FW, DOUBLE), stream, g);
  return check_launch();
}

// pixels of the window under `pixels` consecutive output pixels, at most
long long window_slots(int pixels, int fh, int fw, int oh, int ow, int sh, int sw) {
  const long long out_rows = (pixels + ow - 2) / ow + 1, images = (out_rows + oh - 2) / oh + 1;
  const long long most = (out_rows - 1) * sh + fh + (images - 1) * (fh > sh ? fh - sh : 0);
  return most * ((ow - 1) * sw + fw);
}
bool window_fits(int tm, int fh, int fw, int oh, int ow, int sh, int sw) {
  const long long slots = window_slots(128 * tm, fh, fw, oh, ow, sh, sw);
  return slots <= kWindowItems * kThreads / 4 && window_lds((int)slots, fw, false) <= kLdsBytes;
}

}  // namespace

// The model's constants, as kernel_cost.h's, were fitted to 274 runs of 151 convolutions (0.3 - 60 GFLOP, 8 ... 512 channels, 3 x 3
// and 5 x 5, strides 1 and 2, 7 ... 112 pixels wide); rms error 4 %.  A workgroup has a CU to itself.
int conv2d_window_form(int n, int h, int wd, int ci, int fh, int fw, int co, int oh, int ow, int sh, int sw, double* us) {
  *us = 1e30;
  if ((fw != 3 && fw != 5) || ci % 4 != 0 || sw > 2) return 0;
  const long long m = (long long)n * oh * ow, x_bytes = (long long)n * h * wd * ci * 4, w_bytes = (long long)fh * fw * ci * co * 4;
  if (m > 0x7fffff00LL || x_bytes >= (1ll << 31) || w_bytes >= (1ll << 31)) return 0;
  int form = 0;
  for (int tm = 1; tm <= 2; ++tm) {
    if (!window_fits(tm, fh, fw, oh, ow, sh, sw)) continue;
    const double slots = (double)window_slots(128 * tm, fh, fw, oh, ow, sh, sw), chunks = (ci + kChannels - 1) / kChannels;
    const double r = (double)((m + 128 * tm - 1) / (128 * tm) * ((co + 63) / 64)) / 256., rounds = r <= 4. ? (double)(long long)(r + .999999) : r + .5;
    const double t = tm == 1 ? 1.9 + rounds * (3.3 + chunks * (fh * (.35 + .224 * fw) + .00102 * slots))
                             : 1.1 + rounds * (5.8 + chunks * (fh * (.11 + .439 * fw) + .00103 * slots));
    if (t < *us) *us = t, form = tm;
  }
  return form;
}

int launch_conv2d_window(const float* x, const float* w, const float* bias, float* y, int n, int h, int wd, int ci, int fh, int fw,
                         int co, int oh, int ow, int sh, int sw, int pt, int pl, int act, hipStream_t stream, int form) {
  WindowConv g{};
  g.x = x, g.w = w, g.bias = bias, g.y = y;
  g.N = n, g.H = h, g.W = wd, g.Ci = ci, g.fh = fh, g.Co = co, g.OH = oh, g.OW = ow, g.sh = sh, g.sw = sw, g.pt = pt, g.pl = pl, g.act = act;
  g.M = n * oh * ow;
  g.cols = (ow - 1) * sw + fw, g.half = (g.cols + 1) / 2, g.slots = (int)window_slots(128 * form, fh, fw, oh, ow, sh, sw);
  g.x_bytes = (unsigned)((long long)n * h * wd * ci * 4), g.w_bytes = (unsigned)((long long)fh * fw * ci * co * 4);
  g.by_ow = fast_div((unsigned)ow), g.by_oh = fast_div((unsigned)oh), g.by_cols = fast_div((unsigned)g.cols);
  g.by_rows = fast_div((unsigned)((oh - 1) * sh + fh));
  const bool twice = fh > 1 && window_lds(g.slots, fw, true) <= kLdsBytes;
#define TFX_WINDOW(TM, FW) \
  if (form == TM && fw == FW) return twice ? launch_window<TM, FW, true>(g, stream) : launch_window<TM, FW, false>(g, stream);
  TFX_WINDOW(1, 3)
  TFX_WINDOW(2, 3)
  TFX_WINDOW(1, 5)
  TFX_WINDOW(2, 5)
#undef TFX_WINDOW
  return TFX_ERR_UNSUPPORTED;
}

}  // namespace tfx
