// A depthwise-separable block (depthwise 3x3 + bias + clamp, pointwise 1x1 + bias + clamp) on binary16 storage in one
// launch, for few pixels: the blocks of one image or a small batch (Section 4.1 storage format, the Section 3.9 network).
//
// A workgroup owns patches of 4 x 4 output pixels -- the 16 rows of a v_mfma_f32_16x16x32_f16 -- and 16 JN output columns,
// and splits the channels over its wavefronts, 32 STEPS to each.  A wavefront copies its channels of the input window under
// the patch and of the depthwise filter into an LDS region of its own (every element is fetched once per workgroup, with no
// barrier), computes the depthwise output of exactly the 8 channels per lane that are its matrix operand, rounded to binary16
// as the separate kernel rounds it, and multiplies it by its rows of the pointwise filter, which are loaded straight into
// registers before anything is waited for.  The wavefronts' partial tiles are added through LDS behind the only barrier.
//
// What bounds it is the latency of one launch: one round trip to memory, some 150 multiply-adds per lane and k-step
// pair, one exchange through LDS, the stores.  One image, 14 x 14 x 512 -> 512: 5.5 us, where the depthwise and the pointwise
// kernel took 3.6 + 4.6 and the gap between them; all 13 blocks of the network 69 us where the 26 kernels took 105 under the
// profiler.  The round trip for the arguments before that one is left out (PatchRest): the pass of one image 73.6 -> 67.5 - 70 us
// together with the order of its workgroups, of quarter width at 128 x 128 53 -> 48 - 52, of 16 images of quarter width 83 -> 78.
#include "ragged.h"
#include "stream_f16.h"

namespace tfx {
namespace {

using namespace f16s;

struct PatchBlockArgs {
  const half_t *x, *dw_w, *dw_b, *pw_w, *pw_b;
  half_t* y;
  int H, W, C, N, OH, OW, pt, pl;
  int patches, wk, wp;
  FastDiv row_patches, col_patches;
  unsigned x_bytes;
  int dw_act, pw_act;
};
// What the addresses of a workgroup's loads depend on comes in the 14 dwords of arguments that a wavefront finds in its scalar
// registers when it starts, packed for that: dimensions in halves, `form` with wk (5 bits), wp (3), pt, pl, the shifts of the two
// divisions (5 each) and 256 / wk rounded up (9).  The rest, for what it does with the loads, is read while they are under way.
//
// Workgroups go to the 8 XCDs in turn.  Either the patches come first in the grid, padded to a multiple of 8: the column slices of a
// patch then are on one XCD, whose L2 has its window, and every XCD reads the whole filter; or (bit 29) the column slices, and
// every XCD reads the windows and, of 8 slices, one.  Whichever is less to read: the pass of one image 71.2 us with patches first and
// 68.7, of 8 images 137.8 with slices first and 134.2, of 4 at half width and 192 x 192 66.7 and 63.4.
struct PatchRest {
  const half_t *dw_b, *pw_b;
  half_t* y;
  int OH, OW, dw_act, pw_act;
};

// The window in LDS: strides of a pixel and of a row of pixels in 16-byte pieces, such that the fragment read of a tap is
// free of bank conflicts.
template <int S, int STEPS>
struct PatchWindow {
  static constexpr int SIDE = 3 * S + 3, PIECES = 4 * STEPS;
  struct At {
    int px, row;
    constexpr int operator()(int li, int q) const { return li / 4 * S * row + li % 4 * S * px + q; }
  };
  struct Strides {
    int px, row;
  };
  static constexpr Strides find() {
    for (int px = PIECES;; ++px)
      for (int row = SIDE * px; row < SIDE * px + 16; ++row)
        if (conflict_free(At{px, row})) return {px, row};
  }
  static constexpr Strides kStrides = find();
  static constexpr int HALFS = 8 * SIDE * kStrides.row, FILTER = 9 * 32 * STEPS;
};

template <int JN>
struct HalfsOf {
  typedef _Float16 type __attribute__((ext_vector_type(JN)));
};

template <int S, int STEPS, int JN>
constexpr size_t patch_region_bytes() {
  typedef PatchWindow<S, STEPS> P;
  const size_t in = (size_t)(P::HALFS + P::FILTER) * sizeof(half_t), out = (size_t)256 * JN * sizeof(float);
  return in > out ? in : out;
}

template <int S, int STEPS, int JN>
__global__ __launch_bounds__(JN == 8 ? 512 : 1024) void separable_patch_f16_kernel(
    const half_t* x, const half_t* dw_w, const half_t* pw_w, unsigned x_bytes, unsigned map, unsigned channels, unsigned patches, unsigned by_row,
    unsigned by_col, unsigned per, unsigned form, PatchRest g) {
  typedef PatchWindow<S, STEPS> P;
  typedef typename HalfsOf<JN>::type hj;
  constexpr int LOADS = (P::SIDE * P::SIDE * P::PIECES + 63) / 64, FLOADS = (9 * P::PIECES + 63) / 64;
  extern __shared__ __align__(16) unsigned char lds[];

  const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int li = lane % 16, q = lane / 16;
  const int wk = (int)(form & 31), wp = (int)(form >> 5 & 7), pt = (int)(form >> 8 & 1), pl = (int)(form >> 9 & 1);
  const int H = (int)(map & 0xffff), W = (int)(map >> 16), C = (int)(channels & 0xffff), N = (int)(channels >> 16);
  const FastDiv row_patches{by_row, form >> 10 & 31, per & 0xffff}, col_patches{by_col, form >> 15 & 31, per >> 16};
  const int p = wave * (int)(form >> 20 & 511) >> 8, part = wave - p * wk;  // (wave / wk)
  const bool columns_first = (form >> 29 & 1) != 0;
  const int n0 = (int)(columns_first ? blockIdx.x : blockIdx.y) * 16 * JN, patch = (int)(columns_first ? blockIdx.y : blockIdx.x) * wp + p;
  const bool live = patch < (int)patches;
  if (patch - p >= (int)patches) return;  // (the grid is padded)
  const int strip = (int)div_by((unsigned)patch, row_patches), image = (int)div_by((unsigned)strip, col_patches);
  const int ow0 = 4 * (patch - strip * (int)row_patches.d), oh0 = 4 * (strip - image * (int)col_patches.d), c0 = 32 * STEPS * part;

  half_t* const window = reinterpret_cast<half_t*>(lds + wave * patch_region_bytes<S, STEPS, JN>());
  half_t* const taps = window + P::HALFS;

  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(x), 0, (int)x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t fr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(dw_w), 0, 18 * C, 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(pw_w), 0, 2 * C * N, 0x00020000);

  // Every load of the workgroup, before the first wait.  What lies outside the map, or past the last channel, has an offset
  // past the end and reads zeros.
  u32x4 win[LOADS], fil[FLOADS];
  const int piece = lane % P::PIECES, ch = c0 + 8 * piece;
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int px = (64 * i + lane) / P::PIECES, r = px / P::SIDE, c = px - r * P::SIDE;
    const int ih = oh0 * S - pt + r, iw = ow0 * S - pl + c;
    const bool ok = (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W && px < P::SIDE * P::SIDE && ch < C && live;
    const unsigned off = ok ? 2u * (((unsigned)(image * H + ih) * W + iw) * C + ch) : ~0u;
    win[i] = __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < FLOADS; ++i) {
    const int t = (64 * i + lane) / P::PIECES;
    fil[i] = __builtin_amdgcn_raw_buffer_load_b128(fr, ch < C && t < 9 ? 2u * (unsigned)(t * C + ch) : ~0u, 0, 0);
  }
  const int col = n0 + JN * li < N ? n0 + JN * li : 0;  // past the last column: read, never stored
  hj raw[STEPS][8];
#pragma unroll
  for (int s = 0; s < STEPS; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const unsigned off = 2u * ((unsigned)(c0 + 32 * s + 8 * q + i) * N + col);
      if constexpr (JN == 2) raw[s][i] = __builtin_bit_cast(hj, __builtin_amdgcn_raw_buffer_load_b32(wr, off, 0, 0));
      if constexpr (JN == 4) raw[s][i] = __builtin_bit_cast(hj, __builtin_amdgcn_raw_buffer_load_b64(wr, off, 0, 0));
      if constexpr (JN == 8) raw[s][i] = __builtin_bit_cast(hj, __builtin_amdgcn_raw_buffer_load_b128(wr, off, 0, 0));
    }
  const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(g.dw_b), 0, 2 * C, 0x00020000);
  u32x4 dwb[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) dwb[s] = __builtin_amdgcn_raw_buffer_load_b128(br, 2u * (unsigned)(c0 + 32 * s + 8 * q), 0, 0);
  const hj pwb = *reinterpret_cast<const hj*>(g.pw_b + col);

#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int px = (64 * i + lane) / P::PIECES, r = px / P::SIDE, c = px - r * P::SIDE;
    if (64 * (i + 1) <= P::SIDE * P::SIDE * P::PIECES || px < P::SIDE * P::SIDE)
      *reinterpret_cast<u32x4*>(window + 8 * (r * P::kStrides.row + c * P::kStrides.px + piece)) = win[i];
  }
#pragma unroll
  for (int i = 0; i < FLOADS; ++i)
    if (64 * (i + 1) <= 9 * P::PIECES || 64 * i + lane < 9 * P::PIECES) *reinterpret_cast<u32x4*>(taps + 8 * (64 * i + lane)) = fil[i];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();

  const ActClamp dw_clamp = make_act(g.dw_act), pw_clamp = make_act(g.pw_act);
  f32x4 acc[JN];
#pragma unroll
  for (int j = 0; j < JN; ++j) {
    const float b = part == 0 ? (float)pwb[j] : 0.f;
    acc[j] = f32x4{b, b, b, b};
  }
  const half_t* const mine = window + 8 * (li / 4 * S * P::kStrides.row + li % 4 * S * P::kStrides.px + q);
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    f32x4 d[2];
    const h8 b8 = __builtin_bit_cast(h8, dwb[s]);
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e / 4][e % 4] = (float)b8[e];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const h8 xt = *reinterpret_cast<const h8*>(mine + 8 * (t / 3 * P::kStrides.row + t % 3 * P::kStrides.px + 4 * s));
      const h8 wt = *reinterpret_cast<const h8*>(taps + 32 * STEPS * t + 32 * s + 8 * q);
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e / 4][e % 4] = fmaf((float)xt[e], (float)wt[e], d[e / 4][e % 4]);
    }
    h8 a[1];
    __builtin_amdgcn_sched_barrier(0);  // (else loads move down into the taps, one image 69.1 us instead of 68.4)
    activate_and_pack(d, dw_clamp, a);
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      h8 b;
#pragma unroll
      for (int i = 0; i < 8; ++i) b[i] = raw[s][i][j];
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[0], b, acc[j], 0, 0, 0);
    }
  }

  // lane (li, q) holds columns JN li ... of pixels (row q, column v) of the patch
  auto store = [&](int v, int l, int j, float s0, float s1) __attribute__((always_inline)) {
    typedef half_t h2 __attribute__((ext_vector_type(2)));
    const int oh = oh0 + l / 16, ow = ow0 + v, cn = n0 + JN * (l % 16) + j;
    const h2 o = {(half_t)apply_act(s0, pw_clamp), (half_t)apply_act(s1, pw_clamp)};
    if (live && oh < g.OH && ow < g.OW && cn < N)
      *reinterpret_cast<h2*>(g.y + ((size_t)(image * g.OH + oh) * g.OW + ow) * N + cn) = o;
  };
  if (wk == 1) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int j = 0; j < JN; j += 2) store(v, lane, j, acc[j][v], acc[j + 1][v]);
    return;
  }
  constexpr int REGION = (int)patch_region_bytes<S, STEPS, JN>();
  float* const sums = reinterpret_cast<float*>(lds + wave * REGION);  // [v][lane][JN], over the window, which is read
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int j = 0; j < JN; ++j) sums[(v * 64 + lane) * JN + j] = acc[j][v];
  __syncthreads();
  for (int u = 64 * part + lane; u < 128 * JN; u += 64 * wk) {
    float s0 = 0.f, s1 = 0.f;
    for (int w = 0; w < wk; ++w) {
      const float2 t = reinterpret_cast<const float2*>(lds + (p * wk + w) * REGION)[u];
      s0 += t.x, s1 += t.y;
    }
    const int v = u / (32 * JN), rest = u % (32 * JN);
    store(v, rest / (JN / 2), 2 * (rest % (JN / 2)), s0, s1);
  }
}

struct PatchForm {
  int steps, jn, wk, wp;
};

template <int S, int STEPS, int JN>
int launch_patch(const PatchBlockArgs& args, const PatchForm& f, hipStream_t stream) {
  PatchBlockArgs g = args;
  auto kern = separable_patch_f16_kernel<S, STEPS, JN>;
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), 160 * 1024, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  g.wk = f.wk, g.wp = f.wp;
  const unsigned slices = (unsigned)((g.N + 16 * JN - 1) / (16 * JN)), groups = (unsigned)((g.patches + f.wp - 1) / f.wp);
  const size_t lds_bytes = patch_region_bytes<S, STEPS, JN>() * f.wk * f.wp;
  const bool columns_first = g.x_bytes < 2u * g.C * g.N && groups < 1u << 15;
  const unsigned form = (unsigned)(f.wk | f.wp << 5 | g.pt << 8 | g.pl << 9) | g.row_patches.shift << 10 | g.col_patches.shift << 15 |
                        (256u + f.wk - 1) / f.wk << 20 | (columns_first ? 1u << 29 : 0u);
  const dim3 grid = columns_first ? dim3(slices, groups) : dim3((groups + 7) / 8 * 8, slices);
  hipLaunchKernelGGL(kern, grid, dim3(64u * f.wk * f.wp), lds_bytes, stream, g.x, g.dw_w, g.pw_w, g.x_bytes,
                     (unsigned)g.H | (unsigned)g.W << 16, (unsigned)(g.C | g.N << 16), (unsigned)g.patches, g.row_patches.mul, g.col_patches.mul,
                     g.row_patches.d | g.col_patches.d << 16, form, PatchRest{g.dw_b, g.pw_b, g.y, g.OH, g.OW, g.dw_act, g.pw_act});
  return check_launch();
}

// Wavefronts of up to 256 channels take 32 each (two k-steps of a wavefront cost more than another wavefront: 28 x 28 x 256
// -> 256 5.2 us against 4.6), of more 64, which leaves two workgroups a CU.  Columns of a workgroup: the most that give at
// least 180 workgroups, since all column slices of a patch compute its depthwise layer again (14 x 14 x 512 -> 512, one image:
// 32 columns 5.5 us, 64 5.7, 128 6.6; three images: 8.3, 7.8, 6.6).  Few channels: several patches to a workgroup.
PatchForm patch_form(long long patches, int c, int n) {
  PatchForm f;
  f.steps = c > 256 ? 2 : 1;
  f.wk = (c + 32 * f.steps - 1) / (32 * f.steps);
  f.wp = f.wk == 1 ? 4 : f.wk == 2 ? 2 : 1;
  auto blocks = [&](int jn) { return (patches + f.wp - 1) / f.wp * ((n + 16 * jn - 1) / (16 * jn)); };
  f.jn = f.wk <= 8 && n >= 128 && blocks(8) >= 180 ? 8 : n >= 64 && blocks(4) >= 180 ? 4 : 2;
  return f;
}

}  // namespace

bool separable_patch_f16_supported(int batch, int h, int w, int c, int n, int stride, int oh, int ow, const void* x,
                                   const void* dw_w, const void* dw_b, const void* pw_w, const void* pw_b, const void* y) {
  const void* ptrs[] = {x, dw_w, dw_b, pw_w, pw_b, y};
  bool aligned = true;
  for (const void* p : ptrs) aligned = aligned && reinterpret_cast<uintptr_t>(p) % 16 == 0;
  const long long patches = (long long)batch * ((oh + 3) / 4) * ((ow + 3) / 4), x_bytes = (long long)batch * h * w * c * 2;
  return aligned && (stride == 1 || stride == 2) && c % 8 == 0 && c <= (stride == 1 ? 1024 : 512) && n % 8 == 0 && n <= 1024 && x_bytes < (1ll << 31) &&
         patches < (1ll << 24) && h < 65536 && w < 65536;  // (stride 2: a wavefront's window is 13 KB, and 8 of them fit)
}

int launch_separable_patch_f16(const uint16_t* x, const uint16_t* dw_w, const uint16_t* dw_b, const uint16_t* pw_w,
                               const uint16_t* pw_b, uint16_t* y, int batch, int h, int w, int c, int n, int oh, int ow,
                               int stride, int pt, int pl, int dw_act, int pw_act, hipStream_t stream) {
  auto p = [](const uint16_t* q) { return reinterpret_cast<const half_t*>(q); };
  const int row_patches = (ow + 3) / 4, col_patches = (oh + 3) / 4, patches = batch * col_patches * row_patches;
  const PatchBlockArgs g{p(x), p(dw_w), p(dw_b), p(pw_w), p(pw_b), reinterpret_cast<half_t*>(y), h, w, c, n, oh, ow, pt, pl,
                         patches, 0, 0, fast_div((unsigned)row_patches), fast_div((unsigned)col_patches),
                         (unsigned)((long long)batch * h * w * c * 2), dw_act, pw_act};
  const PatchForm f = patch_form(patches, c, n);
#define TFX_PATCH(S, STEPS, JN) \
  if (stride == S && f.steps == STEPS && f.jn == JN) return launch_patch<S, STEPS, JN>(g, f, stream);
#define TFX_PATCHES(S) TFX_PATCH(S, 1, 2) TFX_PATCH(S, 1, 4) TFX_PATCH(S, 1, 8) TFX_PATCH(S, 2, 2) TFX_PATCH(S, 2, 4) TFX_PATCH(S, 2, 8)
  TFX_PATCHES(1)
  TFX_PATCHES(2)
#undef TFX_PATCHES
#undef TFX_PATCH
  return TFX_ERR_UNSUPPORTED;
}

}  // namespace tfx
