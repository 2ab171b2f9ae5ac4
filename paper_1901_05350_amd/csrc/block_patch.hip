// A depthwise-separable block (depthwise 3x3 + bias + clamp, pointwise 1x1 + bias + clamp) in one launch for few pixels, fp32:
// the blocks of a small batch of the Section 3.9 network, with the structure of block_patch_f16.hip.
//
// A workgroup owns patches of 4 x 4 output pixels -- the 16 rows of a v_mfma_f32_16x16x4_f32 -- and 16 JN output columns, and
// splits the channels over its wavefronts, 32 to each in every one of ROUNDS rounds.  A wavefront copies its channels of the input
// window under the patch and of the depthwise filter into an LDS region of its own (no barrier), computes the depthwise output of
// the 4 channels per lane and group of 16 that are its operand of four matrix instructions, and multiplies it by its rows of the
// pointwise filter, which come straight into registers; the loads of the next round are on their way meanwhile.  The wavefronts'
// partial tiles are added through LDS behind the only barrier.  The fp32 matrix instructions do: split into bf16 parts (split.h), the
// filter would be split again by every patch, for more than the 1 - 3 us that the instructions take here.
//
// Precision: these instructions round after every product, so 16 of them at a time start from zero and are added to the wavefront's
// sum (64 with 128 columns in four rounds, see patch_halves).  Error of the pointwise sum against float64, 2 images, 128 -> 128
// channels / 512 -> 512 / 1024 -> 1024: 7.3 / 9.5 / 10.6e-8, 8.4 / 10.5 / 13.1 with one sum a wavefront, 7.9 / 9.5 / 12.0 of the
// kernels before; it costs 0 - 2 % of a pass (4 images 157.7 -> 161.2 us).
//
// What bounds it is the latency of one launch and of each round of loads (5 us and 2 - 3 a round), and from some 256 workgroups on
// the filter's columns that each of them reads.  14 x 14 x 512 -> 512, us, against the two launches before: 2 images 7.7 (12.0), 3
// 10.9 (14.0), 4 10.9 (15.1); 56 x 56 x 128 -> 128, 2 images 10.4 (13.1), 3 13.9 (17.4); 7 x 7 x 1024 -> 1024, 4 images 12.4 (15.8),
// 8 17.1 (23.6).  The pass: 2 images 145 -> 113, 3 177 -> 151, 4 186 -> 162, 8 217 -> 208; 4 at half width 120 -> 92, 8 152 -> 120.
#include <algorithm>

#include "ragged.h"

namespace tfx {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kChannels32 = 32, kPieces = kChannels32 / 4;

struct PatchArgs {
  const float *x, *dw_w, *dw_b, *pw_w, *pw_b;
  float* y;
  int H, W, C, N, OH, OW, pt, pl;
  int patches;
  FastDiv row_patches, col_patches;
  unsigned x_bytes;
  int dw_act, pw_act;
};
// The arguments as block_patch_f16.hip has them: what the addresses depend on in scalar registers from the start, the rest read while
// the loads are under way.  Patches come first in the grid, padded to a multiple of 8, so that the column slices of a patch are on
// one XCD and its window in one L2 (column slices first where the filter is larger than the map, as there: 2 images 114.4 us, 110.8 so).
// us, before and now: 2 images 114.4 -> 110.8, 4 at quarter width and 192 x 192 75 -> 70.5, 16 at half width 161.6 -> 154.5.
// An XCD then has whole groups of patches, up to one more than another.  Where that puts another workgroup on a CU of the fullest, as
// where all fit into one round only if they are dealt evenly, the grid is not padded and the column slices of a patch go to several XCDs:
// 20 patches of 768 -> 768, 12 slices, 21.4 us padded and 13.1 so; 18 of 384 -> 384 7.4 and 6.1, of 192 -> 384 6.8 and 5.8.
// (Column slices first instead, a bit for the kernel to select by: as fast there, and .05 us more in every launch.)
struct PatchRest {
  const float *pw_w, *pw_b;
  float* y;
  int OH, OW, dw_act, pw_act;
};

// The window in LDS: strides of a pixel and of a row of pixels in 16-byte pieces, such that the fragment read of a tap is
// free of bank conflicts.
template <int S>
struct PatchWindow {
  static constexpr int SIDE = 3 * S + 3;
  struct At {
    int px, row;
    constexpr int operator()(int li, int q) const { return li / 4 * S * row + li % 4 * S * px + q; }
  };
  struct Strides {
    int px, row;
  };
  static constexpr Strides find() {
    for (int px = kPieces;; ++px)
      for (int row = SIDE * px; row < SIDE * px + 32; ++row)
        if (conflict_free(At{px, row})) return {px, row};
  }
  static constexpr Strides kStrides = find();
  static constexpr int FLOATS = 4 * SIDE * kStrides.row, FILTER = 10 * kChannels32;  // (the bias behind the taps)
};

// 128 columns in four rounds: no registers for a second set of sums, so those of the first two rounds lie behind the region
constexpr bool patch_halves(int jn, int rounds) { return jn == 8 && rounds == 4; }

template <int S, int JN, int ROUNDS>
constexpr size_t patch_region_bytes() {
  const size_t in = (size_t)(PatchWindow<S>::FLOATS + PatchWindow<S>::FILTER) * sizeof(float), out = (size_t)256 * JN * sizeof(float);
  return (in > out ? in : out) + (patch_halves(JN, ROUNDS) ? out : 0);
}

// Wavefronts of a workgroup at most: windows of stride 2 are 13 KB each, and 128 columns, or 64 in several rounds, take more than
// 128 registers.
constexpr int most_waves(int s, int jn, int rounds) { return s == 2 || jn == 8 || (jn == 4 && rounds > 1) ? 8 : 16; }

template <int S, int JN, int ROUNDS>
__global__ __launch_bounds__(64 * most_waves(S, JN, ROUNDS)) void separable_patch_kernel(
    const float* x, const float* dw_w, const float* dw_b, unsigned x_bytes, unsigned map, unsigned channels, unsigned patches, unsigned by_row,
    unsigned by_col, unsigned per, unsigned form, PatchRest g) {
  typedef PatchWindow<S> P;
  constexpr int LOADS = (P::SIDE * P::SIDE * kPieces + 63) / 64, FLOADS = (10 * kPieces + 63) / 64, G = kChannels32 / 16;
  constexpr int V = JN < 4 ? 1 : JN / 4;  // loads of a filter row
  extern __shared__ __align__(16) unsigned char lds[];

  const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int li = lane % 16, q = lane / 16;
  const int wk = (int)(form & 31), wp = (int)(form >> 5 & 7), pt = (int)(form >> 8 & 1), pl = (int)(form >> 9 & 1);
  const int H = (int)(map & 0xffff), W = (int)(map >> 16), C = (int)(channels & 0xffff), N = (int)(channels >> 16);
  const FastDiv row_patches{by_row, form >> 10 & 31, per & 0xffff}, col_patches{by_col, form >> 15 & 31, per >> 16};
  const int p = wave * (int)(form >> 20) >> 8, part = wave - p * wk;  // (wave / wk)
  const int n0 = (int)blockIdx.y * 16 * JN, patch = (int)blockIdx.x * wp + p;
  const bool live = patch < (int)patches;
  if (patch - p >= (int)patches) return;  // (the grid is padded)
  const int strip = (int)div_by((unsigned)patch, row_patches), image = (int)div_by((unsigned)strip, col_patches);
  const int ow0 = 4 * (patch - strip * (int)row_patches.d), oh0 = 4 * (strip - image * (int)col_patches.d);

  constexpr bool HALVES = patch_halves(JN, ROUNDS);
  constexpr int REGION = (int)patch_region_bytes<S, JN, ROUNDS>(), SUMS = 256 * JN;
  float* const window = reinterpret_cast<float*>(lds + wave * REGION);
  float* const taps = window + P::FLOATS;

  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, (int)x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t fr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(dw_w), 0, 36 * C, 0x00020000);
  const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(dw_b), 0, 4 * C, 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.pw_w), 0, 4 * C * N, 0x00020000);

  // What lies outside the map, or past the last channel, has an offset past the end and reads zeros.
  const int piece = lane % kPieces;
  unsigned at[LOADS], fat[FLOADS];  // byte offsets, channel 4 * piece
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int px = (64 * i + lane) / kPieces, r = px / P::SIDE, c = px - r * P::SIDE;
    const int ih = oh0 * S - pt + r, iw = ow0 * S - pl + c;
    const bool ok = (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W && px < P::SIDE * P::SIDE && live;
    at[i] = ok ? 4u * (((unsigned)(image * H + ih) * W + iw) * C + 4 * piece) : 0x80000000u;
  }
#pragma unroll
  for (int i = 0; i < FLOADS; ++i) {
    const int t = (64 * i + lane) / kPieces;
    fat[i] = t < 9 ? 4u * (unsigned)(t * C + 4 * piece) : 0x80000000u;
  }
  const int col = n0 + JN * li < N ? n0 + JN * li : 0;  // past the last column: read, never stored

  static_assert(FLOADS == 2, "the bias is in the second load");
  const unsigned bat = (64 + lane) / kPieces == 9 ? 16u * piece : 0x80000000u;
  u32x4 win[LOADS], fil[FLOADS], bias;
  struct Operands {
    float w[G][4][JN];  // rows 16 u + 4 q + s
  };
  auto fetch = [&](int round, Operands& o) __attribute__((always_inline)) {
    const int c0 = kChannels32 * (part + round * wk);
    const bool mine = c0 + 4 * piece < C;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) win[i] = __builtin_amdgcn_raw_buffer_load_b128(xr, mine ? at[i] + 4u * c0 : 0x80000000u, 0, 0);
#pragma unroll
    for (int i = 0; i < FLOADS; ++i) fil[i] = __builtin_amdgcn_raw_buffer_load_b128(fr, mine ? fat[i] + 4u * c0 : 0x80000000u, 0, 0);
    bias = __builtin_amdgcn_raw_buffer_load_b128(br, mine ? bat + 4u * c0 : 0x80000000u, 0, 0);
#pragma unroll
    for (int u = 0; u < G; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const unsigned off = 4u * ((unsigned)(c0 + 16 * u + 4 * q + s) * N + col);
        if constexpr (JN == 2) {
          const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(wr, off, 0, 0));
          o.w[u][s][0] = v[0], o.w[u][s][1] = v[1];
        } else {
#pragma unroll
          for (int h = 0; h < V; ++h) {
            const floatx4 v = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(wr, off + 16 * h, 0, 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) o.w[u][s][4 * h + e] = v[e];
          }
        }
      }
  };

  Operands ops[ROUNDS > 1 ? 2 : 1];
  fetch(0, ops[0]);
  float pwb[JN];
#pragma unroll
  for (int j = 0; j < JN; ++j) pwb[j] = g.pw_b[col + j];

  const ActClamp dw_clamp = make_act(g.dw_act), pw_clamp = make_act(g.pw_act);
  const float dw_lo = dw_clamp.on ? 0.f : -INFINITY;
  floatx4 acc[JN];
#pragma unroll
  for (int j = 0; j < JN; ++j) {
    const float b = part == 0 ? pwb[j] : 0.f;
    acc[j] = floatx4{b, b, b, b};
  }
  constexpr int AT = JN < 4 ? JN : 4;
  const float* const mine = window + 4 * (li / 4 * S * P::kStrides.row + li % 4 * S * P::kStrides.px + q);
#pragma unroll
  for (int round = 0; round < ROUNDS; ++round) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int px = (64 * i + lane) / kPieces, r = px / P::SIDE, c = px - r * P::SIDE;
      if (64 * (i + 1) <= P::SIDE * P::SIDE * kPieces || px < P::SIDE * P::SIDE)
        *reinterpret_cast<u32x4*>(window + 4 * (r * P::kStrides.row + c * P::kStrides.px + piece)) = win[i];
    }
#pragma unroll
    for (int i = 0; i < FLOADS; ++i)
      if (64 * (i + 1) <= 10 * kPieces || 64 * i + lane < 10 * kPieces) *reinterpret_cast<u32x4*>(taps + 4 * (64 * i + lane)) = i == 1 ? fil[i] | bias : fil[i];
    if (round + 1 < ROUNDS) fetch(round + 1, ops[(round + 1) % 2]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const Operands& o = ops[round % 2];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      floatx4 d = *reinterpret_cast<const floatx4*>(taps + kChannels32 * 9 + 16 * u + 4 * q);
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const floatx4 xt = *reinterpret_cast<const floatx4*>(mine + 4 * (t / 3 * P::kStrides.row + t % 3 * P::kStrides.px + 4 * u));
        const floatx4 wt = *reinterpret_cast<const floatx4*>(taps + kChannels32 * t + 16 * u + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = fmaf(xt[e], wt[e], d[e]);
      }
      // the median of three drops a NaN: those are looked for on the side
      floatx4 a;
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = __builtin_amdgcn_fmed3f(d[e], dw_lo, dw_clamp.hi);
      if (__builtin_amdgcn_ballot_w64(__builtin_isunordered(d[0], d[1]) | __builtin_isunordered(d[2], d[3])) != 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = apply_act(d[e], dw_clamp);
      }
#pragma unroll
      for (int j0 = 0; j0 < JN; j0 += AT) {
        const bool begin = HALVES || round + u == 0;
        floatx4 t[AT];
#pragma unroll
        for (int j = 0; j < AT; ++j) t[j] = begin ? acc[j0 + j] : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int j = 0; j < AT; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], o.w[u][s][j0 + j], t[j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < AT; ++j) acc[j0 + j] = begin ? t[j] : acc[j0 + j] + t[j];
        __builtin_amdgcn_sched_barrier(0);  // (fewer registers)
      }
    }
    if (HALVES && round == 1) {
      float* const half = reinterpret_cast<float*>(lds + (wave + 1) * REGION) - SUMS;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < JN; ++j) half[(v * 64 + lane) * JN + j] = acc[j][v];
#pragma unroll
      for (int j = 0; j < JN; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  // lane (li, q) holds columns JN li ... of pixels (row q, column v) of the patch
  auto store = [&](int v, int l, int j, float s0, float s1) __attribute__((always_inline)) {
    const int oh = oh0 + l / 16, ow = ow0 + v, cn = n0 + JN * (l % 16) + j;
    if (live && oh < g.OH && ow < g.OW && cn < N)
      *reinterpret_cast<f32x2*>(g.y + ((size_t)(image * g.OH + oh) * g.OW + ow) * N + cn) = f32x2{apply_act(s0, pw_clamp), apply_act(s1, pw_clamp)};
  };
  if (wk == 1) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int j = 0; j < JN; j += 2) store(v, lane, j, acc[j][v], acc[j + 1][v]);
    return;
  }
  float* const sums = window;  // [v][lane][JN], over the window, which is read
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int j = 0; j < JN; ++j) sums[(v * 64 + lane) * JN + j] = acc[j][v];
  __syncthreads();
  for (int u = 64 * part + lane; u < 128 * JN; u += 64 * wk) {
    float s0 = 0.f, s1 = 0.f;
    for (int w = 0; w < wk; ++w) {
      const f32x2 t = reinterpret_cast<const f32x2*>(lds + (p * wk + w) * REGION)[u];
      s0 += t[0], s1 += t[1];
      if constexpr (HALVES) {
        const f32x2 h = reinterpret_cast<const f32x2*>(lds + (p * wk + w + 1) * REGION - SUMS * sizeof(float))[u];
        s0 += h[0], s1 += h[1];
      }
    }
    const int v = u / (32 * JN), rest = u % (32 * JN);
    store(v, rest / (JN / 2), 2 * (rest % (JN / 2)), s0, s1);
  }
}

struct PatchForm {
  int jn, rounds, wk, wp;
  double us;       // modelled time
  bool one_round;  // all workgroups are resident at once
};

template <int S, int JN, int ROUNDS>
int launch_patch(const PatchArgs& args, const PatchForm& f, hipStream_t stream) {
  const PatchArgs& g = args;
  auto kern = separable_patch_kernel<S, JN, ROUNDS>;
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), 160 * 1024, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  const unsigned slices = (unsigned)((g.N + 16 * JN - 1) / (16 * JN)), groups = (unsigned)((g.patches + f.wp - 1) / f.wp);
  const size_t lds_bytes = patch_region_bytes<S, JN, ROUNDS>() * f.wk * f.wp;
  const bool crowded = f.one_round && ((groups + 7) / 8 * slices + 31) / 32 > (groups * slices + 255) / 256;  // (32 CUs of an XCD)
  const unsigned form = (unsigned)(f.wk | f.wp << 5 | g.pt << 8 | g.pl << 9) | g.row_patches.shift << 10 | g.col_patches.shift << 15 |
                        (256u + f.wk - 1) / f.wk << 20;
  const dim3 grid(crowded ? groups : (groups + 7) / 8 * 8, slices);
  hipLaunchKernelGGL(kern, grid, dim3(64u * f.wk * f.wp), lds_bytes, stream,
                     g.x, g.dw_w, g.dw_b, g.x_bytes, (unsigned)g.H | (unsigned)g.W << 16, (unsigned)(g.C | g.N << 16), (unsigned)g.patches,
                     g.row_patches.mul, g.col_patches.mul, g.row_patches.d | g.col_patches.d << 16, form,
                     PatchRest{g.pw_w, g.pw_b, g.y, g.OH, g.OW, g.dw_act, g.pw_act});
  return check_launch();
}

// Columns of a workgroup: the most that give at least 180 workgroups, since all column slices of a patch compute its depthwise layer
// again; more where that is what it takes for all of them to be resident at once.  The modelled time: a start, another for
// workgroups that wait for others to end, and for each workgroup of a CU and round the matrix instructions of a SIMD's wavefronts
// and the window (within 1.5 us of what 60 launches took, from 7 to 20).
PatchForm patch_form(long long patches, int c, int n, int stride) {
  const int parts = (c + kChannels32 - 1) / kChannels32;
  PatchForm f{};
  f.wp = parts == 1 ? 4 : parts == 2 ? 2 : 1;
  auto with = [&](int jn) {
    f.jn = jn;
    for (f.rounds = 1; f.rounds * most_waves(stride, jn, f.rounds) < parts; f.rounds *= 2) {
    }
    f.wk = (parts + f.rounds - 1) / f.rounds;
    const long long blocks = (patches + f.wp - 1) / f.wp * ((n + 16 * jn - 1) / (16 * jn));
    const int waves = jn == 8 ? (stride == 2 || f.rounds > 1 ? 8 : 12) : f.rounds > 1 ? most_waves(stride, jn, f.rounds) : 20;  // by registers
    f.one_round = blocks <= 256 * std::max(1, waves / (f.wk * f.wp));
    f.us = (f.one_round ? 5. : 8.) + (double)((blocks + 255) / 256) * f.rounds * (.125 * jn * ((f.wk * f.wp + 3) / 4) + stride);
    return blocks;
  };
  int jn = n >= 128 && with(8) >= 180 ? 8 : n >= 64 && with(4) >= 180 ? 4 : 2;
  for (with(jn); jn < 8 && n >= 32 * jn && !f.one_round; with(jn)) jn *= 2;
  return f;
}

}  // namespace

bool separable_patch_supported(int batch, int h, int w, int c, int n, int stride, int oh, int ow, const void* x, const void* dw_w,
                               const void* dw_b, const void* pw_w, const void* pw_b, const void* y) {
  const void* ptrs[] = {x, dw_w, dw_b, pw_w, pw_b, y};
  bool aligned = true;
  for (const void* p : ptrs) aligned = aligned && reinterpret_cast<uintptr_t>(p) % 16 == 0;
  const long long patches = (long long)batch * ((oh + 3) / 4) * ((ow + 3) / 4), x_bytes = (long long)batch * h * w * c * 4;
  return aligned && (stride == 1 || stride == 2) && c % 4 == 0 && c <= (stride == 1 ? 1024 : 512) && n % 8 == 0 && n <= 1024 && x_bytes < (1ll << 31) &&
         patches < (1ll << 24) && h < 65536 && w < 65536;
}

// Against what the block would run as, two launches mostly: 6.5 us, their products, and for large maps the depthwise output's way
// through memory (14 x 14 x 512 -> 512, 2 images 12.0, 4 15.1; 3/4 width 3 images 9.7; 7 x 7 x 1024 -> 1024, 8 images 23.6).
bool separable_patch_pays(int batch, int c, int n, int stride, int oh, int ow) {
  const double rows = (double)batch * oh * ow, products = 1e-6 * rows * c * n;
  double other = 6.5 + .045 * std::min(products, 250.) + .02 * std::max(products - 250., 0.) + std::min(4., .4e-3 * rows);
  const bool fused = batch <= 3 && (c == 128 || c == 256) && n % 64 == 0;  // (block.hip, slower than two launches at 3 images)
  if (fused) other *= 1.35;
  const PatchForm f = patch_form((long long)batch * ((oh + 3) / 4) * ((ow + 3) / 4), c, n, stride);
  return (f.one_round || fused) && f.us < other;
}

int launch_separable_patch(const float* x, const float* dw_w, const float* dw_b, const float* pw_w, const float* pw_b, float* y,
                           int batch, int h, int w, int c, int n, int oh, int ow, int stride, int pt, int pl, int dw_act, int pw_act,
                           hipStream_t stream) {
  const int row_patches = (ow + 3) / 4, col_patches = (oh + 3) / 4, patches = batch * col_patches * row_patches;
  const PatchArgs g{x, dw_w, dw_b, pw_w, pw_b, y, h, w, c, n, oh, ow, pt, pl, patches, fast_div((unsigned)row_patches),
                    fast_div((unsigned)col_patches), (unsigned)((long long)batch * h * w * c * 4), dw_act, pw_act};
  const PatchForm f = patch_form(patches, c, n, stride);
#define TFX_PATCH(S, JN, ROUNDS) \
  if (stride == S && f.jn == JN && f.rounds == ROUNDS) return launch_patch<S, JN, ROUNDS>(g, f, stream);
#define TFX_PATCHES(S, JN) TFX_PATCH(S, JN, 1) TFX_PATCH(S, JN, 2)
  TFX_PATCHES(1, 2) TFX_PATCHES(1, 4) TFX_PATCHES(1, 8) TFX_PATCHES(2, 2) TFX_PATCHES(2, 4) TFX_PATCHES(2, 8)
  TFX_PATCH(1, 4, 4) TFX_PATCH(1, 8, 4)  // (stride 2: up to 512 channels)
#undef TFX_PATCHES
#undef TFX_PATCH
  return TFX_ERR_UNSUPPORTED;
}

}  // namespace tfx
