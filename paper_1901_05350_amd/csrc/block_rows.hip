// The stem (3x3 stride-2 convolution of the image to 8 Q channels) and the first depthwise-separable block (depthwise 3x3 +
// bias + clamp, pointwise 1x1 to 16 Q channels + bias + clamp) of the Section 3.9 network in one launch, fp32: the structure of
// block_rows_f16.hip.  A workgroup walks down a strip of rows of one image, a wavefront for every 16 columns, with four stem
// rows in LDS: three under the depthwise filter and the one it computes for the next step, with one barrier a row.
//
// Contraction of the stem (v_mfma_f32_16x16x4_f32, filters as the first operand, 7 steps): lane (li, q) supplies seven values of
// pixel li's window; for q < 3 the first seven of the nine that lie next to each other in image row q of it, for q = 3 the last
// two of each row.  The depthwise layer: lane (li, q) has channels 16 u + 4 q ... + 3 of pixel li, which are its operands of
// four steps of the pointwise product.
#include "split.h"

namespace tfx {
namespace {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct RowsArgs {
  const float *x, *st_w, *st_b, *dw_w, *dw_b, *pw_w, *pw_b;
  float* y;
  int IH, IW, OH, OW, pt, pl, strips, rows;  // rows of a strip
  unsigned image_bytes, x_bytes, y_bytes;
};

// Pixel stride of the ring in 16-byte pieces: the least without bank conflicts when lane (li, q) reads piece q of pixel li.
struct RowsPixel {
  int pieces;
  constexpr int operator()(int li, int q) const { return li * pieces + q; }
};
template <int G>
constexpr int rows_pixel_pieces() {
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

template <int Q>
__global__ __launch_bounds__(512, 2) void stem_block_rows_kernel(RowsArgs g) {
  constexpr int C = 8 * Q, N = 16 * Q, NB = Q, G = (C + 15) / 16, PX = 4 * rows_pixel_pieces<G>();
  extern __shared__ __align__(16) float ring[];  // [4][16 T + 2][PX]: stem row r in slot r % 4, column c at c + 1
  // what a step reads once or twice stays in LDS
  __shared__ __align__(16) float stem_w[7][64][G], stem_bias[16 * G], dw_bias[16 * G], pw_bias[N];
  const int lane = threadIdx.x % 64, li = lane % 16, q = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int cols = (int)blockDim.x / 4 + 2, slot = cols * PX;
  const int n = blockIdx.x / g.strips, r0 = (blockIdx.x - n * g.strips) * g.rows, r1 = min(r0 + g.rows, g.OH);
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
  floatx4 dww[9][G];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int u = 0; u < G; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = 16 * u + 4 * q + e;
        const float v = g.dw_w[t * C + (k < C ? k : 0)];
        dww[t][u][e] = k < C ? v : 0.f;
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
  unsigned out = in ? 4u * ((unsigned)((n * g.OH + r0) * g.OW + ow) * N) : kNone;  // past the end: not stored
  for (int r = r0; r < r1; ++r, out += 4u * g.OW * N) {
    if (r + 1 < r1) stem(r + 2, next);
    if (r + 2 < r1) fetch(r + 3, next);
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
          d[u] += *reinterpret_cast<const floatx4*>(row + kw * PX + 16 * u) * dww[3 * kh + kw][u];
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
    for (int j = 0; j < NB; ++j)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, relu6(acc[j])), yr, out + 64 * j + 16 * q, 0, 0);
    __syncthreads();
  }
}

constexpr int kRowsMaxWidth = 128;  // columns of the map: 8 wavefronts of 16

template <int Q>
int launch_rows(const RowsArgs& g, int batch, hipStream_t stream) {
  auto kern = stem_block_rows_kernel<Q>;
  const int tiles = (g.OW + 15) / 16;
  // The kernel is allowed once what its widest rows need: a later call may be wider than the first.
  constexpr size_t column = (size_t)4 * 16 * rows_pixel_pieces<(8 * Q + 15) / 16>(), most = (kRowsMaxWidth + 2) * column;
  const size_t lds_bytes = (16 * tiles + 2) * column;
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), most, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, dim3((unsigned)(batch * g.strips)), dim3(64u * tiles), lds_bytes, stream, g);
  return check_launch();
}

}  // namespace

int launch_stem_block_rows(const float* image, const float* st_w, const float* st_b, const float* dw_w, const float* dw_b, const float* pw_w,
                           const float* pw_b, float* y, int batch, int ih, int iw, int oh, int ow, int pt, int pl, int q,
                           hipStream_t stream) {
  const long long in = (long long)ih * iw * 3, out = (long long)oh * ow * 16 * q;  // floats of an image
  if (ow > kRowsMaxWidth || iw < 3 || ih < 3 || reinterpret_cast<uintptr_t>(y) % 16 != 0) return TFX_ERR_UNSUPPORTED;
  const int tiles = (ow + 15) / 16, slots = 256 * ((q <= 2 ? 16 : 8) / tiles > 0 ? (q <= 2 ? 16 : 8) / tiles : 1);
  // byte offsets of a launch stay below 2^31
  const long long most = ((1ll << 29) - 1) / (in > out ? in : out);
  for (long long first = 0; first < batch; first += most) {
    const int images = (int)(batch - first < most ? batch - first : most);
    // Strips of an image: rounds of resident workgroups (their registers leave 8 wavefronts to a CU, of the narrow networks 16)
    // times their rows, and five more for the two rows computed twice and for start and end.  224 x 224, 2 images: 112 strips
    // 10.1 us, 56 11.5; 16: 16 24.6, 28 30.5, 8 36.1; 64: 4 74, 8 81, 16 90.
    int strips = 1;
    double best = 1e30;
    for (int s = 1; s <= oh; ++s) {
      const int rows = (oh + s - 1) / s;
      if ((oh + rows - 1) / rows != s) continue;
      const double cost = (double)(((long long)images * s + slots - 1) / slots) * (rows + 5);
      if (cost < best) best = cost, strips = s;
    }
    const RowsArgs g{image + first * in, st_w, st_b, dw_w, dw_b, pw_w, pw_b, y + first * out, ih, iw, oh, ow, pt, pl, strips,
                     (oh + strips - 1) / strips, (unsigned)(4 * in), (unsigned)(4 * images * in), (unsigned)(4 * images * out)};
    int rc = TFX_ERR_UNSUPPORTED;
    if (q == 1) rc = launch_rows<1>(g, images, stream);
    if (q == 2) rc = launch_rows<2>(g, images, stream);
    if (q == 3) rc = launch_rows<3>(g, images, stream);
    if (q == 4) rc = launch_rows<4>(g, images, stream);
    if (rc) return rc;
  }
  return TFX_OK;
}

}  // namespace tfx
