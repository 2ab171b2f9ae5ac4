// Small outputs with any contraction length, on float and on 16-bit float storage: matMul / batchMatMul of every layout,
// size and alignment (Listing 2, Section 4.1), and conv2d as an implicit GEMM (the NHWC index order of Section 4.1).
//   C[b] = act( op(A[b]) * op(B[b]) + bias )
//
// With fewer output tiles than CUs the contraction is a serial chain: a 64 x 64 tile of the LDS-staged kernels walks
// through K one slice after the other with one memory round trip each (32 x 297 x 3485 on binary16: 101 us), and
// there is no workspace that workgroups could add partial results in.  So a workgroup here is a 16 x 16 TN tile whose
// 4, 8 or 16 wavefronts take k-steps w, w + WAVES, ... each, load the matrix-core operands of U of their steps straight
// into registers at once, and add their partial tiles through LDS once at the end: a few memory round trips whatever K
// is.  Bound by latency (launch, one or two round trips, the reduction), and by L2 once there are many tiles, which is
// where the dispatchers of gemm.hip, gemm_f16.hip and conv_gemm_f16.hip go over to LDS-staged tiles.
//
// A lane holds, of a k-step, PER consecutive k of its row / column: 4 floats (four v_mfma_f32_16x16x4_f32 with the k
// order permuted alike on both sides) or 8 halfs (one v_mfma_f32_16x16x32_f16).  K-contiguous operands are fetched 16
// bytes at a time at any alignment (ragged.h); the others element by element along k, TN adjacent columns per load.
// A convolution's k runs over (tap, channel) with the channels of a tap padded to a multiple of PER, so that a chunk
// never crosses a tap and any channel count works; padding and taps outside the image are zeros.
#include "kernel_cost.h"
#include "ragged.h"

namespace tfx {
namespace {

constexpr int kXcds = 8;

template <typename T>
struct Step;
template <>
struct Step<float> {
  static constexpr int kPer = 4, kK = 16;
};
template <>
struct Step<_Float16> {
  static constexpr int kPer = 8, kK = 32;
};
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ floatx4 mma(const ragged_u32x4& a, const ragged_u32x4& b, floatx4 acc, float) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[s]), __uint_as_float(b[s]), acc, 0, 0, 0);
  return acc;
}
__device__ __forceinline__ floatx4 mma(const ragged_u32x4& a, const ragged_u32x4& b, floatx4 acc, _Float16) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), acc, 0, 0, 0);
}

enum Source { kRowsK, kRowsM, kConv };  // A stored [M,K]; stored [K,M]; the window view of an NHWC image

struct DeepArgs {
  const void *a, *b, *bias;
  void* c;
  int M, N, K;                 // K: channels per tap for a convolution
  unsigned a_total, b_total;   // elements of one batch's operand
  long long strideA, strideB, strideC;
  int tiles_m, tiles_n, total_blocks, m_fastest, act;
  int steps;                   // k-steps in all
  // convolution only
  int H, W, fw, taps, sh, sw, pt, pl;
  FastDiv by_cp, by_fw, by_ow, by_oh;
};

template <typename T, Source A_SRC, bool B_KC, int TN, int WAVES, int U>
__global__ __launch_bounds__(64 * WAVES) void gemm_deep_kernel(DeepArgs g) {
  constexpr int PER = Step<T>::kPer, KSTEP = Step<T>::kK;
  static_assert(TN == 1 || TN == 2, "tile width");
  __shared__ float red[WAVES * TN * 4 * 64];  // partial tiles: [wavefront][column block j][register v][lane]

  const int bid = blockIdx.x;
  const int q8 = g.total_blocks / kXcds, rem = g.total_blocks % kXcds;
  const int xcd = bid % kXcds;
  const int vid = xcd * q8 + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int tiles = g.tiles_m * g.tiles_n;
  const int batch = vid / tiles, t = vid % tiles;
  const int tile_m = g.m_fastest ? t % g.tiles_m : t / g.tiles_n;
  const int tile_n = g.m_fastest ? t / g.tiles_m : t % g.tiles_n;
  const int tid = threadIdx.x, wk = tid / 64, lane = tid % 64, li = lane % 16, q = lane / 16;
  const int m0 = tile_m * 16, n0 = tile_n * 16 * TN;
  const T* const A = static_cast<const T*>(g.a) + (size_t)batch * g.strideA;
  const T* const B = static_cast<const T*>(g.b) + (size_t)batch * g.strideB;

  // rows and columns past the matrix repeat the last one (they only feed outputs that are not stored)
  const int arow = min(m0 + li, g.M - 1);
  const int bcol = min(n0 + TN * li, g.N - TN);  // N % TN == 0
  int origin = 0, ih0 = 0, iw0 = 0;
  if constexpr (A_SRC == kConv) {
    const unsigned r = (unsigned)arow, r2 = div_by(r, g.by_ow), n = div_by(r2, g.by_oh);
    ih0 = (int)(r2 - n * g.by_oh.d) * g.sh - g.pt;
    iw0 = (int)(r - r2 * g.by_ow.d) * g.sw - g.pl;
    origin = (((int)n * g.H + ih0) * g.W + iw0) * g.K;
  }

  // epilogue thread e < 256: register e / 64 of lane e % 64; its bias is fetched now
  const int ev = tid / 64, el = tid % 64;
  const int erow = m0 + 4 * (el / 16) + ev, ecol = n0 + TN * (el % 16);
  float ebias[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
    ebias[j] = tid < 256 && g.bias != nullptr && ecol + j < g.N ? (float)static_cast<const T*>(g.bias)[ecol + j] : 0.f;

  floatx4 acc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};

  for (int step0 = wk; step0 < g.steps; step0 += WAVES * U) {
    ragged_u32x4 a[U], b[U][TN];   // K-contiguous chunks
    T ae[U][PER], be[U][PER][TN];  // elements gathered along k
    int ra[U], rb[U];              // valid k of the lane's chunk
    unsigned sa[U], sb[U][TN];     // elements a chunk was fetched early by
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = (step0 + u * WAVES) * KSTEP + PER * q;
      // (tap, channel) of the chunk; a matrix is one tap
      int tap = 0, c = kk;
      if constexpr (A_SRC == kConv) {
        tap = (int)div_by((unsigned)kk, g.by_cp);
        c = kk - tap * (int)g.by_cp.d;
      }
      const int r = (A_SRC != kConv || tap < g.taps) ? g.K - c : 0;
      ra[u] = rb[u] = r;
      const bool any = r > 0;
      if constexpr (A_SRC == kRowsM) {
#pragma unroll
        for (int e = 0; e < PER; ++e) ae[u][e] = A[(size_t)(e < r ? c + e : 0) * g.M + arow];
      } else {
        unsigned off;
        if constexpr (A_SRC == kConv) {
          const int kh = (int)div_by((unsigned)tap, g.by_fw), kw = tap - kh * g.fw;
          const int ih = ih0 + kh, iw = iw0 + kw;
          const bool in = any && ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
          if (!in) ra[u] = 0;
          off = in ? (unsigned)(origin + (kh * g.W + kw) * g.K + c) : 0u;
        } else {
          off = any ? (unsigned)arow * (unsigned)g.K + (unsigned)c : 0u;
        }
        const unsigned at = min(off, g.a_total - PER);
        sa[u] = off - at;
        a[u] = load16(A + at);
      }
      if constexpr (B_KC) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const unsigned off = any ? (unsigned)(bcol + j) * (unsigned)g.K + (unsigned)c : 0u;
          const unsigned at = min(off, g.b_total - PER);
          sb[u][j] = off - at;
          b[u][j] = load16(B + at);
        }
      } else {
        const int row = tap * g.K + c;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
          typedef T pair __attribute__((ext_vector_type(2), aligned(sizeof(T))));
          const T* p = B + (size_t)(e < r ? row + e : 0) * g.N + bcol;
          if constexpr (TN == 2) {
            const pair v = *reinterpret_cast<const pair*>(p);
            be[u][e][0] = v[0];
            be[u][e][1] = v[1];
          } else {
            be[u][e][0] = *p;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const ragged_u32x4 va = first_elements<T>(ra[u]), vb = first_elements<T>(rb[u]);
      T tmp[PER];
      if constexpr (A_SRC == kRowsM) {
#pragma unroll
        for (int e = 0; e < PER; ++e) tmp[e] = ae[u][e];
        a[u] = __builtin_bit_cast(ragged_u32x4, tmp);
      } else if (__builtin_amdgcn_ballot_w64(sa[u] != 0) != 0) {
        a[u] = shift_down<T>(a[u], sa[u]);
      }
      a[u] &= va;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (B_KC) {
          if (__builtin_amdgcn_ballot_w64(sb[u][j] != 0) != 0) b[u][j] = shift_down<T>(b[u][j], sb[u][j]);
        } else {
#pragma unroll
          for (int e = 0; e < PER; ++e) tmp[e] = be[u][e][j];
          b[u][j] = __builtin_bit_cast(ragged_u32x4, tmp);
        }
        b[u][j] &= vb;
        acc[j] = mma(a[u], b[u][j], acc[j], T());
      }
    }
  }

#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((wk * TN + j) * 4 + v) * 64 + lane] = acc[j][v];
  __syncthreads();
  if (tid < 256 && erow < g.M) {
    const ActClamp clamp = make_act(g.act);
    T* const cp = static_cast<T*>(g.c) + (size_t)batch * g.strideC + (size_t)erow * g.N + ecol;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float sum = ebias[j];
#pragma unroll
      for (int w = 0; w < WAVES; ++w) sum += red[((w * TN + j) * 4 + ev) * 64 + el];
      if (ecol + j < g.N) cp[j] = (T)apply_act(sum, clamp);
    }
  }
}

template <typename T, Source A_SRC, bool B_KC, int TN>
int launch(DeepArgs& g, int batch, hipStream_t stream) {
  g.tiles_m = (g.M + 15) / 16;
  g.tiles_n = (g.N + 16 * TN - 1) / (16 * TN);
  const long long total = (long long)batch * g.tiles_m * g.tiles_n;
  if (total > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  g.total_blocks = (int)total;
  g.m_fastest = g.N > g.M ? 1 : 0;
  // wavefronts enough that each has at most a few steps, loaded in one or two rounds; no more loads in a round than there are
  // steps, since those past the contraction are issued too (halfs, k = 257 ... 512: 4.5 us with 8 x 4, 4.0 with 8 x 2 on
  // average; 794 x 272 x 24 3.9 and 3.2; floats, 280 x 144 x 16 3.8 and 3.0; up to 4 steps 4 x 2 against 4 x 1 is 3 - 4 %).
  // With 8 x 1 for 5 - 8 steps and 16 x 2 for 17 - 32 more wavefronts are started for the same loads: 4 % slower, and no change.
  if (g.steps <= 4) hipLaunchKernelGGL((gemm_deep_kernel<T, A_SRC, B_KC, TN, 4, 1>), dim3((unsigned)total), dim3(256), 0, stream, g);
  else if (g.steps <= 8) hipLaunchKernelGGL((gemm_deep_kernel<T, A_SRC, B_KC, TN, 4, 2>), dim3((unsigned)total), dim3(256), 0, stream, g);
  else if (g.steps <= 16) hipLaunchKernelGGL((gemm_deep_kernel<T, A_SRC, B_KC, TN, 8, 2>), dim3((unsigned)total), dim3(512), 0, stream, g);
  else if (g.steps <= 32) hipLaunchKernelGGL((gemm_deep_kernel<T, A_SRC, B_KC, TN, 8, 4>), dim3((unsigned)total), dim3(512), 0, stream, g);
  else hipLaunchKernelGGL((gemm_deep_kernel<T, A_SRC, B_KC, TN, 16, 4>), dim3((unsigned)total), dim3(1024), 0, stream, g);
  return check_launch();
}

template <typename T, Source A_SRC, bool B_KC>
int launch_width(DeepArgs& g, int batch, hipStream_t stream) {
  return deep_two_columns((long long)batch * ((g.M + 15) / 16), g.N, g.steps) ? launch<T, A_SRC, B_KC, 2>(g, batch, stream)
                                                                              : launch<T, A_SRC, B_KC, 1>(g, batch, stream);
}

template <typename T>
int gemm(const T* a, const T* b, T* c, const T* bias, int batch, int m, int n, int k, bool a_kc, bool b_kc, int act,
         hipStream_t stream) {
  DeepArgs g{};
  g.a = a, g.b = b, g.bias = bias, g.c = c;
  g.M = m, g.N = n, g.K = k, g.act = act;
  g.strideA = (long long)m * k, g.strideB = (long long)n * k, g.strideC = (long long)m * n;
  g.a_total = (unsigned)g.strideA, g.b_total = (unsigned)g.strideB;
  g.steps = (k + Step<T>::kK - 1) / Step<T>::kK;
  if (a_kc) return b_kc ? launch_width<T, kRowsK, true>(g, batch, stream) : launch_width<T, kRowsK, false>(g, batch, stream);
  return b_kc ? launch_width<T, kRowsM, true>(g, batch, stream) : launch_width<T, kRowsM, false>(g, batch, stream);
}

template <typename T>
int conv(const T* x, const T* w, const T* bias, T* y, int n, int h, int wd, int ci, int fh, int fw, int co, int oh, int ow,
         int sh, int sw, int pt, int pl, int act, hipStream_t stream) {
  constexpr int PER = Step<T>::kPer;
  DeepArgs g{};
  const int cp = (ci + PER - 1) / PER * PER;
  g.a = x, g.b = w, g.bias = bias, g.c = y;
  g.M = n * oh * ow, g.N = co, g.K = ci, g.act = act;
  g.a_total = (unsigned)((long long)n * h * wd * ci), g.b_total = (unsigned)((long long)fh * fw * ci * co);
  g.steps = (fh * fw * cp + Step<T>::kK - 1) / Step<T>::kK;
  g.H = h, g.W = wd, g.fw = fw, g.taps = fh * fw, g.sh = sh, g.sw = sw, g.pt = pt, g.pl = pl;
  g.by_cp = fast_div((unsigned)cp), g.by_fw = fast_div((unsigned)fw), g.by_ow = fast_div((unsigned)ow), g.by_oh = fast_div((unsigned)oh);
  return launch_width<T, kConv, false>(g, 1, stream);
}

}  // namespace

int launch_gemm_deep(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, bool a_kc,
                     bool b_kc, int act, hipStream_t stream) {
  return gemm<float>(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream);
}
int launch_gemm_deep_f16(const uint16_t* a, const uint16_t* b, uint16_t* c, const uint16_t* bias, int batch, int m, int n,
                         int k, bool a_kc, bool b_kc, int act, hipStream_t stream) {
  typedef _Float16 H;
  return gemm<H>(reinterpret_cast<const H*>(a), reinterpret_cast<const H*>(b), reinterpret_cast<H*>(c),
                 reinterpret_cast<const H*>(bias), batch, m, n, k, a_kc, b_kc, act, stream);
}
int launch_conv2d_deep(const float* x, const float* w, const float* bias, float* y, int n, int h, int wd, int ci, int fh, int fw,
                       int co, int oh, int ow, int sh, int sw, int pt, int pl, int act, hipStream_t stream) {
  return conv<float>(x, w, bias, y, n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream);
}
int launch_conv2d_deep_f16(const uint16_t* x, const uint16_t* w, const uint16_t* bias, uint16_t* y, int n, int h, int wd, int ci,
                           int fh, int fw, int co, int oh, int ow, int sh, int sw, int pt, int pl, int act,
                           hipStream_t stream) {
  typedef _Float16 H;
  return conv<H>(reinterpret_cast<const H*>(x), reinterpret_cast<const H*>(w), reinterpret_cast<const H*>(bias),
                 reinterpret_cast<H*>(y), n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream);
}

}  // namespace tfx
