// Products with a short contraction, on float and on 16-bit float storage: C[b] = act(op(A[b]) * op(B[b]) + bias) with K <= 32
// floats (any batch and layout) or 64 halfs (one batch, A stored [M,K]), any N and alignment; also 1x1 convolutions of any
// stride (the pixel rows of an NHWC image are A's).
//
// There is little to multiply per byte, so the product should run at the speed of reading A and writing C; the kernels
// that stage tiles or split K over wavefronts spend their time on barriers, reductions and, with K below a slice or a
// k-step per wavefront, on nothing (200704 x 16 x 8 floats: 27 us).  Here a wavefront keeps its 32 TN columns of one
// batch's B in registers for the whole launch and walks over tiles of 32 rows of A, the next one in flight while the
// current one is multiplied: no LDS, no barrier.  Floats on v_mfma_f32_32x32x2_f32, halfs on v_mfma_f32_32x32x16_f16.  B is
// the first operand, so that a lane ends up with four consecutive columns of a row: one 16- (8-) byte store.
// A lane's operand of a k-step of 16 is 8 consecutive k of its row (column), loaded 16 bytes at a time at any alignment
// where these are contiguous, one element at a time (32 rows next to each other) where they are not.
// Bound by the stores: 32 x 1024 x 1024 floats, K = 8: 28 us, 1.05 times the bytes at the rate of a large copy
// (LDS tiles 39 and 49, wavefronts splitting K 80 ... 117).
#include "ragged.h"

#include <algorithm>

namespace tfx {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

template <typename T>
struct ThinArgs {
  const T *a, *b, *bias;
  T* c;
  int M, N, K, b_kc, act;
  int tiles, step_tiles;               // row tiles; how many wavefronts share them
  FastDiv by_groups, by_chains;        // column groups; batch x column groups
  unsigned total;                      // elements of one batch's A
  long long strideA, strideB, strideC;
  // strided 1x1 convolution only
  int H, W, stride;
  FastDiv by_ow, by_oh;
};

enum Rows { kRowsK, kRowsM, kStrided };  // A stored [M,K]; stored [K,M]; the pixels of a strided 1x1 convolution

template <typename T, int STEPS, int TN, Rows ROWS>
__global__ __launch_bounds__(256) void gemm_thin_kernel(ThinArgs<T> g) {
  constexpr bool HALF = sizeof(T) == 2, STRIDED = ROWS == kStrided;
  constexpr int CH = HALF ? 1 : 2, PER = 8 / CH;  // 16-byte chunks per octet of k
  const int lane = threadIdx.x % 64, li = lane % 32, h = lane / 32;
  const int gw = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // uniform: so are the operands' addresses
  const int first = (int)div_by((unsigned)gw, g.by_chains), chain = gw - first * (int)g.by_chains.d;
  const int step_tiles = g.step_tiles;
  if (first >= step_tiles) return;
  const int batch = (int)div_by((unsigned)chain, g.by_groups), n0 = (chain - batch * (int)g.by_groups.d) * 32 * TN;
  const T* const A = g.a + (size_t)batch * g.strideA;
  const T* const B = g.b + (size_t)batch * g.strideB;

  auto row_offset = [&](int tile) __attribute__((always_inline)) {  // element offset of this lane's row (rows past M repeat the last one)
    const int row = min(tile * 32 + li, g.M - 1);
    if constexpr (ROWS == kRowsM) return (unsigned)row;
    if constexpr (STRIDED) {
      const unsigned r2 = div_by((unsigned)row, g.by_ow), n = div_by(r2, g.by_oh);
      const int oh = (int)(r2 - n * g.by_oh.d), ow = row - (int)(r2 * g.by_ow.d);
      return (unsigned)((((int)n * g.H + oh * g.stride) * g.W + ow * g.stride) * g.K);
    } else {
      return (unsigned)row * (unsigned)g.K;
    }
  };
  // chunks past K are fetched from the row's start, ones that would leave A early enough to end with it; settled below
  auto fetch = [&](unsigned row, ragged_u32x4 (&a)[STEPS][CH]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        const int k = 16 * s + 8 * h + PER * q;
        if constexpr (ROWS == kRowsM) {  // one element of each of PER rows of A; k past K repeat the last one
          T v[PER];
#pragma unroll
          for (int e = 0; e < PER; ++e) v[e] = A[(unsigned)min(k + e, g.K - 1) * (unsigned)g.M + row];
          __builtin_memcpy(&a[s][q], v, 16);
        } else {
          a[s][q] = load16(A + min(row + (unsigned)(k < g.K ? k : 0), g.total - (unsigned)PER));
        }
      }
  };
  // the first rows of A are on their way while B comes in
  ragged_u32x4 a[STEPS][CH], next[STEPS][CH];
  unsigned row = row_offset(first);
  fetch(row, a);

  // B: octets of column n0 + 32 j + li, zeros past K and N (every load unconditional, from a valid place): 16 bytes of a
  // column stored [N,K], one element of each of eight rows stored [K,N]
  ragged_u32x4 b[STEPS][TN][CH];
  if (g.b_kc) {
    const unsigned total = (unsigned)g.N * (unsigned)g.K;
    auto offset = [&](int s, int j, int q) __attribute__((always_inline)) {
      const int k = 16 * s + 8 * h + PER * q;
      return (unsigned)min(n0 + 32 * j + li, g.N - 1) * (unsigned)g.K + (unsigned)(k < g.K ? k : 0);
    };
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < CH; ++q) b[s][j][q] = load16(B + min(offset(s, j, q), total - (unsigned)PER));
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < CH; ++q) {
          const unsigned at = offset(s, j, q), early = at - min(at, total - (unsigned)PER);
          if (__builtin_amdgcn_ballot_w64(early != 0) != 0) b[s][j][q] = shift_down<T>(b[s][j][q], early);
        }
  } else {
    T v[STEPS][TN][8];
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[s][j][e] = B[(unsigned)min(16 * s + 8 * h + e, g.K - 1) * (unsigned)g.N + (unsigned)min(n0 + 32 * j + li, g.N - 1)];
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < CH; ++q) __builtin_memcpy(&b[s][j][q], &v[s][j][PER * q], 16);
  }
#pragma unroll
  for (int s = 0; s < STEPS; ++s)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < CH; ++q) b[s][j][q] &= first_elements<T>(n0 + 32 * j + li < g.N ? g.K - (16 * s + 8 * h + PER * q) : 0);
  float bias[TN][16];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) bias[j][v] = 0.f;
  if (g.bias != nullptr) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) bias[j][v] = (float)g.bias[min(n0 + 32 * j + 8 * (v / 4) + 4 * h + v % 4, g.N - 1)];
  }
  const ActClamp clamp = make_act(g.act);

  auto settle = [&](unsigned row, ragged_u32x4 (&a)[STEPS][CH]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (16 * s + 16 <= g.K && s + 1 < STEPS) continue;  // all of it inside K (uniform)
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        const int k = 16 * s + 8 * h + PER * q;
        if constexpr (ROWS != kRowsM) {
          const unsigned at = row + (unsigned)(k < g.K ? k : 0), early = at - min(at, g.total - (unsigned)PER);
          if (__builtin_amdgcn_ballot_w64(early != 0) != 0) a[s][q] = shift_down<T>(a[s][q], early);
        }
        a[s][q] &= first_elements<T>(g.K - k);
      }
    }
  };

  for (int tile = first; tile < g.tiles; tile += step_tiles) {
    const unsigned row_next = row_offset(min(tile + step_tiles, g.tiles - 1));
    fetch(row_next, next);
    settle(row, a);
    floatx16 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if constexpr (HALF) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, b[s][j][0]), __builtin_bit_cast(h8, a[s][0]), acc[j], 0, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(b[s][j][e / PER][e % PER]), __uint_as_float(a[s][e / PER][e % PER]),
                                                          acc[j], 0, 0, 0);
      }
    }
    const int out = tile * 32 + li;
    if (out < g.M) {
      T* const cp = g.c + (size_t)batch * g.strideC + (size_t)out * g.N;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int col = n0 + 32 * j + 8 * v + 4 * h;
          typedef T quad __attribute__((ext_vector_type(4)));
          typedef quad quad_any __attribute__((aligned(sizeof(T))));
          quad o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (T)apply_act(acc[j][4 * v + e] + bias[j][4 * v + e], clamp);
          if (col + 4 <= g.N) {
            *reinterpret_cast<quad_any*>(cp + col) = o;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (col + e < g.N) cp[col + e] = o[e];
          }
        }
    }
    row = row_next;
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int q = 0; q < CH; ++q) a[s][q] = next[s][q];
  }
}

template <typename T, int STEPS, int TN, Rows ROWS>
int launch_cfg(ThinArgs<T>& g, int batch, hipStream_t stream) {
  g.tiles = (g.M + 31) / 32;
  const int groups = (g.N + 32 * TN - 1) / (32 * TN), chains = batch * groups;  // (at most the elements of C)
  g.by_groups = fast_div((unsigned)groups), g.by_chains = fast_div((unsigned)chains);
  // four workgroups per CU, or a tile per wavefront; the same number of wavefronts for every batch and column group
  g.step_tiles = std::min(g.tiles, std::max(1, 4096 / chains));
  const long long waves = (long long)g.step_tiles * chains;
  hipLaunchKernelGGL((gemm_thin_kernel<T, STEPS, TN, ROWS>), dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, stream, g);
  return check_launch();
}
template <typename T, int STEPS, Rows ROWS>
int launch_width(ThinArgs<T>& g, int batch, hipStream_t stream) {
  return g.N <= 32 ? launch_cfg<T, STEPS, 1, ROWS>(g, batch, stream) : launch_cfg<T, STEPS, 2, ROWS>(g, batch, stream);
}
template <typename T, Rows ROWS>
int launch_depth(ThinArgs<T>& g, int batch, hipStream_t stream) {
  if (g.K <= 16) return launch_width<T, 1, ROWS>(g, batch, stream);
  if (g.K <= 32) return launch_width<T, 2, ROWS>(g, batch, stream);
  if constexpr (sizeof(T) == 2) return launch_width<T, 4, ROWS>(g, batch, stream);
  return TFX_ERR_UNSUPPORTED;
}

template <typename T>
int thin(const T* a, const T* b, T* c, const T* bias, int batch, int m, int n, int k, bool a_kc, bool b_kc, int act, hipStream_t stream) {
  ThinArgs<T> g{};
  g.a = a, g.b = b, g.c = c, g.bias = bias;
  g.M = m, g.N = n, g.K = k, g.b_kc = b_kc ? 1 : 0, g.act = act;
  g.strideA = (long long)m * k, g.strideB = (long long)n * k, g.strideC = (long long)m * n;
  g.total = (unsigned)g.strideA;
  if constexpr (sizeof(T) == 4)
    if (!a_kc) return launch_depth<T, kRowsM>(g, batch, stream);
  return launch_depth<T, kRowsK>(g, batch, stream);
}
template <typename T>
int thin_conv(const T* x, const T* w, T* y, const T* bias, int m, int n, int k, int act, hipStream_t stream, int h, int wd, int oh, int ow,
              int stride) {
  ThinArgs<T> g{};
  g.a = x, g.b = w, g.c = y, g.bias = bias;
  g.M = m, g.N = n, g.K = k, g.act = act;
  g.H = h, g.W = wd, g.stride = stride;
  g.by_ow = fast_div((unsigned)ow), g.by_oh = fast_div((unsigned)oh);
  g.total = (unsigned)((long long)m / (oh * ow) * h * wd * k);
  return launch_depth<T, kStrided>(g, 1, stream);
}

}  // namespace

int launch_gemm_thin(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, bool a_kc, bool b_kc,
                     int act, hipStream_t stream) {
  return thin<float>(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream);
}
int launch_gemm_thin_f16(const uint16_t* a, const uint16_t* b, uint16_t* c, const uint16_t* bias, int m, int n, int k, bool b_kc, int act,
                         hipStream_t stream) {
  typedef _Float16 H;
  return thin<H>(reinterpret_cast<const H*>(a), reinterpret_cast<const H*>(b), reinterpret_cast<H*>(c), reinterpret_cast<const H*>(bias),
                 1, m, n, k, true, b_kc, act, stream);
}
int launch_conv1x1_thin(const float* x, const float* w, float* y, const float* bias, int m, int n, int k, int act, hipStream_t stream, int h,
                        int wd, int oh, int ow, int stride) {
  return thin_conv<float>(x, w, y, bias, m, n, k, act, stream, h, wd, oh, ow, stride);
}
int launch_conv1x1_thin_f16(const uint16_t* x, const uint16_t* w, uint16_t* y, const uint16_t* bias, int m, int n, int k, int act,
                            hipStream_t stream, int h, int wd, int oh, int ow, int stride) {
  typedef _Float16 H;
  return thin_conv<H>(reinterpret_cast<const H*>(x), reinterpret_cast<const H*>(w), reinterpret_cast<H*>(y), reinterpret_cast<const H*>(bias),
                      m, n, k, act, stream, h, wd, oh, ow, stride);
}

}  // namespace tfx
