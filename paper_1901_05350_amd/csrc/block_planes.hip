// A depthwise-separable block of a batch (depthwise 3x3 + bias + relu6, pointwise 1x1 + bias + clamp, fp32) as two launches
// that hand the depthwise output over as bf16 planes: the blocks behind the early ones of the MobileNet forward pass.
//
// The pointwise layer is a product on the bf16 matrix cores with three-way split operands (split.h).  There the split costs
// 7 vector instructions per element of a tile in every workgroup that stages the tile, which is what bounds the kernels of
// gemm.hip and gemm_direct.hip at these sizes: an element of the depthwise output is staged by N / 64 or N / 128
// workgroups, one of the filter by M / 64.  Here every element is split once.  The depthwise kernel writes its output as
// the three planes hi, mid, lo (6 bytes a value instead of 4), extra workgroups of the same launch do the same with the
// pointwise filter, and the product kernel only moves planes through LDS into the matrix cores.  It is bound by these and,
// at few tiles, by memory latency.
// Planes are stored by k-slices of 32: plane p, slice s, row r: 32 bf16 at element ((3 s + p) rows + r) 32, so that the
// rows of a tile are one contiguous piece per plane and slice.
//
// Values that the split does not carry (split.h): results that are Inf or NaN are computed again with the fp32
// instructions, and so are small ones where one of a wavefront's rows or columns holds a tiny value, which is looked for in
// the planes when a result is small.  So that it can be seen there, a depthwise output below the smallest bf16 becomes
// that one (2^-133; it loses no more than other tiny values do).  Depthwise outputs are at most 6; a filter value of 2^20 or
// more is stored as NaN, which makes its results NaN and has them computed again.  Operands of the second computation are
// the sums of their planes, which are exact, except for tiny and non-finite ones, computed again from the input.
#include "split.h"

namespace tfx {
namespace {

constexpr int kXcds = 8, kSlice = 32;
typedef float v4f __attribute__((ext_vector_type(4)));

struct PlanesArgs {
  const float *x, *dw_w, *dw_b, *pw_w, *pw_b;
  float* y;
  unsigned short *a, *b;  // planes of the depthwise output [M, C] and of the filter transposed [N, C]
  int H, W, C, OH, OW, N, M, pt, pl;
  int strips, dw_total, dw_blocks;
  int pw_act;
  int tiles_m, tiles_n;
};

__device__ __forceinline__ float dw_value(const PlanesArgs& g, int S, int row, int c) {  // depthwise output, one value
  const int t = row / g.OW, n = t / g.OH, oh = t - n * g.OH, ow = row - t * g.OW;
  float acc = g.dw_b[c];
  for (int kh = 0; kh < 3; ++kh)
    for (int kw = 0; kw < 3; ++kw) {
      const int ih = oh * S - g.pt + kh, iw = ow * S - g.pl + kw;
      if (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W)
        acc += g.x[(((size_t)n * g.H + ih) * g.W + iw) * g.C + c] * g.dw_w[(kh * 3 + kw) * g.C + c];
    }
  return apply_act(acc, TFX_ACT_RELU6);
}

// a float of at least +0: positive ones below 2^-133 become 2^-133
__device__ __forceinline__ float seen_in_planes(float v) {
  const unsigned bits = __float_as_uint(v);
  return __uint_as_float(max(bits, min(bits << 16, 1u << 16)));
}

// Workgroups 0 ... dw_blocks - 1: the depthwise layer as in depthwise.hip (a lane owns four channels of RS output rows of
// one column).  The others: the pointwise filter, 64 columns x 32 k each.
template <int S, int RS>
__global__ __launch_bounds__(256) void depthwise_planes_kernel(PlanesArgs g) {
  int bid = blockIdx.x;
  const int C = g.C;
  if (bid >= g.dw_blocks) {
    bid -= g.dw_blocks;
    const int slices = C / kSlice, slice = bid % slices, n0 = bid / slices * 64;
    // 16 columns x 4 octets of k per wavefront: a column's 32 k are one 64-byte piece of a plane
    const int lane = threadIdx.x % 64, n = n0 + threadIdx.x / 64 * 16 + lane % 16, o = lane / 16;
    const float* p = g.pw_w + (size_t)(slice * kSlice + 8 * o) * g.N + n;
    floatx4 v[2];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e / 4][e % 4] = p[(size_t)e * g.N];
    splitx4 part[2][kParts];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float w = v[q][e];  // (a tiny filter value is found in the filter itself)
        v[q][e] = fabsf(w) < 0x1p20f ? w : NAN;
      }
      unsigned low = 0;  // (what is lost is looked for in the planes and the filter)
      split4(v[q], part[q], low);
    }
#pragma unroll
    for (int q = 0; q < kParts; ++q) {
      typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
      *reinterpret_cast<u32x4*>(g.b + ((size_t)(3 * slice + q) * g.N + n) * kSlice + 8 * o) =
          u32x4{part[0][q][0], part[0][q][1], part[1][q][0], part[1][q][1]};
    }
  } else {
    constexpr int IR = (RS - 1) * S + 3;
    {
      const int nb = g.dw_blocks, q = nb / kXcds, rem = nb % kXcds;
      const int xcd = bid % kXcds;
      bid = xcd * q + (xcd < rem ? xcd : rem) + bid / kXcds;
    }
    const int idx = bid * 256 + threadIdx.x;
    if (idx < g.dw_total) {
      const int C4 = C / 4, c4 = idx % C4;
      int r = idx / C4;
      const int ow = r % g.OW;
      r /= g.OW;
      const int strip = r % g.strips, n = r / g.strips;
      const float* xn = g.x + (size_t)n * g.H * g.W * C + 4 * c4;
      const int iw0 = ow * S - g.pl;
      const bool in0 = iw0 >= 0 && iw0 < g.W, in1 = iw0 + 1 >= 0 && iw0 + 1 < g.W, in2 = iw0 + 2 >= 0 && iw0 + 2 < g.W;
      const int oh0 = strip * RS, ih0 = oh0 * S - g.pt;
      v4f win[IR][3];
      const v4f z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < IR; ++i) {
        const int ih = ih0 + i;
        const bool rok = ih >= 0 && ih < g.H;
        const float* p = xn + ((long long)ih * g.W + iw0) * C;
        win[i][0] = (rok && in0) ? *reinterpret_cast<const v4f*>(p) : z;
        win[i][1] = (rok && in1) ? *reinterpret_cast<const v4f*>(p + C) : z;
        win[i][2] = (rok && in2) ? *reinterpret_cast<const v4f*>(p + 2 * C) : z;
      }
      v4f wt[9];
#pragma unroll
      for (int t = 0; t < 9; ++t) wt[t] = *reinterpret_cast<const v4f*>(g.dw_w + (size_t)t * C + 4 * c4);
      const v4f bv = *reinterpret_cast<const v4f*>(g.dw_b + 4 * c4);
      const ActClamp clamp = make_act(TFX_ACT_RELU6);
      unsigned short* const to = g.a + (size_t)(3 * (c4 / 8)) * g.M * kSlice + 4 * (c4 % 8);
#pragma unroll
      for (int o = 0; o < RS; ++o) {
        if (oh0 + o >= g.OH) break;
        v4f acc = bv;
#pragma unroll
        for (int kh = 0; kh < 3; ++kh)
#pragma unroll
          for (int kw = 0; kw < 3; ++kw) acc += win[o * S + kh][kw] * wt[kh * 3 + kw];
        floatx4 out;
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = seen_in_planes(apply_act(acc[e], clamp));
        splitx4 part[kParts];
        unsigned low = 0;
        split4(out, part, low);
        const size_t row = ((size_t)n * g.OH + oh0 + o) * g.OW + ow;
#pragma unroll
        for (int q = 0; q < kParts; ++q) *reinterpret_cast<splitx4*>(to + ((size_t)q * g.M + row) * kSlice) = part[q];
      }
    }
  }
}

// y = clamp(A W + bias) from the planes: WAVES_M x WAVES_N wavefronts of TM x TN blocks of 32 x 32, k-slices of 32
// double-buffered in LDS.  As in the binary16 pipeline (gemm_f16.hip), after every few matrix instructions one 16-byte slot
// of slice kt + 1 moves from registers to the other buffer and is refilled from slice kt + 2: one barrier per slice.
// LDS: rows of 64 bytes per plane, their four 16-byte pieces turned by row / 8, so that the fragment reads of 32
// consecutive rows spread over all banks.
template <int S, int WAVES_M, int WAVES_N, int TM, int TN>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, 2) void pointwise_planes_kernel(PlanesArgs g) {
  constexpr int NT = 64 * WAVES_M * WAVES_N, BM = 32 * TM * WAVES_M, BN = 32 * TN * WAVES_N;
  constexpr int SA = BM * 4 * kParts / NT, SB = BN * 4 * kParts / NT, SLOTS = SA + SB;
  static_assert(BM * 4 * kParts % NT == 0 && BN * 4 * kParts % NT == 0, "loader shape");
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  constexpr int kA = BM * 64 * kParts, kBuf = kA + BN * 64 * kParts;
  __shared__ __align__(16) char lds[2 * kBuf];

  const int bid = blockIdx.x, total = gridDim.x;
  const int q8 = total / kXcds, rem = total % kXcds, xcd = bid % kXcds;
  const int vid = xcd * q8 + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int m0 = vid / g.tiles_n * BM, n0 = vid % g.tiles_n * BN;
  const int M = g.M, N = g.N, nk = g.C / kSlice;
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, li = lane % 32, h = lane / 32;
  const int wm0 = wave / WAVES_N * 32 * TM, wn0 = wave % WAVES_N * 32 * TN;
  auto at = [](int row, int piece) { return row * 64 + ((piece ^ ((row / 8) & 3)) * 16); };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  float bv[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) bv[j] = g.pw_b[n0 + wn0 + 32 * j + li];

  // slot w: A's for w < SA.  Byte offset in its planes at slice 0, and in LDS
  unsigned from[SLOTS];
  int to[SLOTS];
#pragma unroll
  for (int w = 0; w < SLOTS; ++w) {
    const bool is_a = w < SA;
    const int s = tid + (is_a ? w : w - SA) * NT, rows = is_a ? BM : BN;
    const int p = s / (rows * 4), row = s / 4 % rows, piece = s % 4;
    const int r = is_a ? min(m0 + row, M - 1) : n0 + row;  // rows past M repeat the last one (never stored)
    from[w] = ((unsigned)p * (unsigned)(is_a ? M : N) + (unsigned)r) * 64u + 16u * piece;
    to[w] = (is_a ? 0 : kA) + p * rows * 64 + at(row, piece);
  }
  u32x4 reg[SLOTS];
  auto load = [&](int w, int kt) __attribute__((always_inline)) {
    const char* const base = reinterpret_cast<const char*>(w < SA ? g.a : g.b) + (size_t)kt * (kParts * 64) * (size_t)(w < SA ? M : N);
    reg[w] = *reinterpret_cast<const u32x4*>(base + from[w]);
  };
  auto store = [&](int w, int buf) __attribute__((always_inline)) { *reinterpret_cast<u32x4*>(lds + buf * kBuf + to[w]) = reg[w]; };
#pragma unroll
  for (int w = 0; w < SLOTS; ++w) load(w, 0);
#pragma unroll
  for (int w = 0; w < SLOTS; ++w) {
    store(w, 0);
    load(w, min(1, nk - 1));
  }
  __syncthreads();

  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1, next = min(kt + 2, nk - 1);  // the last two rounds fetch the last slice again (unused)
    const char* const buf = lds + cur * kBuf;
    bf16x8 fa[2][TM][kParts], fb[2][TN][kParts];
    auto read = [&](int step) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int p = 0; p < kParts; ++p)
          fa[step][i][p] = *reinterpret_cast<const bf16x8*>(buf + p * BM * 64 + at(wm0 + 32 * i + li, 2 * step + h));
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int p = 0; p < kParts; ++p)
          fb[step][j][p] = *reinterpret_cast<const bf16x8*>(buf + kA + p * BN * 64 + at(wn0 + 32 * j + li, 2 * step + h));
    };
    read(0);
    constexpr int MF = kSplitPasses * TM * TN, ALL = 2 * MF;
#pragma unroll
    for (int step = 0; step < 2; ++step) {
      if (step == 0) read(1);
      __builtin_amdgcn_sched_barrier(0);  // keep those LDS reads ahead of this step's matrix instructions
#pragma unroll
      for (int x = 0; x < MF; ++x) {
        const int pass = x / (TM * TN), i = x / TN % TM, j = x % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[step][i][split_pass_a(pass)], fb[step][j][split_pass_b(pass)], acc[i][j], 0, 0, 0);
        const int t = step * MF + x;
#pragma unroll
        for (int w = t * SLOTS / ALL; w < (t + 1) * SLOTS / ALL; ++w) {
          store(w, cur ^ 1);
          load(w, next);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
  }

  const float limit = small_limit(g.C);
  unsigned most = 0;
  float least = INFINITY;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        see_result(most, acc[i][j][v]);
        least = fminf(least, fabsf(acc[i][j][v] + bv[j]));
      }
  // eight depthwise outputs of a row from their planes; `bad`: one of them is tiny or not finite
  auto depthwise8 = [&](int row, int k, float (&f)[8], bool& bad) __attribute__((always_inline)) {
    const unsigned short* const p = g.a + ((size_t)(3 * (k / kSlice)) * M + row) * kSlice + k % kSlice;
    typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
    const u16x8 hi = *reinterpret_cast<const u16x8*>(p), mid = *reinterpret_cast<const u16x8*>(p + (size_t)M * kSlice),
                lo = *reinterpret_cast<const u16x8*>(p + (size_t)2 * M * kSlice);
    bad = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float top = __uint_as_float((unsigned)hi[e] << 16);
      f[e] = (__uint_as_float((unsigned)lo[e] << 16) + __uint_as_float((unsigned)mid[e] << 16)) + top;
      bad = bad || is_tiny(top) || !__builtin_isfinite(top);
    }
  };
  bool tiny = false;
  if (__builtin_amdgcn_ballot_w64(least < limit) != 0) {  // look through this wavefront's rows and columns
    bool found = false;
#pragma unroll 1
    for (int at = 8 * lane; at < 32 * TM * g.C; at += 8 * 64) {
      const int row = min(m0 + wm0 + at / g.C, M - 1), k = at % g.C;
      const u32x4 hi = *reinterpret_cast<const u32x4*>(g.a + ((size_t)(3 * (k / kSlice)) * M + row) * kSlice + k % kSlice);
#pragma unroll
      for (int e = 0; e < 4; ++e) found = found || is_tiny(__uint_as_float(hi[e] << 16)) || is_tiny(__uint_as_float(hi[e] & 0xffff0000u));
    }
#pragma unroll 1
    for (int at = 4 * lane; at < 32 * TN * g.C; at += 4 * 64)
      found = found || any_tiny(*reinterpret_cast<const floatx4*>(g.pw_w + (size_t)(at / (32 * TN)) * N + n0 + wn0 + at % (32 * TN)));
    tiny = __builtin_amdgcn_ballot_w64(found) != 0;
  }
  if (tiny || __builtin_amdgcn_ballot_w64(overflowed(most)) != 0) {
#pragma unroll 1
    for (int block = 0; block < TM * TN; ++block) {
      auto wanted = [&](int x, int v) __attribute__((always_inline)) {
        const float r = acc[x / TN][x % TN][v];
        return !__builtin_isfinite(r) || (tiny && fabsf(r + bv[x % TN]) < limit);
      };
      bool any = false;
#pragma unroll
      for (int x = 0; x < TM * TN; ++x)
        if (x == block)
#pragma unroll
          for (int v = 0; v < 16; ++v) any = any || wanted(x, v);
      if (__builtin_amdgcn_ballot_w64(any) == 0) continue;
      const int row = min(m0 + wm0 + 32 * (block / TN) + li, M - 1), col = n0 + wn0 + 32 * (block % TN) + li;
      floatx16 exact;
#pragma unroll
      for (int v = 0; v < 16; ++v) exact[v] = 0.f;
#pragma unroll 1
      for (int k = 8 * h; k < g.C; k += 16) {
        float fa[8], fb[8];
        bool bad;
        depthwise8(row, k, fa, bad);
#pragma unroll
        for (int e = 0; e < 8; ++e) fb[e] = g.pw_w[(size_t)(k + e) * N + col];
        if (bad) {
#pragma unroll 1
          for (int e = 0; e < 8; ++e) {
            const float v = dw_value(g, S, row, k + e);
#pragma unroll
            for (int w = 0; w < 8; ++w) fa[w] = w == e ? v : fa[w];
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) exact = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[e], fb[e], exact, 0, 0, 0);
      }
#pragma unroll
      for (int x = 0; x < TM * TN; ++x)
        if (x == block)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (wanted(x, v)) acc[x / TN][x % TN][v] = exact[v];
    }
  }
  const ActClamp clamp = make_act(g.pw_act);
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = m0 + wm0 + 32 * i + 8 * (v / 4) + 4 * h + v % 4;
        if (row < M) g.y[(size_t)row * N + n0 + wn0 + 32 * j + li] = apply_act(acc[i][j][v] + bv[j], clamp);
      }
}

template <int S, int RS>
int launch_dw(PlanesArgs& g, int n, hipStream_t stream) {
  g.strips = (g.OH + RS - 1) / RS;
  const long long total = (long long)n * g.strips * g.OW * (g.C / 4);
  if (total > 0x7fffff00LL) return TFX_ERR_UNSUPPORTED;
  g.dw_total = (int)total;
  g.dw_blocks = (int)((total + 255) / 256);
  hipLaunchKernelGGL((depthwise_planes_kernel<S, RS>), dim3((unsigned)(g.dw_blocks + g.C / kSlice * (g.N / 64))), dim3(256), 0, stream, g);
  return check_launch();
}

template <int S, int WAVES_M, int WAVES_N, int TM, int TN>
int launch_pw(PlanesArgs& g, hipStream_t stream) {
  constexpr int BM = 32 * TM * WAVES_M, BN = 32 * TN * WAVES_N;
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = g.N / BN;
  hipLaunchKernelGGL((pointwise_planes_kernel<S, WAVES_M, WAVES_N, TM, TN>), dim3((unsigned)(g.tiles_m * g.tiles_n)),
                     dim3(64 * WAVES_M * WAVES_N), 0, stream, g);
  return check_launch();
}

template <int S>
int launch_block(PlanesArgs& g, int n, hipStream_t stream) {
  const long long px = (long long)g.M * (g.C / 4), want = 256LL * 256 * 4;
  int rc;
  if (S == 2) rc = px / 2 >= want / 4 ? launch_dw<S, 2>(g, n, stream) : launch_dw<S, 1>(g, n, stream);
  else if (g.OH % 7 == 0 && (px / 7 >= want * 3 / 4 || (g.OH == 7 && px / 7 >= want / 4))) rc = launch_dw<S, S == 1 ? 7 : 1>(g, n, stream);
  else if (px / 4 >= want / 4) rc = launch_dw<S, S == 1 ? 4 : 1>(g, n, stream);
  else if (px / 2 >= want / 4) rc = launch_dw<S, S == 1 ? 2 : 1>(g, n, stream);
  else rc = launch_dw<S, 1>(g, n, stream);
  if (rc) return rc;
  const long long tiles = (g.M + 63LL) / 64 * (g.N / 64);
  if (tiles < 160) return launch_pw<S, 1, 2, 1, 1>(g, stream);    // 32 x 64, 2 wavefronts
  if (tiles >= 1000) return launch_pw<S, 2, 2, 2, 1>(g, stream);  // 128 x 64, 4 wavefronts
  return launch_pw<S, 2, 2, 1, 1>(g, stream);                                   // 64 x 64, 4 wavefronts
}

}  // namespace

size_t planes_elems(long long rows, int c) { return (size_t)rows * c * kParts; }

bool separable_planes_supported(long long rows, int c, int n, int stride, const void* x, const void* dw_w, const void* dw_b,
                                const void* pw_w, const void* pw_b, const void* y) {
  auto al16 = [](const void* p) { return p != nullptr && reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  return c % kSlice == 0 && n % 64 == 0 && (stride == 1 || stride == 2) && rows * 192 < (1LL << 32) && rows * n < (1LL << 31) &&
         al16(x) && al16(dw_w) && al16(dw_b) && al16(pw_w) && al16(pw_b) && al16(y);
}

int launch_separable_planes(const float* x, const float* dw_w, const float* dw_b, const float* pw_w, const float* pw_b, float* y,
                            void* a_planes, void* b_planes, int batch, int h, int w, int c, int n, int oh, int ow, int stride, int pt,
                            int pl, int pw_act, hipStream_t stream) {
  PlanesArgs g{};
  g.x = x, g.dw_w = dw_w, g.dw_b = dw_b, g.pw_w = pw_w, g.pw_b = pw_b, g.y = y;
  g.a = static_cast<unsigned short*>(a_planes), g.b = static_cast<unsigned short*>(b_planes);
  g.H = h, g.W = w, g.C = c, g.OH = oh, g.OW = ow, g.N = n, g.M = batch * oh * ow, g.pt = pt, g.pl = pl;
  g.pw_act = pw_act;
  return stride == 1 ? launch_block<1>(g, batch, stream) : launch_block<2>(g, batch, stream);
}

}  // namespace tfx
