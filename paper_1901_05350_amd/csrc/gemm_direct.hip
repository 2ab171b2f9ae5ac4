// Products and convolutions of up to a few output tiles per CU, any layout, size and alignment, on float and on 16-bit float
// storage:  C[b] = act( op(A[b]) * op(B[b]) + bias )  (Listing 2, Section 4.1; conv2d: the NHWC index order of Section 4.1).
//
// For such outputs a kernel that walks through K slice by slice is a serial chain: load, (split,) LDS, barrier, multiply, at
// 64 x 64 tiles 0.9 us per 32 k of floats.  Here the wavefronts of a workgroup split K instead: wavefront w takes k-steps
// w, w + WAVES, ... of 16, loads its operands of two steps ahead straight into registers and multiplies the whole
// 32 TM x 32 TN tile; nothing is shared until the partial tiles are added through LDS at the end.
// Floats are split in registers (split.h), every operand element once per workgroup as it would be on the way into LDS, and
// the split's vector instructions (7 per element) are what bounds them; halfs are multiplied as they are
// (v_mfma_f32_32x32x16_f16), bound by what L1 and L2 deliver.
#include "ragged.h"
#include "split.h"

#include <type_traits>

namespace tfx {
namespace {

constexpr int kXcds = 8;

enum Source { kRowsK, kRowsM, kConv };  // A stored [M,K]; stored [K,M]; the window view of an NHWC image

template <typename T>
struct DirectArgs {
  const T *a, *b, *bias;
  T* c;
  int M, N, K;                // K: channels per tap for a convolution
  unsigned a_total, b_total;  // elements of one batch's operand
  long long strideA, strideB, strideC;
  int tiles_m, tiles_n, total_blocks, m_fastest, act;
  int steps, whole_steps;     // k-steps in all; the first ones, whose octets lie inside K (a tap), take the lean loads
  // convolution only: k runs over (tap, channel) with the channels of a tap padded to a multiple of 8
  int H, W, fw, taps, sh, sw, pt, pl;
  FastDiv by_cp, by_fw, by_ow, by_oh;
};

__device__ __align__(16) float kZeros[4] = {0.f, 0.f, 0.f, 0.f};  // never written (not const: same address space as x)

// 8 consecutive k of one row or column: one or two chunks of 16 bytes
template <typename T>
struct Octet {
  static constexpr int kChunks = sizeof(T) / 2, kPer = 8 / kChunks;
  ragged_u32x4 chunk[kChunks];
};
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef unsigned u32_any __attribute__((aligned(2)));

template <typename T, Source A_SRC, bool B_KC, int TM, int TN, int WAVES>
__global__ __launch_bounds__(64 * WAVES, TM * TN == 1 && A_SRC == kConv ? 4 : WAVES / 4) void gemm_direct_kernel(DirectArgs<T> g) {
  constexpr bool CONV = A_SRC == kConv, HALF = sizeof(T) == 2;
  typedef Octet<T> Oct;
  constexpr int PER = Oct::kPer;
  // Halfs whose rows (columns) are the contiguous direction are loaded two at a time, so a lane's two blocks of 32 rows
  // are interleaved: row x of block i is row 2 x + i of the tile (else 32 i + x).
  constexpr bool PAIR_M = HALF && A_SRC == kRowsM && TM == 2, PAIR_N = HALF && !B_KC && TN == 2;
  static_assert(!HALF || B_KC || TN == 2, "[K,N] halfs are loaded in pairs");
  constexpr int QUADS = TM * TN * 4;                       // accumulator quads of a lane
  constexpr int OWN = QUADS / WAVES > 0 ? QUADS / WAVES : 1;  // quads a thread adds up at the end
  static_assert(QUADS % WAVES == 0, "equal shares");
  __shared__ __align__(16) floatx4 red[WAVES * QUADS * 64];  // partial tiles: [wavefront][quad][lane]

  const int bid = blockIdx.x;
  const int q8 = g.total_blocks / kXcds, rem = g.total_blocks % kXcds;
  const int xcd = bid % kXcds;
  const int vid = xcd * q8 + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int tiles = g.tiles_m * g.tiles_n;
  const int batch = vid / tiles, t = vid % tiles;
  const int tile_m = g.m_fastest ? t % g.tiles_m : t / g.tiles_n;
  const int tile_n = g.m_fastest ? t / g.tiles_m : t % g.tiles_n;
  const int tid = threadIdx.x, lane = tid % 64, li = lane % 32, h = lane / 32;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int m0 = tile_m * 32 * TM, n0 = tile_n * 32 * TN;
  const T* const A = g.a + (size_t)batch * g.strideA;
  const T* const B = g.b + (size_t)batch * g.strideB;
  T* const C = g.c + (size_t)batch * g.strideC;

  // rows and columns past the matrix repeat the last one (they only feed outputs that are not stored)
  int arow[TM], bcol[TN], origin[TM], ih0[TM], iw0[TM];
  unsigned seen[TM];  // filter taps inside the image, one bit each (lean loads only)
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    seen[i] = 0;
    arow[i] = min(m0 + (PAIR_M ? 2 * li : 32 * i + li), g.M - (PAIR_M ? 2 : 1));
    if constexpr (CONV) {
      const unsigned r = (unsigned)arow[i], r2 = div_by(r, g.by_ow), n = div_by(r2, g.by_oh);
      ih0[i] = (int)(r2 - n * g.by_oh.d) * g.sh - g.pt;
      iw0[i] = (int)(r - r2 * g.by_ow.d) * g.sw - g.pl;
      origin[i] = (((int)n * g.H + ih0[i]) * g.W + iw0[i]) * g.K;
      if (g.whole_steps > 0)
        for (int tap = 0, kh = 0, kw = 0; tap < g.taps; ++tap) {
          if (ih0[i] + kh >= 0 && ih0[i] + kh < g.H && iw0[i] + kw >= 0 && iw0[i] + kw < g.W) seen[i] |= 1u << tap;
          if (++kw == g.fw) kw = 0, ++kh;
        }
    }
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) bcol[j] = min(n0 + (PAIR_N ? 2 * li : 32 * j + li), g.N - (PAIR_N ? 2 : 1));
  // a pair at the very end of an odd number of rows / columns starts one early
  const bool late_m = PAIR_M && m0 + 2 * li > arow[0], late_n = PAIR_N && n0 + 2 * li > bcol[0];

  // where a lane's octet of a step lies: `valid` k from channel c of filter tap `tap` on (a matrix is one tap)
  struct Place {
    int tap, c, valid, kh, kw;
  };
  auto place = [&](int step) __attribute__((always_inline)) {
    Place p{0, 16 * step + 8 * h, 0, 0, 0};
    if constexpr (CONV) {
      p.tap = (int)div_by((unsigned)p.c, g.by_cp);
      p.c -= p.tap * (int)g.by_cp.d;
      p.kh = (int)div_by((unsigned)p.tap, g.by_fw);
      p.kw = p.tap - p.kh * g.fw;
    }
    p.valid = !CONV || p.tap < g.taps ? g.K - p.c : 0;
    return p;
  };
  auto inside = [&](const Place& p, int i) __attribute__((always_inline)) {
    const int ih = ih0[i] + p.kh, iw = iw0[i] + p.kw;
    return p.valid > 0 && ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
  };
  auto chunk = [&](const T* base, bool in, unsigned off, unsigned total) __attribute__((always_inline)) {
    return load16(base + min(in ? off : 0u, total - (unsigned)PER));
  };
  auto a_offset = [&](const Place& p, int i) __attribute__((always_inline)) {
    return CONV ? (unsigned)(origin[i] + (p.kh * g.W + p.kw) * g.K + p.c) : (unsigned)arow[i] * (unsigned)g.K + (unsigned)p.c;
  };
  Oct a[2][TM], b[2][TN];  // raw operands of two steps
  // The octets of an operand with contiguous rows / columns, lane offsets `offset` (one per octet; PAIR: one for both) from
  // `at`, which is uniform: a uniform address per k plus a lane's own 32-bit offset, so that no vector instruction goes
  // into addresses.  Only the first `valid` k are fetched (the others repeat the first).
  auto columns = [&](auto pair, bool late, const T* at, int ld, const unsigned* offset, int count, int valid, Oct* o) __attribute__((always_inline)) {
    if constexpr (decltype(pair)::value) {
      unsigned v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = *reinterpret_cast<const u32_any*>(at + offset[0]);
        if (e + 1 < valid) at += ld;
      }
      if (__builtin_amdgcn_ballot_w64(late) != 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = late ? v[e] >> 16 : v[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[0].chunk[0][e] = __builtin_amdgcn_perm(v[2 * e + 1], v[2 * e], 0x05040100u);
        o[1].chunk[0][e] = __builtin_amdgcn_perm(v[2 * e + 1], v[2 * e], 0x07060302u);
      }
    } else {
#pragma unroll
      for (int i = 0; i < count; ++i) {
        T v[8];
        const T* p = at;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = p[offset[i]];
          if (e + 1 < valid) p += ld;
        }
        o[i] = __builtin_bit_cast(Oct, v);
      }
    }
  };
  unsigned a_lane[TM], b_lane[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
    a_lane[i] = A_SRC == kRowsM ? 8u * h * (unsigned)g.M + (unsigned)arow[i] : (unsigned)arow[i] * (unsigned)g.K + 8u * h;
#pragma unroll
  for (int j = 0; j < TN; ++j)
    b_lane[j] = B_KC ? (unsigned)bcol[j] * (unsigned)g.K + 8u * h : 8u * h * (unsigned)g.N + (unsigned)bcol[j];
  auto load = [&](int step, Oct (&oa)[TM], Oct (&ob)[TN]) __attribute__((always_inline)) {
    if (step < g.whole_steps) {
      int tap = 0, tap_offset = 0;
      if constexpr (CONV) {
        tap = (int)div_by(16u * (unsigned)step, g.by_cp);
        const int kh = (int)div_by((unsigned)tap, g.by_fw), kw = tap - kh * g.fw;
        tap_offset = (kh * g.W + kw) * g.K + 16 * step - tap * g.K;
      }
      if constexpr (A_SRC == kRowsM) columns(std::bool_constant<PAIR_M>{}, late_m, A + (size_t)(16 * step) * g.M, g.M, a_lane, TM, 8, oa);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if constexpr (A_SRC == kRowsM) continue;
        const T* p = A + 16 * step + a_lane[i];
        if constexpr (CONV) p = A + (ptrdiff_t)(origin[i] + tap_offset + 8 * h);
        const bool in = !CONV || ((seen[i] >> tap) & 1u) != 0;
#pragma unroll
        for (int q = 0; q < Oct::kChunks; ++q) oa[i].chunk[q] = load16(in ? p + PER * q : reinterpret_cast<const T*>(kZeros));
      }
      if constexpr (B_KC) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < Oct::kChunks; ++q) ob[j].chunk[q] = load16(B + 16 * step + b_lane[j] + PER * q);
      } else {
        columns(std::bool_constant<PAIR_N>{}, late_n, B + (size_t)(16 * step) * g.N, g.N, b_lane, TN, 8, ob);
      }
      return;
    }
    // a step at the end of K, or across taps: a lane's own place, masked later
    const Place p = place(step);
    if constexpr (A_SRC == kRowsM) {
      unsigned at[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) at[i] = (unsigned)arow[i];
      columns(std::bool_constant<PAIR_M>{}, late_m, A + (size_t)(p.valid > 0 ? p.c : 0) * g.M, g.M, at, TM, p.valid, oa);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (A_SRC == kRowsM) continue;
      const bool in = CONV ? inside(p, i) : p.valid > 0;
#pragma unroll
      for (int q = 0; q < Oct::kChunks; ++q) oa[i].chunk[q] = chunk(A, in && p.valid > PER * q, a_offset(p, i) + PER * q, g.a_total);
    }
    if constexpr (B_KC) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < Oct::kChunks; ++q)
          ob[j].chunk[q] = chunk(B, p.valid > PER * q, (unsigned)bcol[j] * (unsigned)g.K + (unsigned)(p.c + PER * q), g.b_total);
    } else {
      unsigned at[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) at[j] = (unsigned)bcol[j];
      columns(std::bool_constant<PAIR_N>{}, late_n, B + (size_t)(p.valid > 0 ? p.tap * g.K + p.c : 0) * g.N, g.N, at, TN, p.valid, ob);
    }
  };
  // ... and what makes the registers the operands: chunks fetched early shifted, k past the end and pixels outside zeroed
  auto settle = [&](int step, Oct (&oa)[TM], Oct (&ob)[TN]) __attribute__((always_inline)) {
    if (step < g.whole_steps) return;
    const Place p = place(step);
    auto fix = [&](Oct& o, bool chunks, bool in, unsigned off, unsigned total) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < Oct::kChunks; ++q) {
        if (chunks) {
          const unsigned at = off + PER * q, early = in && p.valid > PER * q ? at - min(at, total - (unsigned)PER) : 0u;
          if (__builtin_amdgcn_ballot_w64(early != 0) != 0) o.chunk[q] = shift_down<T>(o.chunk[q], early);
        }
        o.chunk[q] &= first_elements<T>(in ? p.valid - PER * q : 0);
      }
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
      fix(oa[i], A_SRC != kRowsM, CONV ? inside(p, i) : p.valid > 0, A_SRC == kRowsM ? 0u : a_offset(p, i), g.a_total);
#pragma unroll
    for (int j = 0; j < TN; ++j)
      fix(ob[j], B_KC, p.valid > 0, B_KC ? (unsigned)bcol[j] * (unsigned)g.K + (unsigned)p.c : 0u, g.b_total);
  };

  floatx16 acc[TM][TN];
  SplitGuard guard;
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  };
  auto split8 = [&](const Oct& o, bf16x8 (&part)[kParts]) __attribute__((always_inline)) {
    splitx4 half[2][kParts];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const floatx4 v = __builtin_bit_cast(floatx4, o.chunk[q % Oct::kChunks]);
      guard.split(v, half[q]);
    }
#pragma unroll
    for (int p = 0; p < kParts; ++p)
      part[p] = __builtin_bit_cast(bf16x8, ragged_u32x4{half[0][p][0], half[0][p][1], half[1][p][0], half[1][p][1]});
  };
  auto multiply = [&](int step, int next, Oct (&oa)[TM], Oct (&ob)[TN]) __attribute__((always_inline)) {
    settle(step, oa, ob);
    if constexpr (HALF) {
      h8 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = __builtin_bit_cast(h8, oa[i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = __builtin_bit_cast(h8, ob[j]);
      if (next < g.steps) load(next, oa, ob);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    } else {
      bf16x8 fa[TM][kParts], fb[TN][kParts];
#pragma unroll
      for (int i = 0; i < TM; ++i) split8(oa[i], fa[i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) split8(ob[j], fb[j]);
      if (next < g.steps) load(next, oa, ob);
#pragma unroll
      for (int s = 0; s < kSplitPasses; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][split_pass_a(s)], fb[j][split_pass_b(s)], acc[i][j], 0, 0, 0);
    }
  };

  clear();
  if (wave < g.steps) load(wave, a[0], b[0]);
  if (wave + WAVES < g.steps) load(wave + WAVES, a[1], b[1]);
  // The quads this thread adds up: quad ((i * 4) + v) * TN + j of lane l is column l % 32 of block j, rows
  // 8 v + 4 (l / 32) .. + 3 of block i.
  auto quad_col = [&](int quad) __attribute__((always_inline)) { return n0 + (PAIR_N ? 2 * li + quad % TN : 32 * (quad % TN) + li); };
  auto quad_row = [&](int quad, int r) __attribute__((always_inline)) {
    const int x = 8 * (quad / TN % 4) + 4 * h + r, i = quad / TN / 4;
    return m0 + (PAIR_M ? 2 * x + i : 32 * i + x);
  };
  float bias[OWN];
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    const int col = quad_col(wave * OWN + o);
    bias[o] = g.bias != nullptr && col < g.N ? (float)g.bias[col] : 0.f;
  }
  for (int step = wave; step < g.steps; step += 2 * WAVES) {
    multiply(step, step + 2 * WAVES, a[0], b[0]);
    if (step + WAVES < g.steps) multiply(step + WAVES, step + 3 * WAVES, a[1], b[1]);
  }

  auto add_up = [&](floatx4 (&sum)[OWN]) __attribute__((always_inline)) {  // partial tiles -> sum
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          red[(wave * QUADS + (i * 4 + v) * TN + j) * 64 + lane] =
              floatx4{acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]};
    __syncthreads();
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
      sum[o] = red[(wave * OWN + o) * 64 + lane];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) sum[o] += red[(w * QUADS + wave * OWN + o) * 64 + lane];
    }
  };
  floatx4 sum[OWN];
  add_up(sum);
  if constexpr (!HALF) {
    // values that the split does not carry (split.h): results that are Inf or NaN, and small ones if it lost bits of an operand
    // of this workgroup, once more with the fp32 instructions
    unsigned most = 0;
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
      for (int v = 0; v < 4; ++v) see_result(most, sum[o][v]);
    if (__syncthreads_or(guard.lost() || overflowed(most))) {
      const float limit = !__syncthreads_or(guard.lost()) ? 0.f : __syncthreads_or(guard.large()) ? INFINITY : small_limit(CONV ? g.K * g.taps : g.K);
      auto wanted = [&](int o, int v) __attribute__((always_inline)) {
        return !__builtin_isfinite(sum[o][v]) || fabsf(sum[o][v] + bias[o]) < limit;
      };
      bool any = false;
#pragma unroll
      for (int o = 0; o < OWN; ++o)
#pragma unroll
        for (int v = 0; v < 4; ++v) any = any || wanted(o, v);
      if (__syncthreads_or(any)) {
        clear();
        for (int step = wave; step < g.steps; step += WAVES) {
          load(step, a[0], b[0]);
          settle(step, a[0], b[0]);
#pragma unroll
          for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[0][i].chunk[e / PER][e % PER]),
                                                                 __uint_as_float(b[0][j].chunk[e / PER][e % PER]), acc[i][j], 0, 0, 0);
        }
        floatx4 exact[OWN];
        add_up(exact);
#pragma unroll
        for (int o = 0; o < OWN; ++o)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (wanted(o, v)) sum[o][v] = exact[o][v];
      }
    }
  }
  const ActClamp clamp = make_act(g.act);
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    const int quad = wave * OWN + o, col = quad_col(quad);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = quad_row(quad, r);
      if constexpr (PAIR_N && OWN % 2 == 0) {  // both columns of a pair in one store
        if (o % 2 == 1) continue;
        typedef _Float16 h2 __attribute__((ext_vector_type(2), aligned(2)));
        const h2 v = {(_Float16)apply_act(sum[o][r] + bias[o], clamp), (_Float16)apply_act(sum[o + 1][r] + bias[o + 1], clamp)};
        T* const p = C + (size_t)row * g.N + col;
        if (row < g.M && col + 1 < g.N) *reinterpret_cast<h2*>(p) = v;
        else if (row < g.M && col < g.N) *p = v[0];
      } else {
        if (row < g.M && col < g.N) C[(size_t)row * g.N + col] = (T)apply_act(sum[o][r] + bias[o], clamp);
      }
    }
  }
}

template <typename T, Source A_SRC, bool B_KC, int TM, int TN, int WAVES>
int launch(DirectArgs<T>& g, int batch, hipStream_t stream) {
  g.tiles_m = (g.M + 32 * TM - 1) / (32 * TM);
  g.tiles_n = (g.N + 32 * TN - 1) / (32 * TN);
  const long long total = (long long)batch * g.tiles_m * g.tiles_n;
  if (total > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  g.total_blocks = (int)total;
  g.m_fastest = g.N > g.M ? 1 : 0;
  hipLaunchKernelGGL((gemm_direct_kernel<T, A_SRC, B_KC, TM, TN, WAVES>), dim3((unsigned)total), dim3(64 * WAVES), 0, stream, g);
  return check_launch();
}

template <typename T, Source A_SRC, bool B_KC>
int launch_tile(DirectArgs<T>& g, int batch, hipStream_t stream, int form) {
  if (form == 0) return launch<T, A_SRC, B_KC, 2, 2, 8>(g, batch, stream);
  if (form == 1 || sizeof(T) == 2) return launch<T, A_SRC, B_KC, 1, 2, 4>(g, batch, stream);
  if constexpr (sizeof(T) == 4) return launch<T, A_SRC, B_KC, 1, 1, 4>(g, batch, stream);
}

template <typename T>
int gemm(const T* a, const T* b, T* c, const T* bias, int batch, int m, int n, int k, bool a_kc, bool b_kc, int act,
         hipStream_t stream, int form) {
  DirectArgs<T> g{};
  g.a = a, g.b = b, g.bias = bias, g.c = c;
  g.M = m, g.N = n, g.K = k, g.act = act;
  g.strideA = (long long)m * k, g.strideB = (long long)n * k, g.strideC = (long long)m * n;
  g.a_total = (unsigned)g.strideA, g.b_total = (unsigned)g.strideB;
  g.steps = (k + 15) / 16;
  // (a lane's byte offset has 32 bits)
  const bool lean = (a_kc ? (long long)m * k : 9LL * m) < (1LL << 30) && (b_kc ? (long long)n * k : 9LL * n) < (1LL << 30);
  g.whole_steps = lean ? k / 16 : 0;
  if (a_kc) return b_kc ? launch_tile<T, kRowsK, true>(g, batch, stream, form) : launch_tile<T, kRowsK, false>(g, batch, stream, form);
  return b_kc ? launch_tile<T, kRowsM, true>(g, batch, stream, form) : launch_tile<T, kRowsM, false>(g, batch, stream, form);
}

template <typename T>
int conv(const T* x, const T* w, const T* bias, T* y, int n, int h, int wd, int ci, int fh, int fw, int co, int oh, int ow,
         int sh, int sw, int pt, int pl, int act, hipStream_t stream, int form) {
  DirectArgs<T> g{};
  const int cp = (ci + 7) / 8 * 8;
  g.a = x, g.b = w, g.bias = bias, g.c = y;
  g.M = n * oh * ow, g.N = co, g.K = ci, g.act = act;
  g.a_total = (unsigned)((long long)n * h * wd * ci), g.b_total = (unsigned)((long long)fh * fw * ci * co);
  g.steps = (fh * fw * cp + 15) / 16;
  g.whole_steps = ci % 16 == 0 && fh * fw <= 32 && 9LL * co < (1LL << 30) ? g.steps : 0;  // a step inside one tap
  g.H = h, g.W = wd, g.fw = fw, g.taps = fh * fw, g.sh = sh, g.sw = sw, g.pt = pt, g.pl = pl;
  g.by_cp = fast_div((unsigned)cp), g.by_fw = fast_div((unsigned)fw), g.by_ow = fast_div((unsigned)ow), g.by_oh = fast_div((unsigned)oh);
  return launch_tile<T, kConv, false>(g, 1, stream, form);
}

}  // namespace

int launch_gemm_direct(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, bool a_kc,
                       bool b_kc, int act, hipStream_t stream, int form) {
  return gemm<float>(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream, form);
}
int launch_gemm_direct_f16(const uint16_t* a, const uint16_t* b, uint16_t* c, const uint16_t* bias, int batch, int m, int n,
                           int k, bool a_kc, bool b_kc, int act, hipStream_t stream, int form) {
  typedef _Float16 H;
  return gemm<H>(reinterpret_cast<const H*>(a), reinterpret_cast<const H*>(b), reinterpret_cast<H*>(c),
                 reinterpret_cast<const H*>(bias), batch, m, n, k, a_kc, b_kc, act, stream, form);
}
int launch_conv2d_gemm_direct(const float* x, const float* w, const float* bias, float* y, int n, int h, int wd, int ci, int fh,
                              int fw, int co, int oh, int ow, int sh, int sw, int pt, int pl, int act, hipStream_t stream, int form) {
  return conv<float>(x, w, bias, y, n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream, form);
}
int launch_conv2d_gemm_direct_f16(const uint16_t* x, const uint16_t* w, const uint16_t* bias, uint16_t* y, int n, int h, int wd,
                                  int ci, int fh, int fw, int co, int oh, int ow, int sh, int sw, int pt, int pl, int act,
                                  hipStream_t stream, int form) {
  typedef _Float16 H;
  return conv<H>(reinterpret_cast<const H*>(x), reinterpret_cast<const H*>(w), reinterpret_cast<const H*>(bias),
                 reinterpret_cast<H*>(y), n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream, form);
}

}  // namespace tfx
