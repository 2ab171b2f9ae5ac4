// fp32 products of few output tiles and fp32 convolutions alike, any layout, size and alignment:
//   C[b] = act( op(A[b]) * op(B[b]) + bias )      (Listing 2, Section 4.1; conv2d: the NHWC index order of Section 4.1)
// on the bf16 matrix cores with three-way split operands (split.h).
//
// For outputs of up to a few 64 x 64 tiles per CU a kernel that walks through K slice by slice is a serial chain: load,
// split, LDS, barrier, multiply, 0.9 us per 32 k.  Here the wavefronts of a workgroup split K instead: wavefront w takes
// k-steps w, w + WAVES, ... of 16, loads its operands of two steps ahead straight into registers, splits them there and
// multiplies the whole 32 TM x 32 TN tile; nothing is shared until the partial tiles are added through LDS at the end.
// Every operand element is split once per workgroup, as it would be on the way into LDS, and without the LDS traffic;
// bound by the split's vector instructions (7 per element) and, close behind, the matrix cores.
#include "ragged.h"
#include "split.h"

namespace tfx {
namespace {

constexpr int kXcds = 8;

enum Source { kRowsK, kRowsM, kConv };  // A stored [M,K]; stored [K,M]; the window view of an NHWC image

struct DirectArgs {
  const float *a, *b, *bias;
  float* c;
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

// 8 consecutive k of one row or column
struct Octet {
  ragged_u32x4 lo, hi;
};

template <Source A_SRC, bool B_KC, int TM, int TN, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES / 4) void gemm_direct_kernel(DirectArgs g) {
  constexpr bool CONV = A_SRC == kConv;
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
  const float* const A = g.a + (size_t)batch * g.strideA;
  const float* const B = g.b + (size_t)batch * g.strideB;
  float* const C = g.c + (size_t)batch * g.strideC;

  // rows and columns past the matrix repeat the last one (they only feed outputs that are not stored)
  int arow[TM], bcol[TN], origin[TM], ih0[TM], iw0[TM];
  unsigned seen[TM];  // filter taps inside the image, one bit each (lean loads only)
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    seen[i] = 0;
    arow[i] = min(m0 + 32 * i + li, g.M - 1);
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
  for (int j = 0; j < TN; ++j) bcol[j] = min(n0 + 32 * j + li, g.N - 1);

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
  auto chunk = [&](const float* base, bool in, unsigned off, unsigned total, unsigned* early) __attribute__((always_inline)) {
    off = in ? off : 0u;
    const unsigned at = min(off, total - 4u);
    *early = off - at;
    return load16(base + at);
  };
  auto a_offset = [&](const Place& p, int i) __attribute__((always_inline)) {
    return CONV ? (unsigned)(origin[i] + (p.kh * g.W + p.kw) * g.K + p.c) : (unsigned)arow[i] * (unsigned)g.K + (unsigned)p.c;
  };
  Octet a[2][TM], b[2][TN];  // raw operands of two steps
  auto gather = [&](const float* base, int row, int ld, int col, int valid) __attribute__((always_inline)) {
    Octet o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = base[(size_t)(row + (e < valid ? e : 0)) * ld + col];
      if (e < 4) o.lo[e] = __float_as_uint(v);
      else o.hi[e - 4] = __float_as_uint(v);
    }
    return o;
  };
  // Lean loads: a uniform address per step (and k, where K is not contiguous) plus a lane's own 32-bit offset, so that
  // no vector instruction goes into addresses.
  auto columns = [&](const float* at, int ld, unsigned offset) __attribute__((always_inline)) {
    Octet o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = at[offset];
      at += ld;
      if (e < 4) o.lo[e] = __float_as_uint(v);
      else o.hi[e - 4] = __float_as_uint(v);
    }
    return o;
  };
  unsigned a_lane[TM], b_lane[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
    a_lane[i] = A_SRC == kRowsM ? 8u * h * (unsigned)g.M + (unsigned)arow[i] : (unsigned)arow[i] * (unsigned)g.K + 8u * h;
#pragma unroll
  for (int j = 0; j < TN; ++j)
    b_lane[j] = B_KC ? (unsigned)bcol[j] * (unsigned)g.K + 8u * h : 8u * h * (unsigned)g.N + (unsigned)bcol[j];
  auto load = [&](int step, Octet (&oa)[TM], Octet (&ob)[TN]) __attribute__((always_inline)) {
    if (step < g.whole_steps) {
      int tap = 0, tap_offset = 0;
      if constexpr (CONV) {
        tap = (int)div_by(16u * (unsigned)step, g.by_cp);
        const int kh = (int)div_by((unsigned)tap, g.by_fw), kw = tap - kh * g.fw;
        tap_offset = (kh * g.W + kw) * g.K + 16 * step - tap * g.K;
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if constexpr (A_SRC == kRowsM) {
          oa[i] = columns(A + (size_t)(16 * step) * g.M, g.M, a_lane[i]);
        } else {
          const float* p = A + 16 * step + a_lane[i];
          if constexpr (CONV) p = A + (ptrdiff_t)(origin[i] + tap_offset + 8 * h);
          const bool in = !CONV || ((seen[i] >> tap) & 1u) != 0;
          oa[i].lo = load16(in ? p : kZeros);
          oa[i].hi = load16(in ? p + 4 : kZeros);
        }
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (B_KC) {
          const float* p = B + 16 * step + b_lane[j];
          ob[j].lo = load16(p);
          ob[j].hi = load16(p + 4);
        } else {
          ob[j] = columns(B + (size_t)(16 * step) * g.N, g.N, b_lane[j]);
        }
      }
      return;
    }
    const Place p = place(step);
    unsigned early;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (A_SRC == kRowsM) {
        oa[i] = gather(A, p.valid > 0 ? p.c : 0, g.M, arow[i], p.valid);
      } else {
        const bool in = CONV ? inside(p, i) : p.valid > 0;
        const unsigned off = a_offset(p, i);
        oa[i].lo = chunk(A, in, off, g.a_total, &early);
        oa[i].hi = chunk(A, in && p.valid > 4, off + 4, g.a_total, &early);
      }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if constexpr (B_KC) {
        const unsigned off = (unsigned)bcol[j] * (unsigned)g.K + (unsigned)p.c;
        ob[j].lo = chunk(B, p.valid > 0, off, g.b_total, &early);
        ob[j].hi = chunk(B, p.valid > 4, off + 4, g.b_total, &early);
      } else {
        ob[j] = gather(B, p.valid > 0 ? p.tap * g.K + p.c : 0, g.N, bcol[j], p.valid);
      }
    }
  };
  // ... and what makes the registers the operands: chunks fetched early shifted, k past the end and pixels outside zeroed
  auto settle = [&](int step, Octet (&oa)[TM], Octet (&ob)[TN]) __attribute__((always_inline)) {
    if (step < g.whole_steps) return;
    const Place p = place(step);
    auto fix = [&](ragged_u32x4& v, bool in, unsigned off, unsigned total, int valid) __attribute__((always_inline)) {
      const unsigned early = in ? off - min(off, total - 4u) : 0u;
      if (__builtin_amdgcn_ballot_w64(early != 0) != 0) v = shift_down<float>(v, early);
      v &= first_elements<float>(in ? valid : 0);
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (A_SRC == kRowsM) {
        oa[i].lo &= first_elements<float>(p.valid);
        oa[i].hi &= first_elements<float>(p.valid - 4);
      } else {
        const bool in = CONV ? inside(p, i) : p.valid > 0;
        const unsigned off = a_offset(p, i);
        fix(oa[i].lo, in, off, g.a_total, p.valid);
        fix(oa[i].hi, in && p.valid > 4, off + 4, g.a_total, p.valid - 4);
      }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if constexpr (B_KC) {
        const unsigned off = (unsigned)bcol[j] * (unsigned)g.K + (unsigned)p.c;
        fix(ob[j].lo, p.valid > 0, off, g.b_total, p.valid);
        fix(ob[j].hi, p.valid > 4, off + 4, g.b_total, p.valid - 4);
      } else {
        ob[j].lo &= first_elements<float>(p.valid);
        ob[j].hi &= first_elements<float>(p.valid - 4);
      }
    }
  };

  floatx16 acc[TM][TN];
  TinyGuard guard;
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  };
  auto split8 = [&](const Octet& o, bf16x8 (&part)[kParts]) __attribute__((always_inline)) {
    const floatx4 lo = __builtin_bit_cast(floatx4, o.lo), hi = __builtin_bit_cast(floatx4, o.hi);
    guard.see(lo);
    guard.see(hi);
    splitx4 pl[kParts], ph[kParts];
    split4(lo, pl);
    split4(hi, ph);
#pragma unroll
    for (int p = 0; p < kParts; ++p) part[p] = __builtin_bit_cast(bf16x8, ragged_u32x4{pl[p][0], pl[p][1], ph[p][0], ph[p][1]});
  };
  auto multiply = [&](int step, int next, Octet (&oa)[TM], Octet (&ob)[TN]) __attribute__((always_inline)) {
    settle(step, oa, ob);
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
  };

  clear();
  if (wave < g.steps) load(wave, a[0], b[0]);
  if (wave + WAVES < g.steps) load(wave + WAVES, a[1], b[1]);
  // the quads this thread adds up: quad (i, j, v) of lane l is column 32 j + l % 32, rows 32 i + 8 v + 4 (l / 32) .. + 3
  float bias[OWN];
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    const int quad = wave * OWN + o, col = n0 + 32 * (quad / 4 % TN) + li;
    bias[o] = g.bias != nullptr && col < g.N ? g.bias[col] : 0.f;
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
          red[(wave * QUADS + (i * TN + j) * 4 + v) * 64 + lane] =
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
  unsigned most = 0;
#pragma unroll
  for (int o = 0; o < OWN; ++o)
#pragma unroll
    for (int v = 0; v < 4; ++v) see_result(most, sum[o][v]);
  const bool tiny = __syncthreads_or(guard.tiny());
  if (__syncthreads_or(overflowed(most)) || tiny) {
    // values that the split does not carry: once more with the fp32 instructions, for the results that are Inf or NaN or,
    // after an operand of tiny magnitude, for all
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
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(e < 4 ? a[0][i].lo[e & 3] : a[0][i].hi[e & 3]),
                                                             __uint_as_float(e < 4 ? b[0][j].lo[e & 3] : b[0][j].hi[e & 3]), acc[i][j], 0, 0, 0);
    }
    floatx4 exact[OWN];
    add_up(exact);
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (tiny || !__builtin_isfinite(sum[o][v])) sum[o][v] = exact[o][v];
  }
  const ActClamp clamp = make_act(g.act);
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    const int quad = wave * OWN + o, col = n0 + 32 * (quad / 4 % TN) + li;
    const int row0 = m0 + 32 * (quad / 4 / TN) + 8 * (quad % 4) + 4 * h;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (row0 + v < g.M && col < g.N) C[(size_t)(row0 + v) * g.N + col] = apply_act(sum[o][v] + bias[o], clamp);
  }
}

template <Source A_SRC, bool B_KC, int TM, int TN, int WAVES>
int launch(DirectArgs& g, int batch, hipStream_t stream) {
  g.tiles_m = (g.M + 32 * TM - 1) / (32 * TM);
  g.tiles_n = (g.N + 32 * TN - 1) / (32 * TN);
  const long long total = (long long)batch * g.tiles_m * g.tiles_n;
  if (total > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  g.total_blocks = (int)total;
  g.m_fastest = g.N > g.M ? 1 : 0;
  hipLaunchKernelGGL((gemm_direct_kernel<A_SRC, B_KC, TM, TN, WAVES>), dim3((unsigned)total), dim3(64 * WAVES), 0, stream, g);
  return check_launch();
}

template <Source A_SRC, bool B_KC>
int launch_tile(DirectArgs& g, int batch, hipStream_t stream, int form) {
  if (form == 0) return launch<A_SRC, B_KC, 2, 2, 8>(g, batch, stream);
  if (form == 1) return launch<A_SRC, B_KC, 1, 2, 4>(g, batch, stream);
  return launch<A_SRC, B_KC, 1, 1, 4>(g, batch, stream);
}

}  // namespace

int launch_gemm_direct(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, bool a_kc,
                       bool b_kc, int act, hipStream_t stream, int form) {
  DirectArgs g{};
  g.a = a, g.b = b, g.bias = bias, g.c = c;
  g.M = m, g.N = n, g.K = k, g.act = act;
  g.strideA = (long long)m * k, g.strideB = (long long)n * k, g.strideC = (long long)m * n;
  g.a_total = (unsigned)g.strideA, g.b_total = (unsigned)g.strideB;
  g.steps = (k + 15) / 16;
  // (a lane's byte offset has 32 bits)
  const bool lean = (a_kc ? (long long)m * k : 9LL * m) < (1LL << 30) && (b_kc ? (long long)n * k : 9LL * n) < (1LL << 30);
  g.whole_steps = lean ? k / 16 : 0;
  if (a_kc) return b_kc ? launch_tile<kRowsK, true>(g, batch, stream, form) : launch_tile<kRowsK, false>(g, batch, stream, form);
  return b_kc ? launch_tile<kRowsM, true>(g, batch, stream, form) : launch_tile<kRowsM, false>(g, batch, stream, form);
}

int launch_conv2d_gemm_direct(const float* x, const float* w, const float* bias, float* y, int n, int h, int wd, int ci, int fh,
                              int fw, int co, int oh, int ow, int sh, int sw, int pt, int pl, int act, hipStream_t stream, int form) {
  DirectArgs g{};
  const int cp = (ci + 7) / 8 * 8;
  g.a = x, g.b = w, g.bias = bias, g.c = y;
  g.M = n * oh * ow, g.N = co, g.K = ci, g.act = act;
  g.a_total = (unsigned)((long long)n * h * wd * ci), g.b_total = (unsigned)((long long)fh * fw * ci * co);
  g.steps = (fh * fw * cp + 15) / 16;
  g.whole_steps = ci % 16 == 0 && fh * fw <= 32 && 9LL * co < (1LL << 30) ? g.steps : 0;  // a step inside one tap
  g.H = h, g.W = wd, g.fw = fw, g.taps = fh * fw, g.sh = sh, g.sw = sw, g.pt = pt, g.pl = pl;
  g.by_cp = fast_div((unsigned)cp), g.by_fw = fast_div((unsigned)fw), g.by_ow = fast_div((unsigned)ow), g.by_oh = fast_div((unsigned)oh);
  return launch_tile<kConv, false>(g, 1, stream, form);
}

}  // namespace tfx
