// conv2d on 16-bit float storage as an implicit GEMM on the matrix cores (Section 4.1: 16-bit floating point
// textures; the NHWC index order of the conv2d sampler), for any filter size, stride, padding and channel counts:
//   y[M, Co] = half( act( A[M, K] * filter[K, Co] + bias ) ),  M = n * oh * ow,  K = fh * fw * Ci,
// where row m of A is the 3-D window of output pixel m, never materialised: 8 consecutive k are 8 consecutive
// channels of one input pixel under one filter tap, i.e. one 16-byte load, or zeros where the
// tap falls outside the image.  The channels of a tap are padded to a multiple of 8 for that, and the padding is masked.
// Products are accumulated in fp32 (v_mfma_f32_32x32x16_f16), the result is rounded once.
//
// The loop is the software pipeline of gemm_f16_pipe_kernel: k-slices of 64 halfs are double-buffered in LDS as
// K-contiguous rows of 144 bytes; while slice kt is multiplied, one 16-byte slot after another of slice kt + 1 (fetched
// SETS iterations earlier) moves from registers to the other LDS buffer and is refilled from slice kt + 1 + SETS, spread between
// the MFMAs.  The filter is stored [K, Co] and keeps its k-rows in LDS; its fragments are read with the transposing LDS load (as turned
// in registers, 4 k-rows x 8 columns a thread, its 8-byte LDS writes were waited for: 4 % less over 63 aligned convolutions with the
// tiles as they were).  Tiles of 64 x 128 and 128 x 128 have 8 wavefronts, 64 x 64 and 128 x 32 ones 4: 10 % less over 334 convolutions (3x3,
// 18x19x19x240 -> 152 29.1 -> 20.1 us; 47x17x42x166 -> 32 34.3 -> 24.9).
//
// What bounds it is the latency of a slice where workgroups are few, and the vector-ALU instructions of the addresses
// beside the MFMAs where they are many, hence three forms of the loader:
//   kLean     Ci % 64 == 0: a slice lies inside one tap, the same for every thread, so tap and channel are scalars;
//   kAligned  Ci % 8 == 0 and Co % 8 == 0: a position per thread; taps outside the image and k past the end are fetched from
//             past the end of a buffer descriptor and arrive as zeros, so nothing is masked;
//   kRagged   anything else: loads at any address, masked when they are consumed (ragged.h).
#include "kernel_cost.h"
#include "ragged.h"

#include <type_traits>

namespace tfx {
namespace {

typedef _Float16 half_t;
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef ragged_u32x4 u32x4;

constexpr int kBK = 64;       // halfs per k-slice
constexpr int kLd = kBK + 8;  // LDS row stride in halfs
constexpr int kPad = 16;      // halfs after a k-row of the filter: the four rows of a transposing load lie on different banks
constexpr int kXcds = 8;

enum Form { kLean, kAligned, kRagged };

struct ConvArgs {
  const half_t *x, *w, *bias;
  half_t* y;
  int M, N, Ci, slices;
  unsigned x_total, w_total;  // elements
  int tiles_n, total_blocks, act;
  int H, W, fw, taps, sh, sw, pt, pl;
  FastDiv by_cp, by_fw, by_ow, by_oh;  // cp: channels per tap, padded
};

// A k position: filter tap, channel, and how many channels of the tap are left from there (<= 0: past the end of K).
struct KPos {
  int tap, kh, kw, c, valid;
};
__device__ __forceinline__ KPos k_position(const ConvArgs& g, int kk) {
  KPos p;
  p.tap = (int)div_by((unsigned)kk, g.by_cp);
  p.c = kk - p.tap * (int)g.by_cp.d;
  p.kh = (int)div_by((unsigned)p.tap, g.by_fw);
  p.kw = p.tap - p.kh * g.fw;
  p.valid = p.tap < g.taps ? g.Ci - p.c : 0;
  return p;
}

// WAVES_M x WAVES_N wavefronts, each TM x TN blocks of 32 x 32.
template <int WAVES_M, int WAVES_N, int TM, int TN, Form FORM, int SETS>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void conv_f16_gemm_kernel(ConvArgs g) {
  constexpr int kNT = 64 * WAVES_M * WAVES_N;
  constexpr int WM = 32 * TM, WN = 32 * TN, BM = WM * WAVES_M, BN = WN * WAVES_N;
  constexpr int kLdB = BN + kPad, kTileA = BM * kLd, kTileB = kBK * kLdB;
  constexpr int SA = BM * 8 / kNT, SB = BN * 8 / kNT, SLOTS = SA + SB;  // 16-byte slots per thread and slice
  constexpr int STEPS = kBK / 16, MF = TM * TN;
  static_assert(BM * 8 % kNT == 0 && BN * 8 % kNT == 0, "loader shape");
  extern __shared__ __align__(16) half_t smem_h[];
  half_t* const lds_a = smem_h;  // two A buffers, then two B buffers
  half_t* const lds_b = smem_h + 2 * kTileA;

  // hardware block id b lands on XCD b % 8: give each XCD (own L2) a contiguous range of tiles; the column
  // tiles of one row tile are neighbours, so the window rows they share are fetched once per XCD
  const int bid = blockIdx.x;
  const int q8 = g.total_blocks / kXcds, rem = g.total_blocks % kXcds;
  const int xcd = bid % kXcds;
  const int vid = xcd * q8 + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int m0 = vid / g.tiles_n * BM, n0 = vid % g.tiles_n * BN;
  const int M = g.M, N = g.N, Ci = g.Ci;

  const int tid = threadIdx.x;
  const int wave = tid / 64, lane = tid % 64;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  const int li = lane % 32, hh = lane / 32;

  // A slot i: tile row srow + kRowStep i, halfs scol ... scol + 7 of the slice.  origin: element offset of (window origin,
  // channel 0), outside the tensor where the tap (0, 0) is outside the image.  kLean: with scol in it, one validity bit per tap.
  const int srow = tid / 8, scol = 8 * (tid % 8);
  constexpr int kRowStep = kNT / 8;
  int origin[SA], ih0[SA], iw0[SA];
  unsigned tap_ok[SA];
#pragma unroll
  for (int i = 0; i < SA; ++i) {
    const unsigned r = (unsigned)min(m0 + srow + kRowStep * i, M - 1);  // rows past M repeat the last one (never stored)
    const unsigned r2 = div_by(r, g.by_ow), n = div_by(r2, g.by_oh);
    ih0[i] = (int)(r2 - n * g.by_oh.d) * g.sh - g.pt;
    iw0[i] = (int)(r - r2 * g.by_ow.d) * g.sw - g.pl;
    origin[i] = (((int)n * g.H + ih0[i]) * g.W + iw0[i]) * Ci + (FORM == kLean ? scol : 0);
    if constexpr (FORM == kLean) {
      unsigned ok = 0, bit = 1u;
      for (int ky = 0; ky * g.fw < g.taps; ++ky)
        for (int kx = 0; kx < g.fw; ++kx, bit <<= 1)
          ok |= ((unsigned)(ih0[i] + ky) < (unsigned)g.H && (unsigned)(iw0[i] + kx) < (unsigned)g.W) ? bit : 0u;
      tap_ok[i] = ok;
    }
  }
  // B slot i: k-row brow + kRowsB i of the slice, columns n0 + bcol8 ... + 7; past N: any column block (feeds no stored output)
  constexpr int kRowsB = kNT / (BN / 8);
  const int brow = tid / (BN / 8), bcol8 = 8 * (tid % (BN / 8));
  const unsigned bcol = n0 + bcol8 < N ? (unsigned)(n0 + bcol8) : 0u;
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(g.x), 0, (int)(2u * g.x_total), 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(g.w), 0, (int)(2u * g.w_total), 0x00020000);
  constexpr unsigned kOutside = 0xfffffff0u;

  // What slot loads and stores of one slice need to know: the positions of the slice's A slots and B rows.
  struct Slice {
    KPos a, b[SB];
    int k0;
  };
  auto slice_at = [&](int kt) {
    Slice s;
    s.k0 = min(kt, g.slices - 1) * kBK;  // the last iterations fetch the last slice again (unused)
    s.a = k_position(g, FORM == kLean ? s.k0 : s.k0 + scol);
    if constexpr (FORM == kRagged) {
#pragma unroll
      for (int i = 0; i < SB; ++i) s.b[i] = k_position(g, s.k0 + brow + kRowsB * i);
    }
    return s;
  };
  // Element offset of slot w of a slice in x / the filter.  kRagged: slots that would reach past the end of a tensor
  // start early enough to end with it; *early: by how many elements (nonzero only there).
  auto slot_offset = [&](int w, const Slice& s, unsigned* early, bool* in) {
    unsigned off;
    if (w < SA) {
      if constexpr (FORM == kLean) *in = ((tap_ok[w] >> s.a.tap) & 1u) != 0;
      else *in = s.a.valid > 0 && (unsigned)(ih0[w] + s.a.kh) < (unsigned)g.H && (unsigned)(iw0[w] + s.a.kw) < (unsigned)g.W;
      off = (unsigned)(origin[w] + (s.a.kh * g.W + s.a.kw) * Ci + s.a.c);
    } else if constexpr (FORM == kRagged) {
      const KPos& b = s.b[w < SA ? 0 : w - SA];
      *in = b.valid > 0;
      off = (unsigned)(b.tap * Ci + b.c) * (unsigned)N + bcol;
    } else {
      *in = true;
      off = (unsigned)(s.k0 + brow + kRowsB * (w - SA)) * (unsigned)N + bcol;  // rows past K are past the end of the filter
    }
    *early = 0;
    if constexpr (FORM == kRagged) {
      off = *in ? off : 0u;
      const unsigned at = min(off, (w < SA ? g.x_total : g.w_total) - 8u);
      *early = off - at;
      off = at;
    }
    return off;
  };

  u32x4 reg[SETS][SLOTS];  // slices on their way
  bool inside[SETS][SLOTS];  // kRagged: whether the slot in the registers is one (else zeros)
  // returns nonzero in a lane whose slot was fetched early
  auto load_slot = [&](int set, int w, const Slice& s) __attribute__((always_inline)) {
    unsigned early;
    const unsigned off = slot_offset(w, s, &early, &inside[set][w]);
    // (a buffer load that is not 16-byte aligned is slower than a global one: 3x3, 60x60x100 -> 100 at batch 20 77 against 57 us)
    if constexpr (FORM == kRagged) reg[set][w] = load16((w < SA ? g.x : g.w) + off);
    else reg[set][w] = __builtin_amdgcn_raw_buffer_load_b128(w < SA ? xr : wr, inside[set][w] ? (int)(2u * off) : (int)kOutside, 0, 0);
    return early;
  };
  // once per slice, almost never taken (the last rows of a tensor): shifts what was fetched early down
  auto settle = [&](int set, const Slice& s, unsigned any_early) __attribute__((always_inline)) {
    if (FORM != kRagged || __builtin_amdgcn_ballot_w64(any_early != 0) == 0) return;
#pragma unroll
    for (int w = 0; w < SLOTS; ++w) {
      unsigned early;
      bool in;
      slot_offset(w, s, &early, &in);
      reg[set][w] = shift_down<half_t>(reg[set][w], early);
    }
  };
  auto masked = [&](int set, int w, const u32x4& mask) __attribute__((always_inline)) {
    if constexpr (FORM != kRagged) return reg[set][w];
    const u32x4 zero = {0u, 0u, 0u, 0u};
    return inside[set][w] ? (w < SA ? reg[set][w] & mask : reg[set][w]) : zero;
  };
  auto store_slot = [&](int set, int w, int buf, const u32x4& mask) __attribute__((always_inline)) {
    if (w < SA) {
      *reinterpret_cast<u32x4*>(lds_a + buf * kTileA + (srow + kRowStep * w) * kLd + scol) = masked(set, w, mask);
    } else {
      *reinterpret_cast<u32x4*>(lds_b + buf * kTileB + (brow + kRowsB * (w - SA)) * kLdB + bcol8) = masked(set, w, mask);
    }
  };
  // Fragment of 32 columns x 16 k: lane (li, hh) gets 8 consecutive k from 8 hh on of column li.  The transposing load gives lane i
  // of 16 the four halfs at place i % 4 of the 8-byte pieces that lanes i / 4, i / 4 + 4, ... of the 16 point to: with piece l at
  // k-row l / 4 and columns 4 (l % 4), four k of column i.
  auto filter = [&](const half_t* first, int j, int step) {
    typedef short s4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s4 lds_s4;
    const half_t* const p = first + 32 * j + 16 * step * kLdB;
    const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p)), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p + 4 * kLdB));
    return __builtin_bit_cast(h8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // valid halfs of the A slots in the registers (kRagged)
  int valid[SETS];
  auto fetch = [&](int set, int kt) __attribute__((always_inline)) {
    const Slice at = slice_at(kt);
    unsigned early = 0;
#pragma unroll
    for (int w = 0; w < SLOTS; ++w) early |= load_slot(set, w, at);
    settle(set, at, early);
    valid[set] = at.a.valid;
  };
  // slice 0 goes to LDS, slices 1 ... SETS stay in registers: slice i in set i % SETS
#pragma unroll
  for (int i = 0; i < SETS; ++i) fetch(i, i);
  {
    const u32x4 mask = first_elements<half_t>(valid[0]);
    const Slice at = slice_at(SETS);
    unsigned early = 0;
#pragma unroll
    for (int w = 0; w < SLOTS; ++w) {
      store_slot(0, w, 0, mask);
      early |= load_slot(0, w, at);
    }
    settle(0, at, early);
    valid[0] = at.a.valid;
  }
  __syncthreads();

  auto k_slice = [&](int kt, auto which) __attribute__((always_inline)) {
    constexpr int set = decltype(which)::value;  // of slice kt + 1
    const int cur = kt & 1;
    const Slice after = slice_at(kt + 1 + SETS);
    const u32x4 mask = first_elements<half_t>(valid[set]);
    unsigned early = 0;
    const half_t* la = lds_a + cur * kTileA + (wm0 + li) * kLd + 8 * hh;
    const half_t* lb = lds_b + cur * kTileB + (8 * hh + lane % 16 / 4) * kLdB + wn0 + 16 * (lane / 16 % 2) + 4 * (lane % 4);
    h8 fa[2][TM], fb[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[0][i] = *reinterpret_cast<const h8*>(la + 32 * i * kLd);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = filter(lb, j, 0);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + 1 < STEPS) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[(s + 1) & 1][i] = *reinterpret_cast<const h8*>(la + 32 * i * kLd + 16 * (s + 1));
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[(s + 1) & 1][j] = filter(lb, j, s + 1);
      }
      __builtin_amdgcn_sched_barrier(0);  // keep those LDS reads ahead of this step's MFMAs
      // operands swapped (the filter's fragment first): a lane's registers then hold 4 consecutive output
      // columns of one row
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[s & 1][j], fa[s & 1][i], acc[i][j], 0, 0, 0);
          constexpr int ALL = STEPS * MF;
          const int p = s * MF + i * TN + j;
#pragma unroll
          for (int w = p * SLOTS / ALL; w < (p + 1) * SLOTS / ALL; ++w) {
            store_slot(set, w, cur ^ 1, mask);
            early |= load_slot(set, w, after);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    settle(set, after, early);
    valid[set] = after.a.valid;
    __syncthreads();
  };
  int kt = 0;  // (pairs without a branch between them, across which the compiler would not count loads)
  if constexpr (SETS == 2)
    for (; kt + 1 < g.slices; kt += 2) {
      k_slice(kt, std::integral_constant<int, 1>{});
      k_slice(kt + 1, std::integral_constant<int, 0>{});
    }
  for (; kt < g.slices; ++kt) k_slice(kt, std::integral_constant<int, SETS - 1>{});

  // acc[i][j][v] is the output at row m0 + wm0 + 32 i + li, column n0 + wn0 + 32 j + 8 (v / 4) + 4 hh + v % 4.  Every
  // wavefront converts its block to binary16 in a private LDS region (the slice buffers are free after the loop's last
  // barrier), reads it back row-wise and stores 16 bytes per lane, 128 bytes of a row at a time, at whatever address.
  const ActClamp clamp = make_act(g.act);
  constexpr int kLs = WN + 8;
  static_assert(WAVES_M * WAVES_N * WM * kLs <= 2 * (kTileA + kTileB), "staging fits in the slice buffers");
  half_t* stage = smem_h + wave * WM * kLs;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int cl = 32 * j + 8 * q + 4 * hh, col = n0 + wn0 + cl;
      float bv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) bv[e] = (g.bias != nullptr && col + e < N) ? (float)g.bias[col + e] : 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        h4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = (half_t)apply_act(acc[i][j][4 * q + e] + bv[e], clamp);
        *reinterpret_cast<h4*>(stage + (32 * i + li) * kLs + cl) = pk;
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  constexpr int kLanesPerRow = WN / 8, kRowsPerStep = 64 / kLanesPerRow;
  static_assert(WM % kRowsPerStep == 0, "store steps cover the block");
  const int rr = lane / kLanesPerRow, cc = 8 * (lane % kLanesPerRow);
  const int col = n0 + wn0 + cc;
#pragma unroll
  for (int r0 = 0; r0 < WM; r0 += kRowsPerStep) {
    const int row = m0 + wm0 + r0 + rr;
    const h8 v = *reinterpret_cast<const h8*>(stage + (r0 + rr) * kLs + cc);
    if (row >= M || col >= N) continue;
    half_t* const yp = g.y + (size_t)row * N + col;
    if (col + 8 <= N) {
      *reinterpret_cast<ragged_u32x4_any*>(yp) = __builtin_bit_cast(u32x4, v);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (col + e < N) yp[e] = v[e];
    }
  }
}

template <int WAVES_M, int WAVES_N, int TM, int TN, Form FORM, int SETS>
int launch_sets(ConvArgs& g, hipStream_t stream) {
  constexpr int BM = 32 * TM * WAVES_M, BN = 32 * TN * WAVES_N;
  constexpr size_t lds_bytes = 2 * (size_t)(BM * kLd + kBK * (BN + kPad)) * sizeof(half_t);
  const long long tiles_m = (g.M + (long long)BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  if (tiles_m * tiles_n > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  auto kern = conv_f16_gemm_kernel<WAVES_M, WAVES_N, TM, TN, FORM, SETS>;
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds_bytes, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  g.tiles_n = (int)tiles_n, g.total_blocks = (int)(tiles_m * tiles_n);
  hipLaunchKernelGGL(kern, dim3((unsigned)g.total_blocks), dim3(64 * WAVES_M * WAVES_N), lds_bytes, stream, g);
  return check_launch();
}
template <int WAVES_M, int WAVES_N, int TM, int TN, Form FORM>
int launch(ConvArgs& g, hipStream_t stream) {
  constexpr int BM = 32 * TM * WAVES_M, BN = 32 * TN * WAVES_N;
  const long long tiles = ((g.M + (long long)BM - 1) / BM) * ((g.N + BN - 1) / BN);
  // Two slices on their way in registers where a CU has one workgroup, whose loads nothing else covers, and the contraction is
  // long: 3x3, 8x14x14x512 -> 512 27.7 -> 21.1 us, 28x28x512 -> 512 27.7 -> 20.6, 2x64x64x256 -> 96 14.8 -> 13.4, 6x24x24x129 -> 257
  // 17.9 -> 17.6; none of 19 from 12 slices on slower.
  if (tiles <= 256 && g.slices >= 12) return launch_sets<WAVES_M, WAVES_N, TM, TN, FORM, 2>(g, stream);
  return launch_sets<WAVES_M, WAVES_N, TM, TN, FORM, 1>(g, stream);
}

}  // namespace

bool conv2d_gemm_f16_supported(long long x_elems, int fh, int fw, int ci, int co) {
  const long long k = (long long)fh * fw * ci;
  return x_elems >= 8 && k * co >= 8 && k * co < (1LL << 31) && (long long)fh * fw * (ci + 7) < (1LL << 24);
}

int launch_conv2d_gemm_f16(const uint16_t* x, const uint16_t* w, const uint16_t* bias, uint16_t* y, int n, int h, int wd,
                           int ci, int fh, int fw, int co, int oh, int ow, int sh, int sw, int pt, int pl, int act,
                           hipStream_t stream) {
  ConvArgs g{};
  const int cp = (ci + 7) / 8 * 8;
  g.x = reinterpret_cast<const half_t*>(x), g.w = reinterpret_cast<const half_t*>(w);
  g.bias = reinterpret_cast<const half_t*>(bias), g.y = reinterpret_cast<half_t*>(y);
  g.M = n * oh * ow, g.N = co, g.Ci = ci, g.act = act;
  g.slices = (fh * fw * cp + kBK - 1) / kBK;
  g.x_total = (unsigned)((long long)n * h * wd * ci), g.w_total = (unsigned)((long long)fh * fw * ci * co);
  g.H = h, g.W = wd, g.fw = fw, g.taps = fh * fw, g.sh = sh, g.sw = sw, g.pt = pt, g.pl = pl;
  g.by_cp = fast_div((unsigned)cp), g.by_fw = fast_div((unsigned)fw), g.by_ow = fast_div((unsigned)ow), g.by_oh = fast_div((unsigned)oh);
  // (the byte offset of a filter row past K stays below 2^32)
  const bool aligned = ci % 8 == 0 && co % 8 == 0 && ((long long)fh * fw * ci + kBK) * co < (1LL << 31) && reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(w) % 16 == 0;
  if (fh == 1 && fw == 1 && sh == sw && pt == 0 && pl == 0 && thin_pays(g.M, co, ci, true))
    return launch_conv1x1_thin_f16(x, w, y, bias, g.M, co, ci, act, stream, h, wd, oh, ow, sh);
  // The least modelled time, fitted to 334 convolutions (1x1, 3x3, 5x5, 7 ... 112 pixels a side, 8 ... 512 channels, batch 1 ... 64;
  // near the choice the rms error is 9 - 14 %): LDS tiles of three sizes, or the contraction split over a workgroup's wavefronts
  // with 16 x 32, 32 x 64 or 64 x 64 tiles.  Over these the choice costs 0.9 % on average against the fastest of each, more than 16 %
  // for three (3x3, 36x13x13x160 -> 52: 17.4 us, 12.7 with 64 x 64 split).
  // (5x5, 13x20x20x398 -> 192: 137 us with LDS tiles, 92 split; 3x3, 2x56x56x32 -> 64: 10.8 and 6.4.)
  const int kp = fh * fw * cp, k64 = g.slices * kBK;
  enum { kDeep, kDirect64x64, kDirect32x64, k128x32, k64x64, k64x128, k128x128, kForms };
  const int deep_n = deep_two_columns((g.M + 15) / 16, co, (kp + 31) / 32) ? 32 : 16, odd = aligned ? 0 : 1;
  // Up to 32 columns: tiles of 128 x 32 multiply half as much padding and read a row of A for them once, 20 KB a slice for 128 rows
  // where tiles of 64 x 64 read 32.  Not where more than two of them a CU read windows of 256 channels and more, which leave L2
  // between two taps: 3x3, 30x56x56x256 -> 16 54.5 us, 51.1 without them; 23x78x78x328 -> 16 112 and 107, -> 27 124 and 139.
  // Nor with less than one and a half a CU: a lone workgroup of 4 wavefronts waits for its loads (15x38x38x18 -> 15 8.6 us, 5.9
  // without, 16x48x48x11 -> 20 9.5 and 8.0).
  // us before and with them: 28x103x103x54 -> 16 55 -> 38, 40x51x51x140 -> 16 49 -> 29, 10x87x87x96 -> 22 (5x5) 66 -> 45; of 450
  // drawn with up to 64 columns a seventh are more than 8 % faster, none more than 5 % slower (6 %: the margin at which that holds).
  const bool narrow = co <= 32 && g.M > 384 * 128 && (ci < 256 || g.M <= 512 * 128);
  const double us[kForms] = {1.05 * PipeCost{16, deep_n, 3.42, .019, .0021, .89, 1.31, .05, 1.45}.us(1, g.M, co, kp, odd),
                             co >= 2 ? PipeCost{64, 64, .79, 3.94, .0064, .65, .87, .30, .86}.us(1, g.M, co, kp, odd) : 1e30,
                             co >= 2 ? PipeCost{32, 64, 1.51, 2.78, .0074, .24, .37, .31, .015, .0014}.us(1, g.M, co, kp, odd) : 1e30,
                             narrow ? 1.06 * PipeCost{128, 32, 2.47, 2.34, .0061, .2, .55, .7, 0.}.us(1, g.M, co, k64, odd) : 1e30,
                             PipeCost{64, 64, 4.04, .74, .0054, .34, .50, .77, .69}.us(1, g.M, co, k64, odd),
                             PipeCost{64, 128, 3.19, 1.55, .0065, .57, .69, .72, .67}.us(1, g.M, co, k64, odd),
                             PipeCost{128, 128, 4.52, 1.11, .0082, .72, .99, .50, .52, .0001}.us(1, g.M, co, k64, odd)};
  int form = 0;
  for (int f = 1; f < kForms; ++f)
    if (us[f] < us[form]) form = f;
  if (form == kDeep) return launch_conv2d_deep_f16(x, w, bias, y, n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream);
  if (form == kDirect64x64 || form == kDirect32x64)
    return launch_conv2d_gemm_direct_f16(x, w, bias, y, n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream, form == kDirect32x64);
  auto tiles = [&](auto loader) {
    constexpr Form FORM = decltype(loader)::value;
    if (form == k128x32) return launch<4, 1, 1, 1, FORM>(g, stream);
    if (form == k64x64) return launch<2, 2, 1, 1, FORM>(g, stream);
    if (form == k64x128) return launch<2, 4, 1, 1, FORM>(g, stream);
    return launch<2, 4, 2, 1, FORM>(g, stream);
  };
  if (!aligned) return tiles(std::integral_constant<Form, kRagged>{});
  return ci % 64 == 0 && fh * fw <= 32 ? tiles(std::integral_constant<Form, kLean>{}) : tiles(std::integral_constant<Form, kAligned>{});
}

}  // namespace tfx
