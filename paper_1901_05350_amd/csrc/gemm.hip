// fp32 MFMA GEMM for gfx950: C[b] = act(op(A[b]) * op(B[b]) + bias).
//
// This one kernel family serves matMul / batchMatMul (Section 4.1, Listing 2 of the
// TensorFlow.js paper defines the op: one dot product per output value) and the 1x1
// "pointwise" conv2d, which is the same contraction with M = N*H*W, K = inC, N = outC.
// The paper's shader computes one output per fragment with no data sharing; here a
// workgroup computes a tile, stages A and B k-slices through LDS and feeds the matrix cores
// (64-wide wavefronts): v_mfma_f32_32x32x16_bf16 on three-way split operands (split.h) in the tiled kernel for
// medium and large problems, v_mfma_f32_16x16x4_f32 in the 16-row kernel for small M x N.
//
// Layout of one MFMA 32x32x16 (wave64), used below:
//   A operand: lane l holds A[i = l % 32][k = 8*(l/32) .. + 7]
//   B operand: lane l holds B[k = 8*(l/32) .. + 7][j = l % 32]
//   D result : register v of lane l holds D[i = 8*(v/4) + 4*(l/32) + v%4][j = l % 32]
#include "kernel_cost.h"
#include "ragged.h"
#include "split.h"

#include <cmath>
#include <type_traits>

namespace tfx {

namespace {

constexpr int kXcds = 8;  // workgroups are dealt round-robin to the 8 XCDs, each with its own L2

// Branch-free loads for k-slices that lie entirely inside K.  A thread's slots keep a
// pointer each, set up once: rows past the end of the operand are clamped to a valid row instead of masked --
// they only feed output rows / columns that are never stored -- so a k-slice is NSLOT unconditional loads and
// no other vector instruction (on this chip every vector-ALU instruction takes issue time away from the
// matrix cores: the masked loader's compares, zero fills and branches cost ~10% of the main loop).  The loads need no
// alignment; a slot of a row-contiguous operand may reach past the end of its row into the next one, so the slice with
// the last row is not one of these when the row length is no multiple of 4.
//
// Slots of the tiled kernel: s = tid + it * NT;
//   KC : row s / (BK/4), k = 4 * (s % (BK/4)) .. + 3
//   !KC: a thread's four slots are four consecutive k of the same four rows (block b = tid: rows 4 * (b % (ROWS/4)),
//        k = 4 * (b / (ROWS/4)) + it), so that it can hand each row's four k on together
template <int ROWS, int BK, bool KC, int NT, int NSLOT>
__device__ __forceinline__ int slot_row(int tid, int it) {
  static_assert(KC || (NSLOT == 4 && ROWS * BK == 16 * NT), "one 4 x 4 block per thread");
  return KC ? (tid + it * NT) / (BK / 4) : 4 * (tid % (ROWS / 4));
}
template <int ROWS, int BK, bool KC, int NT>
__device__ __forceinline__ int slot_k(int tid, int it) {
  return KC ? 4 * ((tid + it * NT) % (BK / 4)) : 4 * (tid / (ROWS / 4)) + it;
}
template <int ROWS, int BK, bool KC, int NT, int NSLOT>
__device__ __forceinline__ void slot_pointers(const float* __restrict__ g, int ld, int rows_total, int row0, int tid,
                                              const float* (&ptr)[NSLOT]) {
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    int gr = row0 + slot_row<ROWS, BK, KC, NT, NSLOT>(tid, it);
    const int k = slot_k<ROWS, BK, KC, NT>(tid, it);
    if (KC) {
      gr = min(gr, rows_total - 1);
      ptr[it] = g + (size_t)gr * ld + k;
    } else {
      if (gr >= rows_total) gr = 0;
      ptr[it] = g + (size_t)k * ld + gr;
    }
  }
}
__device__ __forceinline__ float4 load_quad(const float* p) { return __builtin_bit_cast(float4, load16(p)); }
template <int NSLOT>
__device__ __forceinline__ void load_tile_full(const float* (&ptr)[NSLOT], size_t k_offset, float4 (&reg)[NSLOT]) {
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) reg[it] = load_quad(ptr[it] + k_offset);
}

// The same for any k-slice and operand of at least 4 elements: the loads of a slice (every one unconditional, from a
// valid place) and, when its registers are consumed, what makes them the slice: quads that would have left the operand
// were fetched a few elements early and are shifted down, elements past K are zeroed.
// CV: the operand is a convolution's filter [taps * Ci, N] seen with the channels of a tap padded to a multiple of 4
// (`by_cp.d`), k_total channels per tap.
struct FilterK {
  FastDiv by_cp;
  int taps;
};
template <int ROWS, int BK, bool KC, bool CV, int NT, int NSLOT>
__device__ __forceinline__ unsigned slot_offset(int ld, int rows_total, int k_total, int row0, int k0, int tid, int it,
                                                unsigned total, const FilterK& fk, unsigned* early, int* valid) {
  int gr = row0 + slot_row<ROWS, BK, KC, NT, NSLOT>(tid, it), gk = k0 + slot_k<ROWS, BK, KC, NT>(tid, it);
  unsigned off;
  if (KC) {
    gr = min(gr, rows_total - 1);
    *valid = k_total - gk;
    off = (unsigned)gr * (unsigned)ld + (unsigned)(*valid > 0 ? gk : 0);
  } else {
    if (gr >= rows_total) gr = 0;
    bool in;
    if constexpr (CV) {
      const int tap = (int)div_by((unsigned)gk, fk.by_cp), c = gk - tap * (int)fk.by_cp.d;
      in = tap < fk.taps && c < k_total;
      gk = tap * k_total + c;
    } else {
      in = gk < k_total;
    }
    *valid = in ? 4 : 0;
    off = (unsigned)(in ? gk : 0) * (unsigned)ld + (unsigned)gr;
  }
  const unsigned at = min(off, total - 4u);
  *early = off - at;
  return at;
}
template <int ROWS, int BK, bool KC, bool CV, int NT, int NSLOT>
__device__ __forceinline__ void load_tile_any(const float* __restrict__ g, int ld, int rows_total, int k_total, int row0, int k0,
                                              int tid, unsigned total, const FilterK& fk, float4 (&reg)[NSLOT]) {
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    unsigned early;
    int valid;
    reg[it] = load_quad(g + slot_offset<ROWS, BK, KC, CV, NT, NSLOT>(ld, rows_total, k_total, row0, k0, tid, it, total, fk, &early, &valid));
  }
}
template <int ROWS, int BK, bool KC, bool CV, int NT, int NSLOT>
__device__ __forceinline__ void settle_tile(int ld, int rows_total, int k_total, int row0, int k0, int tid, unsigned total,
                                            const FilterK& fk, float4 (&reg)[NSLOT]) {
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    unsigned early;
    int valid;
    slot_offset<ROWS, BK, KC, CV, NT, NSLOT>(ld, rows_total, k_total, row0, k0, tid, it, total, fk, &early, &valid);
    ragged_u32x4 v = __builtin_bit_cast(ragged_u32x4, reg[it]);
    if (__builtin_amdgcn_ballot_w64(early != 0) != 0) v = shift_down<float>(v, early);
    reg[it] = __builtin_bit_cast(float4, v & first_elements<float>(valid));
  }
}

// Implicit-GEMM view of a convolution input (NHWC): GEMM row = output pixel (n, oh, ow), GEMM
// column k = (kh, kw, c) with c fastest, so A[row][k] = x[n, oh*sh - pt + kh, ow*sw - pl + kw, c]
// (zero outside the image) and B = the HWIO filter seen as [fh*fw*Ci, Co].
struct ConvA {
  const float* x;
  int H, W, Ci, OH, OW, fw, sh, sw, pt, pl;
  unsigned total;  // elements of x
  FastDiv by_fw, by_ow, by_oh;
  FilterK fk;      // channels of a tap padded to a multiple of 4
};

// A-tile loader of the implicit GEMM for any channel count.  k runs over (tap, channel) with the channels of a tap
// padded to a multiple of 4, so a quad never crosses a filter tap; all slots of a thread share the same k offset (NT is
// a multiple of BK/4), which is decoded once per thread and slice (two multiplications by reciprocals).  Every load is
// unconditional: for a quad outside the image or past K from the first element of x, zeroed when the registers are
// consumed; one that would leave x is fetched early and shifted (load_tile_any).
struct ConvRow {  // what a thread knows about the output pixel of one of its slots
  int ih0, iw0;   // input coordinates of filter tap (0, 0)
  int origin;     // element offset of that tap's channel 0 (negative or past x where the tap is outside the image)
};
template <int BM, int BK, int NT, int NSLOT>
__device__ __forceinline__ void conv_rows(const ConvA& cv, int M, int m0, int tid, ConvRow (&rows)[NSLOT]) {
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    const unsigned r = (unsigned)min(m0 + (tid + it * NT) / (BK / 4), M - 1);  // rows past M repeat the last one
    const unsigned t = div_by(r, cv.by_ow), n = div_by(t, cv.by_oh);
    rows[it].ih0 = (int)(t - n * cv.by_oh.d) * cv.sh - cv.pt;
    rows[it].iw0 = (int)(r - t * cv.by_ow.d) * cv.sw - cv.pl;
    rows[it].origin = (((int)n * cv.H + rows[it].ih0) * cv.W + rows[it].iw0) * cv.Ci;
  }
}
struct ConvK {  // a thread's k position in a slice
  int kh, kw, add, valid;
};
template <int BK>
__device__ __forceinline__ ConvK conv_k(const ConvA& cv, int k0, int tid) {
  const int gk = k0 + 4 * (tid % (BK / 4));
  const int tap = (int)div_by((unsigned)gk, cv.fk.by_cp), c = gk - tap * (int)cv.fk.by_cp.d;
  ConvK p;
  p.kh = (int)div_by((unsigned)tap, cv.by_fw);
  p.kw = tap - p.kh * cv.fw;
  p.add = (p.kh * cv.W + p.kw) * cv.Ci + c;
  p.valid = tap < cv.fk.taps ? cv.Ci - c : 0;
  return p;
}
__device__ __forceinline__ unsigned conv_offset(const ConvA& cv, const ConvRow& row, const ConvK& p, unsigned* early, bool* in) {
  const int ih = row.ih0 + p.kh, iw = row.iw0 + p.kw;
  *in = p.valid > 0 && ih >= 0 && ih < cv.H && iw >= 0 && iw < cv.W;
  const unsigned off = *in ? (unsigned)(row.origin + p.add) : 0u, at = min(off, cv.total - 4u);
  *early = off - at;
  return at;
}
template <int BK, int NSLOT>
__device__ __forceinline__ void load_tile_conv(const ConvA& cv, int k0, int tid, const ConvRow (&rows)[NSLOT],
                                               float4 (&reg)[NSLOT]) {
  const ConvK p = conv_k<BK>(cv, k0, tid);
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    unsigned early;
    bool in;
    reg[it] = load_quad(cv.x + conv_offset(cv, rows[it], p, &early, &in));
  }
}
// RAGGED: Ci % 4 != 0 (else a quad inside the image is valid as it is)
template <int BK, bool RAGGED, int NSLOT>
__device__ __forceinline__ void settle_tile_conv(const ConvA& cv, int k0, int tid, const ConvRow (&rows)[NSLOT],
                                                 float4 (&reg)[NSLOT]) {
  const ConvK p = conv_k<BK>(cv, k0, tid);
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    unsigned early;
    bool in;
    conv_offset(cv, rows[it], p, &early, &in);
    ragged_u32x4 v = __builtin_bit_cast(ragged_u32x4, reg[it]);
    if constexpr (RAGGED) {
      if (__builtin_amdgcn_ballot_w64(early != 0) != 0) v = shift_down<float>(v, early);
      v &= first_elements<float>(in ? p.valid : 0);
    } else {
      v &= in ? ~0u : 0u;
    }
    reg[it] = __builtin_bit_cast(float4, v);
  }
}

// Lean A-tile loader of the implicit GEMM for Ci % BK == 0 (vector loads, at most 32 filter taps): a k-slice
// then lies inside one filter tap, so the tap (kh, kw) and the channel offset are the same for the whole
// workgroup and live in scalar registers.  A slot keeps, from set-up, the address of its pixel's tap (0, 0) and
// one validity bit per tap; per k-slice it adds the slice's uniform offset and, for a tap outside the image,
// reads a zero quad instead: 5 vector-ALU instructions per slot where the general loader spends ~100 on
// decoding and range checks (which take their issue time from the matrix cores).
__device__ __align__(16) float kZeroQuad[4] = {0.f, 0.f, 0.f, 0.f};  // never written (not const: same address space as x)

template <int BM, int BK, int NT, int NSLOT>
__device__ __forceinline__ void conv_lean_rows(const ConvA& cv, int M, int K, int m0, int tid, const float* (&p0)[NSLOT],
                                               unsigned (&ok)[NSLOT]) {
  const int fh = K / (cv.fw * cv.Ci);
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    const int r = min(m0 + (tid + it * NT) / (BK / 4), M - 1);  // rows past M repeat the last row (never stored)
    const int ow = r % cv.OW;
    const int t = r / cv.OW;
    const int oh = t % cv.OH;
    const int n = t / cv.OH;
    const int ih0 = oh * cv.sh - cv.pt, iw0 = ow * cv.sw - cv.pl;
    // address of tap (0, 0), channel 4 * (tid % (BK/4)); outside the image for border pixels, where only the taps
    // whose bit is set are ever dereferenced
    const long long e = (((long long)n * cv.H + ih0) * cv.W + iw0) * cv.Ci + 4 * (tid % (BK / 4));
    p0[it] = cv.x + e;
    unsigned bits = 0;
    for (int kh = 0; kh < fh; ++kh)
      for (int kw = 0; kw < cv.fw; ++kw)
        if (ih0 + kh >= 0 && ih0 + kh < cv.H && iw0 + kw >= 0 && iw0 + kw < cv.W) bits |= 1u << (kh * cv.fw + kw);
    ok[it] = bits;
  }
}

template <int NSLOT>
__device__ __forceinline__ void load_tile_conv_lean(const float* (&p0)[NSLOT], const unsigned (&ok)[NSLOT], int tap,
                                                    long long slice_offset, float4 (&reg)[NSLOT]) {
  const unsigned bit = 1u << tap;
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    const float* p = (ok[it] & bit) ? p0[it] + slice_offset : kZeroQuad;
    const floatx4 v = *reinterpret_cast<const floatx4*>(p);  // as a vector: a struct copy from a selected pointer stays in memory
    reg[it] = make_float4(v[0], v[1], v[2], v[3]);
  }
}

__device__ __forceinline__ float f4_get(const float4& v, int s) {
  return s == 0 ? v.x : (s == 1 ? v.y : (s == 2 ? v.z : v.w));
}

// LDS tile of one operand of the tiled kernel: three planes (hi, mid, lo) of ROWS rows of 32 k, k contiguous, in
// pieces of 8 k (16 bytes).  Rows of a !KC operand are stored in the order row % 4, row / 4: then the writes of a
// wavefront, one row of every thread's 4 x 4 block at a time, and the fragment reads, 32 consecutive rows, both spread
// over all banks with the piece order rotated as below.
template <int ROWS, bool KC>
struct PlaneTile {
  static constexpr int kPlane = ROWS * 64;  // bytes
  static constexpr int kBytes = kParts * kPlane;
  static __device__ __forceinline__ int at(int row, int piece) {  // byte offset of a piece in its plane
    const int r = KC ? row : (row % 4) * (ROWS / 4) + row / 4;
    const int turn = KC ? (r / 8) & 3 : ((r / 8) ^ row) & 3;
    return r * 64 + ((piece ^ turn) * 16);
  }
};

// Registers -> LDS: splits a thread's slots and writes four k of a row at a time (8 bytes per plane).
template <int ROWS, int BK, bool KC, int NT, int NSLOT>
__device__ __forceinline__ void store_planes(char* __restrict__ lds, int tid, const float4 (&reg)[NSLOT], SplitGuard& guard) {
  using T = PlaneTile<ROWS, KC>;
  static_assert(BK == 32, "rows of 32 k");
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    floatx4 v;
    int row = slot_row<ROWS, BK, KC, NT, NSLOT>(tid, KC ? it : 0), k;
    if constexpr (KC) {
      v = floatx4{reg[it].x, reg[it].y, reg[it].z, reg[it].w};
      k = slot_k<ROWS, BK, KC, NT>(tid, it);
    } else {
      row += it;
      v = floatx4{f4_get(reg[0], it), f4_get(reg[1], it), f4_get(reg[2], it), f4_get(reg[3], it)};
      k = slot_k<ROWS, BK, KC, NT>(tid, 0);
    }
    splitx4 part[kParts];
    guard.split(v, part);
    char* const p = lds + T::at(row, k / 8) + (k % 8) * 2;
#pragma unroll
    for (int q = 0; q < kParts; ++q) *reinterpret_cast<splitx4*>(p + q * T::kPlane) = part[q];
  }
}


// Tiled kernel for medium and large problems: BM x BN tile, k-slices of 32 in LDS as bf16 planes, the next slice in
// registers meanwhile; WAVES_M x WAVES_N wavefronts each owning a (BM/WAVES_M) x (BN/WAVES_N) sub-tile.
// CONV: the A operand is the implicit im2col view `cv` of a convolution input instead of a matrix.
// (A convolution: its output channels contiguous in B.)  CONV_RAGGED: its channel count is no multiple of 4.
enum ConvForm { kNoConv, kConvLean, kConvAligned, kConvRagged };
template <int BM, int BN, int BK, int WAVES_M, int WAVES_N, bool A_KC, bool B_KC, ConvForm FORM>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_mfma_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, const float* __restrict__ bias,
    int M, int N, int K, int nk, int nk_full, int tiles_m, int tiles_n, int total_blocks, long long strideA,
    long long strideB, long long strideC, int act, int m_fastest, ConvA cv) {
  constexpr bool CONV = FORM != kNoConv, LEAN = FORM == kConvLean;
  static_assert(!CONV || (A_KC && !B_KC), "the im2col view is K-contiguous, the filter [K,N]");
  constexpr int NT = 64 * WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 32, TN = WN / 32;
  static_assert(WM % 32 == 0 && WN % 32 == 0 && BK == 32, "tile shape");
  using TA = PlaneTile<BM, A_KC>;
  using TB = PlaneTile<BN, B_KC>;
  static_assert(BM * BK / 4 % NT == 0 && BN * BK / 4 % NT == 0, "loader shape");
  constexpr int SA = BM * BK / 4 / NT, SB = BN * BK / 4 / NT;

  __shared__ __align__(16) char lds_a[TA::kBytes];
  __shared__ __align__(16) char lds_b[TB::kBytes];

  // XCD-aware block order: hardware block id x lands on XCD x % 8.  Give each XCD a contiguous
  // range of logical tiles (same batch, neighbouring tiles) so that its L2 sees each A / B panel once.
  // Within a batch, consecutive tiles walk along M when B is the larger operand (every XCD then owns
  // a column slice of B and only the smaller A is fetched by several L2s), along N otherwise.
  const int bid = blockIdx.x;
  const int q = total_blocks / kXcds, rem = total_blocks % kXcds;
  const int xcd = bid % kXcds;
  const int vid = xcd * q + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int tiles = tiles_m * tiles_n;
  const int batch = vid / tiles;
  const int t = vid % tiles;
  const int tile_m = m_fastest ? t % tiles_m : t / tiles_n;
  const int tile_n = m_fastest ? t / tiles_m : t % tiles_n;

  const int lda = A_KC ? K : M;
  const int ldb = B_KC ? K : N;
  A += (size_t)batch * strideA;
  B += (size_t)batch * strideB;
  C += (size_t)batch * strideC;

  const int tid = threadIdx.x;
  const int wave = tid / 64, lane = tid % 64;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  const int li = lane % 32, h = lane / 32;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // bias for this lane's output columns, fetched now so that its latency hides under the main loop
  float bv[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn0 + 32 * j + li;
    bv[j] = (bias != nullptr && col < N) ? bias[col] : 0.f;
  }

  float4 ra[SA], rb[SB];
  ConvRow crow[CONV && !LEAN ? SA : 1];
  if constexpr (CONV && !LEAN) conv_rows<BM, BK, NT, SA>(cv, M, m0, tid, crow);
  const float* cp0[SA];  // lean loader only
  unsigned cok[SA];
  // filter tap (kh, kw), its index and the channel offset of the next slice load_a is asked for (slices are
  // requested in order 0, 1, 2, ...); uniform across the workgroup
  int tap_c0 = 0, tap_kh = 0, tap_kw = 0, tap_idx = 0;
  if constexpr (LEAN) conv_lean_rows<BM, BK, NT, SA>(cv, M, K, m0, tid, cp0, cok);
  // k-slices that lie entirely inside K take the branch-free loaders
  const float* pa[SA];
  const float* pb[SB];
  if constexpr (!CONV) slot_pointers<BM, BK, A_KC, NT, SA>(A, lda, M, m0, tid, pa);
  if constexpr (FORM != kConvRagged) slot_pointers<BN, BK, B_KC, NT, SB>(B, ldb, N, n0, tid, pb);
  const size_t step_a = A_KC ? (size_t)BK : (size_t)BK * lda, step_b = B_KC ? (size_t)BK : (size_t)BK * ldb;
  const unsigned total_a = (unsigned)strideA, total_b = (unsigned)strideB;
  const int kb = FORM == kConvRagged ? cv.Ci : K;  // valid k of B (per tap)
  // FULL: k-slice kt is known to lie inside K (for both operands)
  auto load_a = [&](int kt, auto full) __attribute__((always_inline)) {
    if constexpr (LEAN) {
      load_tile_conv_lean<SA>(cp0, cok, tap_idx, ((long long)tap_kh * cv.W + tap_kw) * cv.Ci + tap_c0, ra);
      tap_c0 += BK;
      if (tap_c0 >= cv.Ci) {
        tap_c0 = 0;
        ++tap_idx;
        if (++tap_kw == cv.fw) {
          tap_kw = 0;
          ++tap_kh;
        }
      }
    } else if constexpr (CONV) load_tile_conv<BK, SA>(cv, kt * BK, tid, crow, ra);
    else if constexpr (decltype(full)::value) load_tile_full<SA>(pa, kt * step_a, ra);
    else load_tile_any<BM, BK, A_KC, false, NT, SA>(A, lda, M, K, m0, kt * BK, tid, total_a, cv.fk, ra);
  };
  auto load_b = [&](int kt, auto full) __attribute__((always_inline)) {
    if constexpr (FORM != kConvRagged && decltype(full)::value) load_tile_full<SB>(pb, kt * step_b, rb);
    else load_tile_any<BN, BK, B_KC, FORM == kConvRagged, NT, SB>(B, ldb, N, kb, n0, kt * BK, tid, total_b, cv.fk, rb);
  };
  SplitGuard guard;
  auto store = [&](int kt, auto full) __attribute__((always_inline)) {
    if constexpr (CONV && !LEAN) settle_tile_conv<BK, FORM == kConvRagged, SA>(cv, kt * BK, tid, crow, ra);
    else if constexpr (!CONV && !decltype(full)::value)
      settle_tile<BM, BK, A_KC, false, NT, SA>(lda, M, K, m0, kt * BK, tid, total_a, cv.fk, ra);
    if constexpr (FORM == kConvRagged || !decltype(full)::value)
      settle_tile<BN, BK, B_KC, FORM == kConvRagged, NT, SB>(ldb, N, kb, n0, kt * BK, tid, total_b, cv.fk, rb);
    store_planes<BM, BK, A_KC, NT, SA>(lds_a, tid, ra, guard);
    store_planes<BN, BK, B_KC, NT, SB>(lds_b, tid, rb, guard);
  };
  auto first = [&](auto full) __attribute__((always_inline)) {
    load_a(0, full);
    load_b(0, full);
    store(0, full);
  };
  if (nk_full > 0) first(std::true_type{});
  else first(std::false_type{});
  __syncthreads();

  // where this lane's fragments start: row of the tile, piece h of k-step 0 (piece 2 + h of k-step 1)
  auto read = [&](const char* lds, auto tile, int row, int step, bf16x8 (&frag)[kParts]) __attribute__((always_inline)) {
    using T = decltype(tile);
#pragma unroll
    for (int p = 0; p < kParts; ++p) frag[p] = *reinterpret_cast<const bf16x8*>(lds + T::at(row, 2 * step + h) + p * T::kPlane);
  };
  // One k-slice: fetch slice kt + 1 into registers, multiply slice kt from LDS, hand the registers to LDS once every
  // wavefront has read it.  NEXT_FULL: slice kt + 1 exists and lies inside K.
  auto k_slice = [&](int kt, auto next_full) __attribute__((always_inline)) {
    constexpr bool NEXT_FULL = decltype(next_full)::value;
    if (NEXT_FULL || kt + 1 < nk) {
      load_a(kt + 1, next_full);
      load_b(kt + 1, next_full);
    }
    __builtin_amdgcn_s_setprio(1);  // MFMA phase: do not let the co-resident workgroup's wave cut in
#pragma unroll
    for (int step = 0; step < BK / 16; ++step) {
      bf16x8 fa[TM][kParts], fb[TN][kParts];
#pragma unroll
      for (int i = 0; i < TM; ++i) read(lds_a, TA(), wm0 + 32 * i + li, step, fa[i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) read(lds_b, TB(), wn0 + 32 * j + li, step, fb[j]);
#pragma unroll
      for (int s = 0; s < kSplitPasses; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][split_pass_a(s)], fb[j][split_pass_b(s)], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_s_setprio(0);
    if (NEXT_FULL || kt + 1 < nk) {
      __syncthreads();
      store(kt + 1, next_full);
      __syncthreads();
    }
  };
  int kt = 0;
  for (; kt + 1 < nk_full; ++kt) k_slice(kt, std::true_type{});
  for (; kt < nk; ++kt) k_slice(kt, std::false_type{});
  const ActClamp clamp = make_act(act);
  // Epilogue: bias[col] then activation, one dword per lane per register (two 128-byte rows per store).
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn0 + 32 * j + li;
    if (col >= N) continue;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = m0 + wm0 + 32 * i + 8 * (v / 4) + 4 * h + (v % 4);
        if (row < M) C[(size_t)row * N + col] = apply_act(acc[i][j][v] + bv[j], clamp);
      }
    }
  }
  // Values that the split does not carry (split.h): results that are Inf or NaN, and small ones if it lost bits of an operand
  // of this workgroup, once more with the fp32 instructions,
  // over what was stored.
  unsigned most = 0;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) see_result(most, acc[i][j][v]);
  bool again = overflowed(most);
  float limit = 0.f;
  if (__syncthreads_or(guard.lost())) {
    limit = __syncthreads_or(guard.large()) ? INFINITY : small_limit(CONV ? cv.Ci * cv.fk.taps : K);
    float least = INFINITY;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) least = fminf(least, fabsf(acc[i][j][v] + bv[j]));
    again = again || least < limit;
  }
  auto wanted = [&](float r, float b) __attribute__((always_inline)) { return !__builtin_isfinite(r) || fabsf(r + b) < limit; };
  if (__builtin_amdgcn_ballot_w64(again) != 0) {
    const int depth = CONV ? cv.Ci : K, taps = CONV ? cv.fk.taps : 1;
    // 8 consecutive k of a row or column, next to each other or `ld` elements apart, zeros from `valid` on
    auto fetch = [&](const float* p, auto contiguous, int ld, int valid, float (&f)[8]) __attribute__((always_inline)) {
      constexpr bool KC = decltype(contiguous)::value;
      if (KC && valid >= 8) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float4 v = load_quad(p + 4 * q);
          f[4 * q] = v.x, f[4 * q + 1] = v.y, f[4 * q + 2] = v.z, f[4 * q + 3] = v.w;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = e < valid ? p[KC ? (size_t)e : (size_t)e * ld] : 0.f;
      }
    };
#pragma unroll
    for (int block = 0; block < TM * TN; ++block) {
      const floatx16& r = acc[block / TN][block % TN];
      const float b = bv[block % TN];
      bool any = false;
#pragma unroll
      for (int v = 0; v < 16; ++v) any = any || wanted(r[v], b);
      if (__builtin_amdgcn_ballot_w64(any) == 0) continue;
      const int row = min(m0 + wm0 + 32 * (block / TN) + li, M - 1), col = min(n0 + wn0 + 32 * (block % TN) + li, N - 1);
      floatx16 exact;
#pragma unroll
      for (int v = 0; v < 16; ++v) exact[v] = 0.f;
      for (int tap = 0; tap < taps; ++tap) {
        const float* ap = A + (A_KC ? (size_t)row * lda : (size_t)row);
        bool inside = true;
        if constexpr (CONV) {
          const int t = row / cv.OW, n = t / cv.OH, kh = tap / cv.fw;
          const int ih = (t - n * cv.OH) * cv.sh - cv.pt + kh, iw = (row - t * cv.OW) * cv.sw - cv.pl + tap - kh * cv.fw;
          inside = ih >= 0 && ih < cv.H && iw >= 0 && iw < cv.W;
          ap = cv.x + (inside ? (((size_t)n * cv.H + ih) * cv.W + iw) * cv.Ci : 0);
        }
        const float* bp = B + (B_KC ? (size_t)col * ldb : (size_t)tap * depth * ldb + col);
#pragma unroll 1
        for (int k = 8 * h; k - 8 * h < depth; k += 16) {
          float fa[8], fb[8];
          fetch(ap + (A_KC ? (size_t)k : (size_t)k * lda), std::bool_constant<A_KC>{}, lda, inside ? depth - k : 0, fa);
          fetch(bp + (B_KC ? (size_t)k : (size_t)k * ldb), std::bool_constant<B_KC>{}, ldb, depth - k, fb);
#pragma unroll
          for (int e = 0; e < 8; ++e) exact = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[e], fb[e], exact, 0, 0, 0);
        }
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int out = m0 + wm0 + 32 * (block / TN) + 8 * (v / 4) + 4 * h + (v % 4);
        if (wanted(r[v], b) && out < M && n0 + wn0 + 32 * (block % TN) + li < N) C[(size_t)out * N + col] = apply_act(exact[v] + b, clamp);
      }
    }
  }
}

template <int BM, int BN, int BK, int WAVES_M, int WAVES_N, bool A_KC, bool B_KC, ConvForm FORM = kNoConv>
int launch_cfg(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, int act,
               hipStream_t stream, const ConvA& cv = ConvA{}) {
  auto kern = gemm_mfma_kernel<BM, BN, BK, WAVES_M, WAVES_N, A_KC, B_KC, FORM>;
  const int tiles_m = (m + BM - 1) / BM, tiles_n = (n + BN - 1) / BN;
  const long long total = (long long)batch * tiles_m * tiles_n;
  if (total > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  // k-slices, and how many of them lie inside K and (rows of no multiple of 4 elements) before a row-contiguous
  // operand's last row; with fewer than 4 rows / columns a quad reaches past more than one row: none
  const int kp = FORM == kConvRagged ? cv.fk.taps * (int)cv.fk.by_cp.d : k;
  const bool whole = (FORM != kNoConv || A_KC || m % 4 == 0) && (B_KC || n % 4 == 0);
  int full = whole ? k / BK : (k - 1) / BK;
  if ((FORM == kNoConv && !A_KC && m < 4) || (!B_KC && n < 4) || FORM == kConvRagged) full = 0;
  hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(64 * WAVES_M * WAVES_N), 0, stream, a, b, c,
                     bias, m, n, k, (kp + BK - 1) / BK, full, tiles_m, tiles_n, (int)total, (long long)m * k, (long long)n * k,
                     (long long)m * n, act, n > m ? 1 : 0, cv);
  return check_launch();
}

template <int BM, int BN, int BK, int WAVES_M, int WAVES_N>
int launch_layout(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k,
                  bool a_kc, bool b_kc, int act, hipStream_t stream) {
  if (a_kc)
    return b_kc ? launch_cfg<BM, BN, BK, WAVES_M, WAVES_N, true, true>(a, b, c, bias, batch, m, n, k, act, stream)
                : launch_cfg<BM, BN, BK, WAVES_M, WAVES_N, true, false>(a, b, c, bias, batch, m, n, k, act, stream);
  return b_kc ? launch_cfg<BM, BN, BK, WAVES_M, WAVES_N, false, true>(a, b, c, bias, batch, m, n, k, act, stream)
              : launch_cfg<BM, BN, BK, WAVES_M, WAVES_N, false, false>(a, b, c, bias, batch, m, n, k, act, stream);
}

// ---------------------------------------------------------------------------------------------
// Layout of one MFMA 16x16x4 (wave64): A: lane l holds A[i = l % 16][k = l / 16]; B: lane l holds
// B[k = l / 16][j = l % 16]; D: register v of lane l holds D[i = 4 * (l / 16) + v][j = l % 16].
// Within a group of 16 consecutive k, lane quarter q = l / 16 takes k = 16g + 4q + s in step s.

// 16-row tiles without operand staging, for A stored [M,K], B stored [K,N] (the pointwise-conv layout) and
// K = 64 ... 1024 (a multiple of 16 per wavefront): the WAVES_K wavefronts of a workgroup split K into chunks of 16 ... 128, and every
// wavefront loads the MFMA operands of its chunk straight into registers -- its row of A as 128-bit loads (4
// consecutive k, the contraction order permuted inside groups of 16) and, for the same
// k, TN adjacent columns of B as one load (TN = 2: 16 lanes read 128 contiguous bytes of a row of B; output
// column 2c + j of the 32-column tile is then column c of MFMA column block j).  All loads of a wavefront are
// issued before its first MFMA; there is no LDS fill and no barrier before the split-K reduction, which takes
// 0.4-0.7 us off kernels that last 4-6 us (the batch-1 network's 56x56 ... 7x7 pointwise layers).
// CONV: A is the implicit-GEMM view of a convolution input with Ci = CHUNK channels and WAVES_K filter taps, one
// tap per wavefront (K = taps x Ci): a lane's A operand is 4 consecutive channels of its output pixel's input
// pixel under that tap, or zeros if the tap falls outside the image.
template <int CHUNK, int WAVES_K, int TN, bool CONV = false>
__global__ __launch_bounds__(64 * WAVES_K) void gemm_m16_direct_kernel(const float* __restrict__ A,
                                                                       const float* __restrict__ B, float* __restrict__ C,
                                                                       const float* __restrict__ bias, int M, int N, int K,
                                                                       int tiles_m, int tiles_n, int total_blocks, int act,
                                                                       int m_fastest, ConvA cv) {
  constexpr int G = CHUNK / 16;  // k-groups of 16 per wavefront
  static_assert(CHUNK % 16 == 0 && CHUNK <= 128 && (TN == 1 || TN == 2) && 64 * WAVES_K >= 256, "shape");
  __shared__ float red[WAVES_K * TN * 4 * 64];  // split-K partials: [wavefront][column block j][register v][lane]

  const int bid = blockIdx.x;
  const int q8 = total_blocks / kXcds, rem = total_blocks % kXcds;
  const int xcd = bid % kXcds;
  const int vid = xcd * q8 + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int tile_m = m_fastest ? vid % tiles_m : vid / tiles_n;
  const int tile_n = m_fastest ? vid / tiles_m : vid % tiles_n;
  const int tid = threadIdx.x, wk = tid / 64, lane = tid % 64, li = lane % 16, q = lane / 16;
  const int m0 = tile_m * 16, n0 = tile_n * 16 * TN;

  // operand addresses: rows / columns past the matrix are clamped (they only feed outputs that are not stored)
  const int arow = min(m0 + li, M - 1);
  const int bcol = min(n0 + TN * li, N - TN);
  const float* ap;
  bool inside = true;
  if constexpr (CONV) {
    const int ow = arow % cv.OW;
    const int t = arow / cv.OW;
    const int oh = t % cv.OH;
    const int n = t / cv.OH;
    const int ih = oh * cv.sh - cv.pt + wk / cv.fw, iw = ow * cv.sw - cv.pl + wk % cv.fw;
    inside = ih >= 0 && ih < cv.H && iw >= 0 && iw < cv.W;
    // outside the image: load from the (valid) clamped pixel, zero the values below
    const int ihc = min(max(ih, 0), cv.H - 1), iwc = min(max(iw, 0), cv.W - 1);
    ap = cv.x + (((size_t)n * cv.H + ihc) * cv.W + iwc) * CHUNK + 4 * q;
  } else {
    ap = A + (size_t)arow * K + wk * CHUNK + 4 * q;
  }
  const float* bp = B + (size_t)(wk * CHUNK + 4 * q) * N + bcol;
  float4 a[G];
  float b[G][4][TN];
#pragma unroll
  for (int g = 0; g < G; ++g) a[g] = *reinterpret_cast<const float4*>(ap + 16 * g);
  if constexpr (CONV) {
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (!inside) a[g] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const float* p = bp + (size_t)(16 * g + s) * N;
      if constexpr (TN == 2) {
        const float2 t = *reinterpret_cast<const float2*>(p);
        b[g][s][0] = t.x;
        b[g][s][1] = t.y;
      } else {
        b[g][s][0] = *p;
      }
    }

  // epilogue thread e < 256 owns register v = e / 64 of lane l = e % 64: row 4 (l / 16) + v, columns
  // TN (l % 16) ... + TN - 1; fetch its bias now
  const int ev = tid / 64, el = tid % 64;
  const int erow = m0 + 4 * (el / 16) + ev, ecol = n0 + TN * (el % 16);
  float ebias[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) ebias[j] = (tid < 256 && bias != nullptr && ecol + j < N) ? bias[ecol + j] : 0.f;

  floatx4 acc[2][TN];  // [chain][column block]
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[c][j][v] = 0.f;
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[s & 1][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f4_get(a[g], s), b[g][s][j], acc[s & 1][j], 0, 0, 0);
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((wk * TN + j) * 4 + v) * 64 + lane] = acc[0][j][v] + acc[1][j][v];
  __syncthreads();
  if (tid < 256 && erow < M) {
    const ActClamp clamp = make_act(act);
    float o[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float sum = ebias[j];
#pragma unroll
      for (int w = 0; w < WAVES_K; ++w) sum += red[((w * TN + j) * 4 + ev) * 64 + el];
      o[j] = apply_act(sum, clamp);
    }
    float* cp = C + (size_t)erow * N + ecol;
    if constexpr (TN == 2) {
      if (ecol + 1 < N) *reinterpret_cast<float2*>(cp) = make_float2(o[0], o[1]);
    } else {
      if (ecol < N) *cp = o[0];
    }
  }
}

// K one of the supported depths in 64 ... 1024, N even, 16-byte aligned A (K % 4 == 0 holds), 8-byte aligned B, C and bias.
bool m16_direct_supported(const float* a, const float* b, const float* c, const float* bias, int batch, int n, int k,
                          bool a_kc, bool b_kc) {
  const bool aligned = reinterpret_cast<uintptr_t>(a) % 16 == 0 && reinterpret_cast<uintptr_t>(b) % 8 == 0 &&
                       reinterpret_cast<uintptr_t>(c) % 8 == 0 && reinterpret_cast<uintptr_t>(bias) % 8 == 0;
  return batch == 1 && a_kc && !b_kc && aligned && n % 2 == 0 && n >= 2 &&
         (k == 64 || k == 96 || k == 128 || k == 192 || k == 256 || k == 384 || k == 512 || k == 768 || k == 1024);
}

template <int TN>
int launch_m16_direct(const float* a, const float* b, float* c, const float* bias, int m, int n, int k, int act,
                      hipStream_t stream) {
  const int tiles_m = (m + 15) / 16, tiles_n = (n + 16 * TN - 1) / (16 * TN);
  const long long total = (long long)tiles_m * tiles_n;
  if (total > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
#define TFX_DIRECT(CHUNK, WK)                                                                                      \
  hipLaunchKernelGGL((gemm_m16_direct_kernel<CHUNK, WK, TN>), dim3((unsigned)total), dim3(64 * WK), 0, stream, a, b, c, \
                     bias, m, n, k, tiles_m, tiles_n, (int)total, act, n > m ? 1 : 0, ConvA{})
  // K = chunk x wavefronts (the channel counts of the MobileNet family at widths 0.5, 0.75 and 1)
  if (k == 64) TFX_DIRECT(16, 4);
  else if (k == 96) TFX_DIRECT(16, 6);
  else if (k == 128) TFX_DIRECT(16, 8);
  else if (k == 192) TFX_DIRECT(32, 6);
  else if (k == 256) TFX_DIRECT(32, 8);
  else if (k == 384) TFX_DIRECT(48, 8);
  else if (k == 512) TFX_DIRECT(64, 8);
  else if (k == 768) TFX_DIRECT(96, 8);
  else TFX_DIRECT(128, 8);
#undef TFX_DIRECT
  return check_launch();
}

// One thread per output element: operands of fewer elements than a 16-byte load.
__global__ __launch_bounds__(256) void gemm_tiny_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                        float* __restrict__ C, const float* __restrict__ bias, int M, int N, int K,
                                                        int a_kc, int b_kc, long long total, int act) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int col = (int)(e % N);
  const long long r = e / N, batch = r / M;
  const int row = (int)(r % M);
  float sum = 0.f;
  for (int k = 0; k < K; ++k)
    sum += A[batch * M * K + (a_kc ? (long long)row * K + k : (long long)k * M + row)] *
           B[batch * N * K + (b_kc ? (long long)col * K + k : (long long)k * N + col)];
  C[e] = apply_act(sum + (bias != nullptr ? bias[col] : 0.f), act);
}

}  // namespace

int launch_gemm(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, bool a_kc,
                bool b_kc, int act, hipStream_t stream) {
  if ((long long)m * k < 4 || (long long)n * k < 4) {
    const long long total = (long long)batch * m * n;
    hipLaunchKernelGGL(gemm_tiny_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, a, b, c, bias, m, n, k,
                       a_kc ? 1 : 0, b_kc ? 1 : 0, total, act);
    return check_launch();
  }
  // Which kernel (kernel_cost.h).  Below 128 the contraction has constants of its own, in whole slices of the LDS tiles and
  // whole steps of the wavefronts that split it.
  double us128, us64, deep, direct[3];
  if (k < 128) {
    const int k32 = (k + 31) / 32 * 32, k64 = k < 64 ? 64 : k;
    us128 = KernelCost{128, 128, 5.26, .0258, 2.43, .0331, 2}.us(batch, m, n, k32);
    us64 = KernelCost{64, 64, 4.34, .0273, .686, .0116, 4}.us(batch, m, n, k32);
    deep = shallow_deep_us(batch, m, n, k);
    direct[0] = KernelCost{64, 64, 1.55, 0., 3.6, .0076}.us(batch, m, n, k);
    direct[1] = KernelCost{32, 64, 2.2, .0071, .69, .0125}.us(batch, m, n, k64);
    direct[2] = KernelCost{32, 32, 2.8, .0039, .33, .0069}.us(batch, m, n, k64);
  } else {
    us128 = KernelCost{128, 128, 1.5, .026, 4.7, .027, 2}.us(batch, m, n, k);
    us64 = KernelCost{64, 64, 3.6, .026, 1.27, .0102, 4}.us(batch, m, n, k);
    deep = KernelCost{16, n % 2 == 0 ? 32 : 16, 3.2, 0., .245, .0035}.us(batch, m, n, k);
    direct[0] = KernelCost{64, 64, 1.33, 0., 3.36, .0148}.us(batch, m, n, k);
    direct[1] = KernelCost{32, 64, 3.05, .0010, .88, .0090}.us(batch, m, n, k);
    direct[2] = KernelCost{32, 32, 3.48, .0012, .28, .0053}.us(batch, m, n, k);
  }
  // one or two products: the fp32 instructions are the more accurate ones (split.h)
  if (k <= kFewProducts) us128 = us64 = direct[0] = direct[1] = direct[2] = 1e30;
  const int form = direct[0] < direct[1] ? (direct[0] < direct[2] ? 0 : 2) : (direct[1] < direct[2] ? 1 : 2);
  const double best = fmin(fmin(us128, us64), fmin(deep, direct[form]));
  if (k <= 32 && (long long)m * k >= 8 && (long long)n * k >= 8 && thin_us(batch, m, n, k) <= best)
    return launch_gemm_thin(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream);
  if (m16_direct_supported(a, b, c, bias, batch, n, k, a_kc, b_kc)) {
    const bool wide = (long long)((m + 15) / 16) * ((n + 31) / 32) >= 160;
    if (KernelCost{16, wide ? 32 : 16, 2.63, 0., 0., .0041}.us(1, m, n, k) <= best)
      return wide ? launch_m16_direct<2>(a, b, c, bias, m, n, k, act, stream)
                  : launch_m16_direct<1>(a, b, c, bias, m, n, k, act, stream);
  }
  if (us128 == best) return launch_layout<128, 128, 32, 2, 2>(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream);
  if (us64 == best) return launch_layout<64, 64, 32, 1, 2>(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream);
  if (deep == best) return launch_gemm_deep(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream);
  return launch_gemm_direct(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream, form);
}

// 3x3 convolution of a small feature map (few 16 x 32 output tiles) with 16 / 32 / 64 / 128 input channels: one
// filter tap per wavefront, operands straight from memory (gemm_m16_direct_kernel<..., CONV>).
template <int CI>
int launch_conv3x3_direct(const ConvA& cv, const float* w, const float* bias, float* y, int m, int co, int act,
                          hipStream_t stream) {
  const int tiles_m = (m + 15) / 16, tiles_n = (co + 31) / 32;
  const int total = tiles_m * tiles_n;
  hipLaunchKernelGGL((gemm_m16_direct_kernel<CI, 9, 2, true>), dim3((unsigned)total), dim3(64 * 9), 0, stream, nullptr, w, y,
                     bias, m, co, 9 * CI, tiles_m, tiles_n, total, act, co > m ? 1 : 0, cv);
  return check_launch();
}

// Any geometry and channel counts with at least 8 elements of x and filter (conv2d_gemm_supported).
bool conv2d_gemm_supported(long long x_elems, int fh, int fw, int ci, int co) {
  const long long k = (long long)fh * fw * ci;
  return x_elems >= 8 && k * co >= 8 && k * co < (1LL << 31) && (long long)fh * fw * (ci + 7) < (1LL << 24);
}

int launch_conv2d_gemm(const float* x, const float* w, const float* bias, float* y, int n, int h, int wd, int ci, int fh,
                       int fw, int co, int oh, int ow, int sh, int sw, int pt, int pl, int act, hipStream_t stream) {
  const long long m = (long long)n * oh * ow, k = (long long)fh * fw * ci;
  if (m > 0x7fffffffLL || k > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  const ConvA cv{x,  h,  wd, ci, oh, ow, fw, sh, sw, pt, pl, (unsigned)((long long)n * h * wd * ci), fast_div((unsigned)fw),
                 fast_div((unsigned)ow), fast_div((unsigned)oh), FilterK{fast_div((unsigned)((ci + 3) / 4 * 4)), fh * fw}};
  const bool vec = reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(w) % 16 == 0 &&
                   ci % 4 == 0 && co % 4 == 0;
  // small maps (at most 512 tiles of 16 x 32: the tiled kernel would leave most CUs idle and run its 9 Ci / 32 k-slices
  // one after the other on the rest)
  const long long tiles16x32 = ((m + 15) / 16) * ((co + 31) / 32);
  if (vec && fh == 3 && fw == 3 && tiles16x32 <= 512 && reinterpret_cast<uintptr_t>(y) % 8 == 0 &&
      reinterpret_cast<uintptr_t>(bias) % 8 == 0) {
    if (ci == 16) return launch_conv3x3_direct<16>(cv, w, bias, y, (int)m, co, act, stream);
    if (ci == 32) return launch_conv3x3_direct<32>(cv, w, bias, y, (int)m, co, act, stream);
    if (ci == 64) return launch_conv3x3_direct<64>(cv, w, bias, y, (int)m, co, act, stream);
    if (ci == 128) return launch_conv3x3_direct<128>(cv, w, bias, y, (int)m, co, act, stream);
  }
  if (fh == 1 && fw == 1 && sh == sw && pt == 0 && pl == 0 && thin_pays(m, co, ci, false))
    return launch_conv1x1_thin(x, w, y, bias, (int)m, co, ci, act, stream, h, wd, oh, ow, sh);
  const double kp = (double)fh * fw * ((ci + 7) / 8 * 8);
  const double us128 = KernelCost{128, 128, 3.84, .031, 2.58, .0335, 2}.us(1, m, co, kp);
  const double us64 = KernelCost{64, 64, 4.49, .033, .79, .0138, 4}.us(1, m, co, kp);
  const double deep = KernelCost{16, co % 2 == 0 ? 32 : 16, 2.94, 0., .31, .0046}.us(1, m, co, kp);
  const double direct[3] = {KernelCost{64, 64, 1.17, 0., 3.72, .0167}.us(1, m, co, kp),
                            KernelCost{32, 64, 2.74, .0036, 1.16, .0095}.us(1, m, co, kp),
                            KernelCost{32, 32, 3.12, .0042, .49, .0057}.us(1, m, co, kp)};
  const int form = direct[0] < direct[1] ? (direct[0] < direct[2] ? 0 : 2) : (direct[1] < direct[2] ? 1 : 2);
  const double best = fmin(fmin(us128, us64), fmin(deep, direct[form]));
  // the window kernel where it is clearly ahead (the tiled kernels' times are modelled to 14 %; over 151 convolutions this line
  // costs 0.2 % against the faster kernel of each, and 10 % at most)
  double window_us;
  const int window = conv2d_window_form(n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, &window_us);
  if (window != 0 && window_us < .93 * best)
    return launch_conv2d_window(x, w, bias, y, n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream, window);
  if (deep == best || k <= kFewProducts) return launch_conv2d_deep(x, w, bias, y, n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream);
  if (direct[form] == best)
    return launch_conv2d_gemm_direct(x, w, bias, y, n, h, wd, ci, fh, fw, co, oh, ow, sh, sw, pt, pl, act, stream, form);
  // k-slices of 32 inside one filter tap, one validity bit per tap: the lean loader
  const bool lean = vec && ci % 32 == 0 && fh * fw <= 32;
#define TFX_CONV(T, FORM) launch_cfg<T, T, 32, T / 64, 2, true, false, FORM>(nullptr, w, y, bias, 1, (int)m, co, (int)k, act, stream, cv)
  if (us128 == best) return lean ? TFX_CONV(128, kConvLean) : ci % 4 == 0 ? TFX_CONV(128, kConvAligned) : TFX_CONV(128, kConvRagged);
  return lean ? TFX_CONV(64, kConvLean) : ci % 4 == 0 ? TFX_CONV(64, kConvAligned) : TFX_CONV(64, kConvRagged);
#undef TFX_CONV
}

}  // namespace tfx
