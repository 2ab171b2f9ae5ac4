// batchMatMul on 16-bit float storage for gfx950 (Section 4.1: the same matMul renders to a 32-bit
// or a 16-bit floating point texture; Listing 2 defines the product).
//   C[b] = half( act( op(A[b]) * op(B[b]) + bias[col] ) ),  operands, bias and result IEEE binary16,
// products accumulated in fp32 on the matrix cores (v_mfma_f32_32x32x16_f16: 32x32 outputs, 16 k
// per instruction, 8 consecutive k per lane and operand).
//
// A workgroup of WAVES_M x WAVES_N wavefronts computes a (32 TM WAVES_M) x (32 TN WAVES_N) tile;
// k-slices of 64 halfs are double-buffered in LDS as K-contiguous rows of 144 bytes (128 + 16
// padding: the 16-byte fragment reads of 32 consecutive rows fall on distinct banks).  The MFMA is
// issued with the operands swapped (B's fragment first), so a lane's accumulator registers hold 4
// consecutive output columns of one row and the epilogue stores 8 bytes at a time.
// One software-pipelined kernel takes every layout, size and alignment (ragged.h has the loads); small outputs with a
// long contraction go to gemm_deep.hip.
#include "kernel_cost.h"
#include "ragged.h"

#include <type_traits>

namespace tfx {
namespace {

typedef _Float16 half_t;
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kBK = 64;       // halfs per k-slice
constexpr int kLd = kBK + 8;  // LDS row stride in halfs
constexpr int kXcds = 8;

// One thread per output element: operands of fewer elements than a 16-byte load.
__global__ __launch_bounds__(256) void gemm_tiny_f16_kernel(const half_t* __restrict__ A, const half_t* __restrict__ B,
                                                            half_t* __restrict__ C, const half_t* __restrict__ bias, int M, int N,
                                                            int K, int a_kc, int b_kc, long long total, int act) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int col = (int)(e % N);
  const long long r = e / N, batch = r / M;
  const int row = (int)(r % M);
  float sum = 0.f;
  for (int k = 0; k < K; ++k)
    sum += (float)A[batch * M * K + (a_kc ? (long long)row * K + k : (long long)k * M + row)] *
           (float)B[batch * N * K + (b_kc ? (long long)col * K + k : (long long)k * N + col)];
  C[e] = (half_t)apply_act(sum + (bias != nullptr ? (float)bias[col] : 0.f), act);
}

// A slice of an operand in LDS: K-contiguous rows of kLd halfs, or (stored [K,N] or [K,M]) its 64 k-rows, each `rows` halfs and
// kPad, which puts the four k-rows of a transposing load on different banks.
constexpr int kPad = 32;
constexpr int tile_halfs(bool kc, int rows) { return kc ? rows * kLd : kBK * (rows + kPad); }

// Fragment of 32 rows (columns) x 16 k, from where lane 0's starts: lane (li, hh) gets 8 consecutive k from 8 hh on of row li.
// The transposing load gives lane i of 16 the four halfs at place i % 4 of the 8-byte pieces that lanes i / 4, i / 4 + 4, ... of
// the 16 point to: with piece l at k-row l / 4 and columns 4 (l % 4), four k of column i.
template <bool KC, int ROWS>
__device__ __forceinline__ int first_fragment(int row0, int lane) {
  if constexpr (KC) return (row0 + lane % 32) * kLd + 8 * (lane / 32);
  return (8 * (lane / 32) + lane % 16 / 4) * (ROWS + kPad) + row0 + 16 * (lane / 16 % 2) + 4 * (lane % 4);
}
template <bool KC, int ROWS>
__device__ __forceinline__ h8 fragment(const half_t* first, int block, int step) {
  if constexpr (KC) return *reinterpret_cast<const h8*>(first + 32 * block * kLd + 16 * step);
  typedef short s4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s4 lds_s4;
  const half_t* const p = first + 32 * block + 16 * step * (ROWS + kPad);
  const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p)), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p + 4 * (ROWS + kPad)));
  return __builtin_bit_cast(h8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Software-pipelined tile kernel.  The vector memory
// path delivers 64 bytes per clock to a CU, so a k-slice's global loads take a large part of the
// slice's MFMA time and must be spread evenly through it; the same holds for the LDS writes.
// Iteration kt (slice kt in LDS buffer kt & 1):
// after every few MFMAs one 16-byte slot of slice kt+1 (loaded SETS iterations earlier) moves from
// its registers to the other LDS buffer and the same registers are refilled with that slot of slice
// kt+1+SETS; one barrier per slice.
//
// Alignment and remainders cost nothing in that loop: the 16-byte loads and stores work at any address (rows that start
// at an odd half cost 5 - 20 % of the kernel's time, 4-byte aligned ones nothing), and only slices that reach past K,
// or hold a [K,N] operand's last row when N % 8 != 0, go through the masked form -- none of a contraction of whole slices (its last
// two did: 1024 x 1024 x 1024 7.6 -> 7.0 us, 16 x 1024 x 256 x 512 11.5 -> 10.7).  (Fetched half by half,
// 1999 x 1001 x 1023 took 42 us, now 12.5.)
template <int WAVES_M, int WAVES_N, int TM, int TN, bool A_KC, bool B_KC, int SETS>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_f16_pipe_kernel(
    const half_t* __restrict__ A, const half_t* __restrict__ B, half_t* __restrict__ C, const half_t* __restrict__ bias,
    int M, int N, int K, int tiles_m, int tiles_n, int total_blocks, int full_slices, long long strideA, long long strideB,
    long long strideC, int act, int group_m) {
  constexpr int kNT = 64 * WAVES_M * WAVES_N;
  constexpr int WM = 32 * TM, WN = 32 * TN;
  constexpr int BM = WM * WAVES_M, BN = WN * WAVES_N;
  constexpr int kTileA = tile_halfs(A_KC, BM), kTileB = tile_halfs(B_KC, BN);
  constexpr int SA = BM * 8 / kNT, SB = BN * 8 / kNT, SLOTS = SA + SB;  // 16-byte slots per thread and slice
  constexpr int STEPS = kBK / 16, MF = TM * TN;  // k-steps per slice, MFMAs per step
  static_assert(BM * 8 % kNT == 0 && BN * 8 % kNT == 0, "loader shape");
  extern __shared__ __align__(16) half_t smem_h[];
  half_t* const lds_a = smem_h;
  half_t* const lds_b = smem_h + 2 * kTileA;

  const int bid = blockIdx.x;
  const int q = total_blocks / kXcds, rem = total_blocks % kXcds;
  const int xcd = bid % kXcds;
  const int vid = xcd * q + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int tiles = tiles_m * tiles_n;
  const int batch = vid / tiles;
  const int t = vid % tiles;
  const int band = t / (group_m * tiles_n);
  const int band_rows = min(group_m, tiles_m - band * group_m);
  const int tb = t - band * group_m * tiles_n;
  const int tile_m = band * group_m + tb % band_rows;
  const int tile_n = tb / band_rows;

  A += (size_t)batch * strideA;
  B += (size_t)batch * strideB;
  C += (size_t)batch * strideC;

  const int tid = threadIdx.x;
  const int wave = tid / 64, lane = tid % 64;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  const int li = lane % 32, hh = lane / 32;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // slot w of a slice: w < SA is A's slot w, else B's slot w - SA; slot i of a K-contiguous operand covers
  // tile row (tid + i * kNT) / 8, halfs 8 * ((tid + i * kNT) % 8) ... + 7.  Rows past the matrix
  // are clamped to its last row (they only feed outputs that are never stored) and k-slices are
  // clamped to the last one, so every load is unconditional and in bounds; halfs past K are zeroed
  // with a mask.  The loop body therefore has no branch.
  //
  // An operand stored [K,N] or [K,M] keeps its k-rows in LDS: slot i covers row (tid + i * kNT) / (BN / 8), 16 bytes of it, and the
  // fragments are read with the transposing LDS load.  (Turned in registers, 4 k-rows x 8 columns a thread, into the
  // K-contiguous form, its 8-byte LDS writes, two to a bank, were what the kernel waited for: 2048 x 1024 x 1024 14.0 us,
  // now 10.6; 4096 x 2048 x 512 23.3 and 17.7.)
  const int srow = tid / 8, scol = 8 * (tid % 8);
  constexpr int kRowStep = kNT / 8;
  typedef ragged_u32x4 u32x4;
  u32x4 reg[SETS][SLOTS];
  unsigned boff[SLOTS];  // byte offset of the slot at k0 = 0 from its operand's base (operands hold < 2^31 elements)
  // row of slot i of such an operand, and its columns (past the matrix: any valid ones)
  auto krow = [&](bool is_a, int i) { return (tid + i * kNT) / ((is_a ? BM : BN) / 8); };
  auto kcol = [&](bool is_a, int i) {
    const int c = 8 * ((tid + i * kNT) % ((is_a ? BM : BN) / 8));
    return is_a ? (m0 + c < M ? (unsigned)(m0 + c) : 0u) : (n0 + c < N ? (unsigned)(n0 + c) : 0u);
  };
#pragma unroll
  for (int w = 0; w < SLOTS; ++w) {
    const bool is_a = w < SA;
    const int i = is_a ? w : w - SA;
    if (is_a ? A_KC : B_KC) {
      const int row = min((is_a ? m0 : n0) + srow + i * kRowStep, (is_a ? M : N) - 1);
      boff[w] = 2u * ((unsigned)row * (unsigned)K + (unsigned)scol);
    } else {
      boff[w] = 2u * ((unsigned)krow(is_a, i) * (unsigned)(is_a ? M : N) + kcol(is_a, i));
    }
  }
  const int nk = (K + kBK - 1) / kBK;
  const int k_last = (nk - 1) * kBK;
  // Where the masked form of slot w of the slice at k0 starts (element offset; any valid place for a slot past K), and
  // how many halfs early it is fetched so as not to leave the operand.
  auto masked_offset = [&](int w, int k0, unsigned* early) {
    const bool is_a = w < SA;
    unsigned off;
    if (is_a ? A_KC : B_KC) {
      off = boff[w] / 2u + (k0 + scol < K ? (unsigned)k0 : 0u - (unsigned)scol);
    } else {
      const int i = is_a ? w : w - SA, k = k0 + krow(is_a, i);
      off = (k < K ? (unsigned)k : 0u) * (unsigned)(is_a ? M : N) + kcol(is_a, i);
    }
    const unsigned at = min(off, (unsigned)(is_a ? strideA : strideB) - 8u);
    *early = off - at;
    return at;
  };
  // FULL: the slice starting at k0 lies inside K.  Then a load is the operand's base advanced by the slice
  // (uniform, scalar registers) plus the slot's constant 32-bit offset, and a store needs no mask: no vector
  // ALU instruction per slot (each one would take issue time from the matrix cores).
  auto load_slot = [&](int set, int w, int k0, auto full) __attribute__((always_inline)) {
    const bool is_a = w < SA;
    const half_t* g = is_a ? A : B;
    if constexpr (decltype(full)::value) {
      const size_t advance = (is_a ? A_KC : B_KC) ? (size_t)k0 : (size_t)k0 * (size_t)(is_a ? M : N);
      reg[set][w] = load16(reinterpret_cast<const half_t*>(reinterpret_cast<const char*>(g + advance) + boff[w]));
    } else {
      unsigned early;
      reg[set][w] = load16(g + masked_offset(w, k0, &early));
    }
  };
  // k0: first k of the slice the registers hold; the zeroing of halfs past K happens here, when the
  // registers are consumed, so that nothing waits on a load right after issuing it
  auto settled = [&](int set, int w, int k0) __attribute__((always_inline)) {
    unsigned early;
    masked_offset(w, k0, &early);
    return __builtin_amdgcn_ballot_w64(early != 0) != 0 ? shift_down<half_t>(reg[set][w], early) : reg[set][w];
  };
  auto store_slot = [&](int set, int w, int buf, int k0, auto full) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full)::value;
    const bool is_a = w < SA;
    const int i = is_a ? w : w - SA;
    half_t* const l = is_a ? lds_a + buf * kTileA : lds_b + buf * kTileB;
    if (is_a ? A_KC : B_KC) {
      *reinterpret_cast<u32x4*>(l + (srow + i * kRowStep) * kLd + scol) =
          FULL ? reg[set][w] : settled(set, w, k0) & first_elements<half_t>(K - (k0 + scol));
    } else {
      const int row = krow(is_a, i);
      const unsigned mask = FULL || k0 + row < K ? 0xffffffffu : 0u;
      *reinterpret_cast<u32x4*>(l + row * ((is_a ? BM : BN) + kPad) + 8 * ((tid + i * kNT) % ((is_a ? BM : BN) / 8))) =
          FULL ? reg[set][w] : settled(set, w, k0) & mask;
    }
  };
  constexpr std::false_type kMasked{};

  // slice 0 goes to LDS, slices 1 ... SETS stay in registers: slice i in set i % SETS
  auto prologue = [&](auto full) {
    constexpr bool FULL = decltype(full)::value;
#pragma unroll
    for (int i = 0; i < SETS; ++i)
#pragma unroll
      for (int w = 0; w < SLOTS; ++w) load_slot(i, w, FULL ? i * kBK : min(i * kBK, k_last), full);
#pragma unroll
    for (int w = 0; w < SLOTS; ++w) {
      store_slot(0, w, 0, 0, full);
      load_slot(0, w, FULL ? SETS * kBK : min(SETS * kBK, k_last), full);
    }
  };
  if (full_slices >= SETS + 1) prologue(std::true_type{});
  else prologue(kMasked);
  __syncthreads();

  // One k-slice: slice kt + 1 is stored, from set `which`, slice kt + 1 + SETS is fetched; `full`, `fetch_full`: they lie inside K.
  auto k_slice = [&](int kt, auto which, auto full, auto fetch_full) __attribute__((always_inline)) {
    constexpr int set = decltype(which)::value;
    const int cur = kt & 1;
    // the last iterations refetch the last slice (unused)
    const int k_next = min((kt + 1 + SETS) * kBK, k_last);
    const half_t* const la = lds_a + cur * kTileA + first_fragment<A_KC, BM>(wm0, lane);
    const half_t* const lb = lds_b + cur * kTileB + first_fragment<B_KC, BN>(wn0, lane);
    h8 fa[2][TM], fb[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[0][i] = fragment<A_KC, BM>(la, i, 0);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = fragment<B_KC, BN>(lb, j, 0);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + 1 < STEPS) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[(s + 1) & 1][i] = fragment<A_KC, BM>(la, i, s + 1);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[(s + 1) & 1][j] = fragment<B_KC, BN>(lb, j, s + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[s & 1][j], fa[s & 1][i], acc[i][j], 0, 0, 0);
          // memory instructions due after this MFMA: slots [p * SLOTS / ALL, (p + 1) * SLOTS / ALL) of the slice.
          // A slot's registers (slice kt+1, loaded one iteration ago) go to the other LDS buffer and are
          // refilled at once with the same slot of slice kt+2.
          constexpr int ALL = STEPS * MF;
          const int p = s * MF + i * TN + j;
#pragma unroll
          for (int w = p * SLOTS / ALL; w < (p + 1) * SLOTS / ALL; ++w) {
            store_slot(set, w, cur ^ 1, (kt + 1) * kBK, full);
            load_slot(set, w, k_next, fetch_full);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __syncthreads();
  };
  int kt = 0;
  constexpr std::true_type kFull{};
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, SETS - 1>;
  const bool even = full_slices == nk;  // no ragged slice: all fetches are full ones
  if constexpr (SETS == 1) {
    for (const int end = even ? nk : full_slices - 2; kt < end; ++kt) k_slice(kt, Set0{}, kFull, kFull);
    if constexpr (SLOTS <= 4)
      for (; kt < full_slices - 1; ++kt) k_slice(kt, Set0{}, kFull, kMasked);
    for (; kt < nk; ++kt) k_slice(kt, Set0{}, kMasked, kMasked);
  } else {
    // Pairs without a branch between them, across which the compiler would not count loads: slices whose fetch is full, then those
    // whose store is, then the rest.
    auto pairs = [&](int end, auto full, auto fetch_full) __attribute__((always_inline)) {
      for (; kt + 1 < end; kt += 2) {
        k_slice(kt, Set1{}, full, fetch_full);
        k_slice(kt + 1, Set0{}, full, fetch_full);
      }
    };
    pairs(even ? nk : full_slices - 1 - SETS, kFull, kFull);
    if (even) {
      if (kt < nk) k_slice(kt, Set1{}, kFull, kFull);
    } else {
      pairs(full_slices - 1, kFull, kMasked);
      pairs(nk, kMasked, kMasked);
      if (kt < nk) k_slice(kt, Set1{}, kMasked, kMasked);
    }
  }

  // Epilogue: every wavefront converts its WM x WN block to binary16 in a private LDS region (all k-slice buffers are
  // free after the loop's last barrier), then reads it back row-wise and stores 16 bytes per lane, 128 bytes of a row at
  // a time, at whatever address that is.
  const ActClamp clamp = make_act(act);
  constexpr int kLs = WN + 8;  // staging row stride in halfs
  static_assert((size_t)WAVES_M * WAVES_N * WM * kLs <= 2 * (size_t)(kTileA + kTileB), "staging fits in the slice buffers");
  half_t* stage = smem_h + wave * WM * kLs;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int cl = 32 * j + 8 * g + 4 * hh;  // column inside the wave's block
      const int col = n0 + wn0 + cl;
      float bv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) bv[e] = (bias != nullptr && col + e < N) ? (float)bias[col + e] : 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        h4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = (half_t)apply_act(acc[i][j][4 * g + e] + bv[e], clamp);
        *reinterpret_cast<h4*>(stage + (32 * i + li) * kLs + cl) = pk;
      }
    }
  }
  constexpr int kLanesPerRow = WN / 8, kRowsPerStep = 64 / kLanesPerRow;
  const int rr = lane / kLanesPerRow, cc = 8 * (lane % kLanesPerRow);
  const int col = n0 + wn0 + cc;
#pragma unroll
  for (int r0 = 0; r0 < WM; r0 += kRowsPerStep) {
    const int row = m0 + wm0 + r0 + rr;
    const h8 v = *reinterpret_cast<const h8*>(stage + (r0 + rr) * kLs + cc);
    if (row >= M || col >= N) continue;
    half_t* const cp = C + (size_t)row * N + col;
    if (col + 8 <= N) {
      *reinterpret_cast<ragged_u32x4_any*>(cp) = __builtin_bit_cast(u32x4, v);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (col + e < N) cp[e] = v[e];
    }
  }
}

// slices that need no mask: inside K, and without the last row of an operand whose rows end inside a 16-byte load
// (fewer than 8 columns: every load of a row reaches into later ones, so none)
int full_slices(bool a_kc, bool b_kc, int m, int n, int k) {
  auto rows_of_8 = [](bool kc, int inner) { return kc || inner % 8 == 0; };
  if ((!a_kc && m < 8) || (!b_kc && n < 8)) return 0;
  return rows_of_8(a_kc, m) && rows_of_8(b_kc, n) ? k / kBK : (k - 1) / kBK;
}

template <int WAVES_M, int WAVES_N, int TM, int TN, bool A_KC, bool B_KC, int SETS>
int launch_pipe_sets(const half_t* a, const half_t* b, half_t* c, const half_t* bias, int batch, int m, int n, int k, int act,
                hipStream_t stream) {
  constexpr int BM = 32 * TM * WAVES_M, BN = 32 * TN * WAVES_N, NT = 64 * WAVES_M * WAVES_N;
  constexpr size_t lds_bytes = 2 * (size_t)(tile_halfs(A_KC, BM) + tile_halfs(B_KC, BN)) * sizeof(half_t);
  static_assert(lds_bytes <= 160 * 1024, "LDS budget per workgroup");
  auto kern = gemm_f16_pipe_kernel<WAVES_M, WAVES_N, TM, TN, A_KC, B_KC, SETS>;
  static std::atomic<uint64_t> lds_allowed{0};
  if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds_bytes, lds_allowed) != TFX_OK) return TFX_ERR_LAUNCH;
  const int tiles_m = (m + BM - 1) / BM, tiles_n = (n + BN - 1) / BN;
  const long long total = (long long)batch * tiles_m * tiles_n;
  if (total > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  const int full = full_slices(A_KC, B_KC, m, n, k);
  hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(NT), lds_bytes, stream, a, b, c, bias, m, n, k, tiles_m, tiles_n,
                     (int)total, full, (long long)m * k, (long long)n * k, (long long)m * n, act, 4);
  return check_launch();
}

template <int WAVES_M, int WAVES_N, int TM, int TN, bool A_KC, bool B_KC>
int launch_pipe(const half_t* a, const half_t* b, half_t* c, const half_t* bias, int batch, int m, int n, int k, int act,
                hipStream_t stream) {
  constexpr int BM = 32 * TM * WAVES_M, BN = 32 * TN * WAVES_N;
  if constexpr (TM * TN <= 2) {
    const long long tiles = (long long)batch * ((m + BM - 1) / BM) * ((n + BN - 1) / BN);
    // Two slices on their way in registers where a CU has one workgroup, whose loads nothing else covers, and the contraction is
    // long: us with one set and with two, 1024 x 4096 x 1024 23.7 / 18.5, 2048 x 4000 x 300 23.3 / 17.4, 1500 x 896 x 800 7.9 / 7.5,
    // 2000 x 1024 x 1000 10.4 / 10.1, 512 x 512 x 512 four times 5.06 / 5.16; with a ragged last slice, which takes more of them
    // through the masked form, 900 x 2001 x 900 14.5 / 13.5, 1999 x 1023 x 1001 12.6 / 13.0, 1001 x 777 x 1003 7.7 / 8.1.
    const int nk = (k + kBK - 1) / kBK;
    if (tiles <= 256 && nk >= (full_slices(A_KC, B_KC, m, n, k) == nk ? 12 : 20))
      return launch_pipe_sets<WAVES_M, WAVES_N, TM, TN, A_KC, B_KC, 2>(a, b, c, bias, batch, m, n, k, act, stream);
  }
  return launch_pipe_sets<WAVES_M, WAVES_N, TM, TN, A_KC, B_KC, 1>(a, b, c, bias, batch, m, n, k, act, stream);
}

// Small M x N: too few 64 x 64 tiles for 256 CUs, and each tile is bound by memory latency, not by the matrix cores.
// 16 x 32 tiles (v_mfma_f32_16x16x32_f16), a tile as deep as K up to 512 so that the whole K panel is
// in flight in one memory round trip, the depth split over 8 wavefronts whose partial tiles are
// added through LDS by the 512 threads that also apply the epilogue.  A stored [M,K], B stored
// [K,N] (N % 8 == 0, K % 8 == 0, 16-byte aligned); B goes through the 4 x 8 register transpose
// of the pipelined kernel.
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(512) void gemm_f16_small_kernel(const half_t* __restrict__ A, const half_t* __restrict__ B,
                                                             half_t* __restrict__ C, const half_t* __restrict__ bias,
                                                             int M, int N, int K, int tiles_m, int tiles_n,
                                                             int total_blocks, long long strideA, long long strideB,
                                                             long long strideC, int act) {
  constexpr int BM = 16, BN = 32, BKS = 512, LD = BKS + 8, NT = 512, WAVES_K = 8;
  __shared__ __align__(16) half_t lds[(BM + BN) * LD];
  half_t* const lds_a = lds;
  half_t* const lds_b = lds + BM * LD;

  const int bid = blockIdx.x;
  const int q8 = total_blocks / kXcds, rem = total_blocks % kXcds;
  const int xcd = bid % kXcds;
  const int vid = xcd * q8 + (xcd < rem ? xcd : rem) + bid / kXcds;
  const int tiles = tiles_m * tiles_n;
  const int batch = vid / tiles;
  const int t = vid % tiles;
  const int tile_m = t % tiles_m, tile_n = t / tiles_m;  // consecutive workgroups share a column panel of B

  A += (size_t)batch * strideA;
  B += (size_t)batch * strideB;
  C += (size_t)batch * strideC;

  const int tid = threadIdx.x;
  const int wk = tid / 64, lane = tid % 64;
  const int li = lane % 16, q = lane / 16;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  // epilogue thread e owns the value of register v of lane l of column block j, e = (j * 4 + v) * 64 + l
  const int ej = tid / 256, ev = (tid / 64) % 4, el = tid % 64;
  const int erow = m0 + 4 * (el / 16) + ev, ecol = n0 + 16 * ej + el % 16;
  float ebias = 0.f;
  if (bias != nullptr && ecol < N) ebias = (float)bias[ecol];

  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  // A: 2 slots per thread, slot s = tid + 512 i: row s / 64, halfs 8 (s % 64) ... + 7
  // B: thread (kq = tid / 4, nb = tid % 4) owns k-rows 4 kq ... + 3 of columns 8 nb ... + 7
  u32x4 ra[2], rb[4];
  const int kq = tid / 4, nb = tid % 4;
  const unsigned bcol = n0 + 8 * nb < N ? (unsigned)(n0 + 8 * nb) : 0u;
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int s = tid + i * NT;
      const int row = min(m0 + s / 64, M - 1), k = k0 + 8 * (s % 64);
      ra[i] = *reinterpret_cast<const u32x4*>(A + (size_t)((unsigned)row * (unsigned)K + (k < K ? (unsigned)k : 0u)));
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int k = k0 + 4 * kq + kk;
      rb[kk] = *reinterpret_cast<const u32x4*>(B + (size_t)((k < K ? (unsigned)k : 0u) * (unsigned)N + bcol));
    }
  };
  auto store = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int s = tid + i * NT;
      const unsigned mask = k0 + 8 * (s % 64) < K ? 0xffffffffu : 0u;
      *reinterpret_cast<u32x4*>(lds_a + (s / 64) * LD + 8 * (s % 64)) = ra[i] & mask;
    }
    h8 r[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const unsigned mask = k0 + 4 * kq + kk < K ? 0xffffffffu : 0u;
      r[kk] = __builtin_bit_cast(h8, rb[kk] & mask);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const h4 o = {r[0][i], r[1][i], r[2][i], r[3][i]};
      *reinterpret_cast<h4*>(lds_b + (8 * nb + i) * LD + 4 * kq) = o;
    }
  };

  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  const int nk = (K + BKS - 1) / BKS;
  load(0);
  for (int kt = 0; kt < nk; ++kt) {
    if (kt > 0) __syncthreads();  // everyone has finished reading the previous slice
    store(kt * BKS);
    __syncthreads();
    if (kt + 1 < nk) load((kt + 1) * BKS);
#pragma unroll
    for (int s = 0; s < BKS / WAVES_K / 32; ++s) {
      const int kb = wk * (BKS / WAVES_K) + 32 * s;  // this wavefront's 32 k of the slice
      if (kt * BKS + kb >= K) break;                 // past the end of K: zeros
      const h8 fa = *reinterpret_cast<const h8*>(lds_a + li * LD + kb + 8 * q);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const h8 fb = *reinterpret_cast<const h8*>(lds_b + (16 * j + li) * LD + kb + 8 * q);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa, fb, acc[j], 0, 0, 0);
      }
    }
  }

  // add the 8 partial tiles through LDS: layout [wk][j][v][lane]
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds);
  static_assert(WAVES_K * 2 * 4 * 64 * sizeof(float) <= sizeof(lds), "reduction reuses the slice buffers");
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[(wk * 8 + j * 4 + v) * 64 + lane] = acc[j][v];
  __syncthreads();
  float sum = ebias;
#pragma unroll
  for (int w = 0; w < WAVES_K; ++w) sum += red[w * 512 + tid];
  if (erow < M && ecol < N) C[(size_t)erow * N + ecol] = (half_t)apply_act(sum, make_act(act));
}

int launch_small(const half_t* a, const half_t* b, half_t* c, const half_t* bias, int batch, int m, int n, int k,
                 int act, hipStream_t stream) {
  const int tiles_m = (m + 15) / 16, tiles_n = (n + 31) / 32;
  const long long total = (long long)batch * tiles_m * tiles_n;
  if (total > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(gemm_f16_small_kernel, dim3((unsigned)total), dim3(512), 0, stream, a, b, c, bias, m, n, k,
                     tiles_m, tiles_n, (int)total, (long long)m * k, (long long)n * k, (long long)m * n, act);
  return check_launch();
}

}  // namespace

int launch_gemm_f16(const uint16_t* a16, const uint16_t* b16, uint16_t* c16, const uint16_t* bias16, int batch, int m,
                    int n, int k, bool a_kc, bool b_kc, int act, hipStream_t stream) {
  const half_t* a = reinterpret_cast<const half_t*>(a16);
  const half_t* b = reinterpret_cast<const half_t*>(b16);
  half_t* c = reinterpret_cast<half_t*>(c16);
  const half_t* bias = reinterpret_cast<const half_t*>(bias16);
  if ((long long)m * k < 8 || (long long)n * k < 8) {
    const long long total = (long long)batch * m * n;
    hipLaunchKernelGGL(gemm_tiny_f16_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, a, b, c, bias, m, n, k,
                       a_kc ? 1 : 0, b_kc ? 1 : 0, total, act);
    return check_launch();
  }
  // the pointwise-convolution layout with a thin or deep filter held in LDS; short contractions
  if (batch == 1 && a_kc && !b_kc && pointwise_stream_f16_supported(m, k, n, a, b, c))
    return launch_pointwise_stream_f16(a16, b16, bias16, c16, m, k, n, act, stream);
  if (batch == 1 && a_kc && !b_kc && pointwise_slab_f16_supported(m, k, n, a, b, c))
    return launch_pointwise_slab_f16(a16, b16, bias16, c16, m, k, n, act, stream);
  if (batch == 1 && a_kc && thin_pays(m, n, k, true))
    return launch_gemm_thin_f16(a16, b16, c16, bias16, m, n, k, b_kc, act, stream);

  // Which kernel: the modelled time, fitted to 900 products (16 ... 4096 each way, batch 1 ... 32, every layout, half of the sizes of
  // no multiple of 8; near the choice the rms error is 5 - 8 % for the tiles and the small kernel, 12 and 15 % for the two others
  // that split the contraction).  Over these the choice costs 1.2 % on average against the fastest kernel of each, more than 25 %
  // for ten of them (32 x 121 x 442, 26 of a batch: 5.2 us, 4.2 with the direct kernel).
  const int k64 = (k + 63) / 64 * 64, k512 = (k + (k + 511) / 512 * 512) / 2;  // (the small kernel's slices are 512 deep)
  // operands whose rows have an odd number of halfs; they halve what 16-byte loads deliver to a kernel that does not share them
  // through LDS (2000 x 1000 x 1024 with B [N,K] 21 us, x 1023 53)
  const int odd = (a_kc ? k : m) % 2 + (b_kc ? k : n) % 2;
  const bool small = a_kc && !b_kc && k % 8 == 0 && n % 8 == 0 && reinterpret_cast<uintptr_t>(a) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(b) % 16 == 0;
  const bool direct = (k % 2 == 0 || !(a_kc || b_kc)) && n >= 2 && m >= 2;
  enum { kDeep, kSmall, kDirect, k64x64, k64x128, k128x128, k256x256, kForms };
  const int deep_n = deep_two_columns((long long)batch * ((m + 15) / 16), n, (k + 31) / 32) ? 32 : 16;
  const double us[kForms] = {1.05 * PipeCost{16, deep_n, 2.75, .011, .0017, 1., 1.39, .49, 1.5}.us(batch, m, n, k, odd),
                             small ? PipeCost{16, 32, 2.68, 0., .0019, .77, 1.07, 0., 1.5}.us(batch, m, n, k512, 0) : 1e30,
                             direct ? PipeCost{32, 64, 2.28, .99, .0055, .32, .61, .19, .13}.us(batch, m, n, k, odd) : 1e30,
                             PipeCost{64, 64, 3.73, .19, .0028, .78, 1.37, .27, .47, .0008}.us(batch, m, n, k64, odd),
                             PipeCost{64, 128, 3.34, .53, .0050, .91, 1.14, .22, .52, .0002}.us(batch, m, n, k64, odd),
                             PipeCost{128, 128, 4.20, .35, .0072, .91, 1.21, .20, .48}.us(batch, m, n, k64, odd),
                             PipeCost{256, 256, 7.14, 1.41, .0150, .90, 2., .14, .45, .0040}.us(batch, m, n, k64, odd)};
  int form = 0;
  for (int f = 1; f < kForms; ++f)
    if (us[f] < us[form]) form = f;
  if (form == kSmall) return launch_small(a, b, c, bias, batch, m, n, k, act, stream);
  if (form == kDeep) return launch_gemm_deep_f16(a16, b16, c16, bias16, batch, m, n, k, a_kc, b_kc, act, stream);
  if (form == kDirect) return launch_gemm_direct_f16(a16, b16, c16, bias16, batch, m, n, k, a_kc, b_kc, act, stream, 1);
  auto pick = [&](auto akc, auto bkc) {
    constexpr bool A_KC = decltype(akc)::value, B_KC = decltype(bkc)::value;
    if (form == k64x64) return launch_pipe<2, 2, 1, 1, A_KC, B_KC>(a, b, c, bias, batch, m, n, k, act, stream);
    if (form == k64x128) return launch_pipe<2, 4, 1, 1, A_KC, B_KC>(a, b, c, bias, batch, m, n, k, act, stream);
    if (form == k128x128) return launch_pipe<2, 4, 2, 1, A_KC, B_KC>(a, b, c, bias, batch, m, n, k, act, stream);
    return launch_pipe<2, 4, 4, 2, A_KC, B_KC>(a, b, c, bias, batch, m, n, k, act, stream);
  };
  if (a_kc) return b_kc ? pick(std::true_type{}, std::true_type{}) : pick(std::true_type{}, std::false_type{});
  return b_kc ? pick(std::false_type{}, std::true_type{}) : pick(std::false_type{}, std::false_type{});
}

}  // namespace tfx
