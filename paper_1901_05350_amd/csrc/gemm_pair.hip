// fp32 products of long contractions, C[b] = act(op(A[b]) * op(B[b]) + bias): the tiled kernel of gemm.hip on the binary16 matrix cores,
// operands split in two (pair.h).
//
// Against three bf16 parts (gemm.hip) a product takes three matrix instructions instead of six and LDS two planes instead of three;
// the split takes as many vector instructions (6 a value, of which 2.5 only look for values that it does not carry), and they are
// what bounds it now: 8 x 1024^3, of the SIMDs' cycles vector ALU 48 %, matrix pipe 28 %, at 2.2 GHz.  us, three parts and now:
// 8 x 1024^3 91 -> 68 - 72, 4096 x 1024 x 4096 236 -> 141, 2000^3 120 -> 79, 13 x 3225 x 961 x 725 396 -> 278; short ones, whose
// start (the scales are agreed on between two barriers) weighs more, stay in gemm.hip.
// Error against float64, normal operands, K = 1024 / 2048 / 4096: 128 x 128 2.2e-7 / 3.0e-7 / 4.1e-7, three parts 4.9 / 6.9 / 10.0;
// 64 x 64, whose sums are taken in parts, K = 325 / 2464 1.1e-7 / 1.6e-7, the kernels that split the contraction 1.3 / 2.7.
#include "gemm_slots.h"
#include "pair.h"

#include <cmath>
#include <type_traits>
#include <utility>

namespace tfx {
namespace {

// f(0) ... f(N - 1) with the number as a type: arrays indexed by it stay in registers however large the loop is
template <class F, int... I>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  for_each_index(f, std::make_integer_sequence<int, N>{});
}

constexpr int kXcds = 8;  // workgroups are dealt round-robin to the 8 XCDs, each with its own L2

// Loads of k-slices that lie entirely inside K: buffer loads from the tile's first element of the slice, whose bounds are
// the operand's end, at a 32-bit offset that is the same for all of a thread's slots but for a scalar (pointers for each took
// registers that the second accumulators need).  Rows past the end read zeros or, of a row-contiguous operand, other rows; they only
// feed output rows / columns that are never stored.  A slot of a row-contiguous operand may reach past the end of its row
// into the next one, so the slice with the last row is not one of these when the row length is no multiple of 4.
// byte offset of a thread's first slot from the tile's first element of a slice, and of slot `it` from that
template <int ROWS, int BK, bool KC, int NT, int NSLOT>
__device__ __forceinline__ unsigned slot_base(int ld, int tid) {
  const unsigned row = (unsigned)slot_row<ROWS, BK, KC, NT, NSLOT>(tid, 0), k = (unsigned)slot_k<ROWS, BK, KC, NT>(tid, 0);
  return 4u * (KC ? row * (unsigned)ld + k : k * (unsigned)ld + row);
}
template <int BK, bool KC, int NT>
__device__ __forceinline__ unsigned slot_step(int ld, int it) {
  return 4u * (unsigned)it * (unsigned)ld * (KC ? (unsigned)(NT / (BK / 4)) : 1u);
}
template <int BK, bool KC>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slice_buffer(const float* g, int ld, long long total, int row0, int kt) {
  const long long first = KC ? (long long)row0 * ld + (long long)kt * BK : (long long)kt * BK * ld + row0;
  const long long bytes = 4 * (total - first);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g) + first, 0, (int)(unsigned)(bytes < 0xffffffffll ? bytes : 0xffffffffll), 0x00020000);
}
__device__ __forceinline__ float4 load_slot(__amdgpu_buffer_rsrc_t from, unsigned offset) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(from, (int)offset, 0, 0));
}

// Registers -> LDS: splits a thread's slot (of a !KC operand, row `it` of its block) and writes its four k (8 bytes per plane), in
// three parts of eight vector instructions; `half` is what the second leaves for the third.
template <int ROWS, int BK, bool KC, int NT, int NSLOT, int it, int PART>
__device__ __forceinline__ void store_slot(char* __restrict__ lds, int tid, const float4 (&reg)[NSLOT], const PairScale& s, PairSeen& seen,
                                           pairx4& half) {
  using T = PlaneTile<ROWS, KC, 2>;
  static_assert(BK == 32, "rows of 32 k");
  const floatx4 v = KC ? floatx4{reg[it].x, reg[it].y, reg[it].z, reg[it].w}
                       : floatx4{f4_get(reg[0], it), f4_get(reg[1], it), f4_get(reg[2], it), f4_get(reg[3], it)};
  const float scale = s.scale();
  if constexpr (PART == 0) seen.see(v, s.tiny());
  if constexpr (PART == 1) {
    unsigned h, l;
    split2(v[0], v[1], scale, h, l);
    half = pairx4{h, l};
  }
  if constexpr (PART == 2) {
    unsigned h, l;
    split2(v[2], v[3], scale, h, l);
    const int row = slot_row<ROWS, BK, KC, NT, NSLOT>(tid, KC ? it : 0) + (KC ? 0 : it), k = slot_k<ROWS, BK, KC, NT>(tid, KC ? it : 0);
    char* const p = lds + T::at(row, k / 8) + (k % 8) * 2;
    *reinterpret_cast<pairx4*>(p) = pairx4{half[0], h};
    *reinterpret_cast<pairx4*>(p + T::kPlane) = pairx4{half[1], l};
  }
}

template <int NSLOT>
__device__ __forceinline__ float largest_of(const float4 (&reg)[NSLOT]) {
  float most = 0.f;
#pragma unroll
  for (int it = 0; it < NSLOT; ++it) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(most) : "v"(reg[it].x), "v"(reg[it].y));
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(most) : "v"(reg[it].z), "v"(reg[it].w));
  }
  return most < INFINITY ? most : 0.f;
}

// BM x BN tile, k-slices of 32 in LDS as two planes of halfs, double-buffered, the slice after that in registers; WAVES_M x WAVES_N
// wavefronts each owning a (BM/WAVES_M) x (BN/WAVES_N) sub-tile.
template <int BM, int BN, int BK, int WAVES_M, int WAVES_N, bool A_KC, bool B_KC>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, 2) void gemm_pair_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, const float* __restrict__ bias,
    int M, int N, int K, int nk, int nk_full, int tiles_m, int tiles_n, int total_blocks, long long strideA,
    long long strideB, long long strideC, int act, int m_fastest) {
  constexpr int NT = 64 * WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr bool FINE = BM == 64;
  static_assert(WM % 32 == 0 && WN % 32 == 0 && BK == 32, "tile shape");
  using TA = PlaneTile<BM, A_KC, 2>;
  using TB = PlaneTile<BN, B_KC, 2>;
  static_assert(BM * BK / 4 % NT == 0 && BN * BK / 4 % NT == 0, "loader shape");
  constexpr int SA = BM * BK / 4 / NT, SB = BN * BK / 4 / NT;

  __shared__ __align__(16) char lds_a[2 * TA::kBytes];
  __shared__ __align__(16) char lds_b[2 * TB::kBytes];
  __shared__ int largest[2];  // bits of the operands' largest values

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

  int tid, lane, li, h, wm0, wn0;
  // The empty asm keeps what depends on the thread from being computed once for both attempts and kept: there are no registers for it.
  auto place = [&]() __attribute__((always_inline)) {
    tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave = tid / 64;
    lane = tid % 64, li = lane % 32, h = lane / 32;
    wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  };
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  floatx16 acc[TM][TN], mixed[TM][TN];  // products of the first parts, and the others times 2^11 (pair.h)

  float4 ra[SA], rb[SB];
  // k-slices that lie entirely inside K take the branch-free loaders
  unsigned base_a, base_b;  // byte offsets of the first slots in a slice
  auto fetch_a = [&](int w, int kt) __attribute__((always_inline)) {
    ra[w] = load_slot(slice_buffer<BK, A_KC>(A, lda, strideA, m0, kt), base_a + slot_step<BK, A_KC, NT>(lda, w));
  };
  auto fetch_b = [&](int w, int kt) __attribute__((always_inline)) {
    rb[w] = load_slot(slice_buffer<BK, B_KC>(B, ldb, strideB, n0, kt), base_b + slot_step<BK, B_KC, NT>(ldb, w));
  };
  const unsigned total_a = (unsigned)strideA, total_b = (unsigned)strideB;
  // FULL: k-slice kt is known to lie inside K (for both operands)
  auto load_a = [&](int kt, auto full) __attribute__((always_inline)) {
    if constexpr (decltype(full)::value) {
#pragma unroll
      for (int w = 0; w < SA; ++w) fetch_a(w, kt);
    } else {
      load_tile_any<BM, BK, A_KC, false, NT, SA>(A, lda, M, K, m0, kt * BK, tid, total_a, FilterK{}, ra);
    }
  };
  auto load_b = [&](int kt, auto full) __attribute__((always_inline)) {
    if constexpr (decltype(full)::value) {
#pragma unroll
      for (int w = 0; w < SB; ++w) fetch_b(w, kt);
    } else {
      load_tile_any<BN, BK, B_KC, false, NT, SB>(B, ldb, N, K, n0, kt * BK, tid, total_b, FilterK{}, rb);
    }
  };
  auto load = [&](int kt, auto full) __attribute__((always_inline)) {
    load_a(kt, full);
    load_b(kt, full);
  };
  auto settle = [&](int kt, auto full) __attribute__((always_inline)) {  // (a slice inside K comes out of this as it went in)
    if constexpr (!decltype(full)::value) {
      settle_tile<BM, BK, A_KC, false, NT, SA>(lda, M, K, m0, kt * BK, tid, total_a, FilterK{}, ra);
      settle_tile<BN, BK, B_KC, false, NT, SB>(ldb, N, K, n0, kt * BK, tid, total_b, FilterK{}, rb);
    }
  };
  // The scales are those of the first slice, whose largest values are the tile's or not far from them.  A tile with values that these
  // do not carry, or with lost bits because they are far larger than the rest, is computed a second time, with the scales of all it
  // has seen.
  PairScale scale_a(0), scale_b(0);
  PairSeen seen_a, seen_b;
  auto agree = [&](float a, float b) __attribute__((always_inline)) {  // the largest values of all threads, in `largest`
    if (tid < 2) largest[tid] = 0;
    __syncthreads();
    float most[2] = {a, b};
#pragma unroll
    for (int o = 0; o < 2; ++o) {
#pragma unroll
      for (int m = 32; m > 0; m /= 2) most[o] = fmaxf(most[o], __shfl_xor(most[o], m));
      if (lane == 0) atomicMax(&largest[o], __float_as_int(most[o]));
    }
    __syncthreads();
    scale_a = PairScale(__builtin_amdgcn_readfirstlane(largest[0]));
    scale_b = PairScale(__builtin_amdgcn_readfirstlane(largest[1]));
  };
  // part c % 3 of slot c / 3 of slice kt to its buffer: A's first
  pairx4 half;
  auto store = [&](auto number, int kt) __attribute__((always_inline)) {
    constexpr int w = decltype(number)::value / 3, part = decltype(number)::value % 3;
    if constexpr (w < SA) store_slot<BM, BK, A_KC, NT, SA, w, part>(lds_a + (kt & 1) * TA::kBytes, tid, ra, scale_a, seen_a, half);
    else store_slot<BN, BK, B_KC, NT, SB, w - SA, part>(lds_b + (kt & 1) * TB::kBytes, tid, rb, scale_b, seen_b, half);
  };

  // where this lane's fragments start: row of the tile, piece h of k-step 0 (piece 2 + h of k-step 1)
  auto read = [&](const char* lds, auto tile, int row, int step, h8 (&frag)[2]) __attribute__((always_inline)) {
    using T = decltype(tile);
#pragma unroll
    for (int p = 0; p < 2; ++p) frag[p] = *reinterpret_cast<const h8*>(lds + T::at(row, 2 * step + h) + p * T::kPlane);
  };
  // One k-slice: multiplies slice kt from its buffer, splits slice kt + 1, which is in registers, into the other one and fetches slice
  // kt + 2.  FULL: both of those exist and lie inside K; a part of a slot is then split, or a slot fetched again, after every matrix
  // instruction (the split of a slice takes as many cycles as its products: 4096 x 1024 x 4096 176 us with the split behind the
  // products, 141 so).
  auto k_slice = [&](int kt, auto next_full) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(next_full)::value;
    const char* const buf_a = lds_a + (kt & 1) * TA::kBytes;
    const char* const buf_b = lds_b + (kt & 1) * TB::kBytes;
    constexpr int STEPS = BK / 16, MF = 3 * TM * TN, SLOTS = SA + SB;
    if (!FULL) __builtin_amdgcn_s_setprio(1);  // do not let the co-resident workgroup's wave cut in
    static_for<STEPS>([&](auto step_index) __attribute__((always_inline)) {
      constexpr int step = decltype(step_index)::value;
      h8 fa[TM][2], fb[TN][2];
#pragma unroll
      for (int i = 0; i < TM; ++i) read(buf_a, TA(), wm0 + 32 * i + li, step, fa[i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) read(buf_b, TB(), wn0 + 32 * j + li, step, fb[j]);
      static_for<MF>([&](auto index) __attribute__((always_inline)) {
        constexpr int x = decltype(index)::value, pass = x / (TM * TN), i = x / TN % TM, j = x % TN;
        // passes (low, high), (high, high), (high, low)
        if constexpr (pass == 1) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i][0], fb[j][0], acc[i][j], 0, 0, 0);
        else mixed[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i][pass == 0], fb[j][pass == 2], mixed[i][j], 0, 0, 0);
        if constexpr (FULL) {
          constexpr int t = step * MF + x, from = t * 3 * SLOTS / (STEPS * MF), count = (t + 1) * 3 * SLOTS / (STEPS * MF) - from;
          static_for<count>([&](auto number) __attribute__((always_inline)) {
            constexpr int c = from + decltype(number)::value, w = c / 3;
            store(std::integral_constant<int, c>{}, kt + 1);
            if constexpr (c % 3 == 2) {
              if constexpr (w < SA) {
                if constexpr (A_KC) fetch_a(w, kt + 2);
                else if constexpr (w == SA - 1) load_a(kt + 2, std::true_type{});
              } else {
                if constexpr (B_KC) fetch_b(w - SA, kt + 2);
                else if constexpr (w == SLOTS - 1) load_b(kt + 2, std::true_type{});
              }
            }
          });
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    });
    if constexpr (!FULL) {
      __builtin_amdgcn_s_setprio(0);
      if (kt + 1 < nk) {
        settle(kt + 1, next_full);
        static_for<3 * SLOTS>([&](auto c) __attribute__((always_inline)) { store(c, kt + 1); });
        if (kt + 2 < nk) load(kt + 2, next_full);
      }
    }
    __syncthreads();
  };
  // FINE: the large products of four slices are summed apart from those before, as many roundings as a sum of K / 128 parts has
  // besides the eight of a part, not K / 16: the products that gemm_direct.hip would take otherwise stay as exact as there.
  // (The 128 x 128 tile has no registers for it.)
  floatx16 total[FINE ? TM : 1][FINE ? TN : 1];
  auto fold = [&]() __attribute__((always_inline)) {
    if constexpr (FINE) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) total[i][j][v] += acc[i][j][v], acc[i][j][v] = 0.f;
    }
  };
  int lost = 0;
#pragma unroll 1
  for (int attempt = 0; attempt < 2; ++attempt) {
    place();
    base_a = slot_base<BM, BK, A_KC, NT, SA>(lda, tid);
    base_b = slot_base<BN, BK, B_KC, NT, SB>(ldb, tid);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc[i][j][v] = mixed[i][j][v] = 0.f;
          if constexpr (FINE) total[i][j][v] = 0.f;
        }
    auto start = [&](auto full) __attribute__((always_inline)) {
      load(0, full);
      settle(0, full);
      if (attempt == 0) agree(largest_of(ra), largest_of(rb));
      seen_a.least = seen_b.least = ~0u, seen_a.largest = seen_b.largest = 0;
      static_for<3 * (SA + SB)>([&](auto c) __attribute__((always_inline)) { store(c, 0); });
      if (decltype(full)::value || nk > 1) load(1, full);
    };
    if (nk_full >= 2) start(std::true_type{});
    else start(std::false_type{});
    __syncthreads();
    int kt = 0;
    for (; kt + 2 < nk_full; ++kt) {
      k_slice(kt, std::true_type{});
      if (FINE && kt % 4 == 3) fold();
    }
    for (; kt < nk; ++kt) k_slice(kt, std::false_type{});
    fold();
    const bool over = __syncthreads_or(seen_a.over(scale_a) || seen_b.over(scale_b)) != 0;
    const int mine = seen_a.lost(scale_a) | seen_b.lost(scale_b);
    lost = __syncthreads_or(mine != 0) == 0                   ? 0
           : __syncthreads_or((mine & kLostMost) != 0) != 0 ? kLostMost | kLostTiny
                                                              : kLostTiny;
    if (attempt == 1 || !(over || lost != 0)) break;
    const PairScale a = scale_a, b = scale_b;
    agree(seen_a.most < INFINITY ? seen_a.most : 0.f, seen_b.most < INFINITY ? seen_b.most : 0.f);
    if (!over && scale_a.e <= a.e && scale_b.e <= b.e) {  // (larger only where the first slice was zeros)
      scale_a = a, scale_b = b;
      break;
    }
  }
  place();
  float bv[TN];  // bias of this lane's output columns
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn0 + 32 * j + li;
    bv[j] = (bias != nullptr && col < N) ? bias[col] : 0.f;
  }
  const int exponent = scale_a.e + scale_b.e;
  const ActClamp clamp = make_act(act);
  const float lowest = clamp.on ? 0.f : -INFINITY;
  float finite = 0.f;  // NaN where a result is not
  // Epilogue: bias[col] then activation, one dword per lane per register (two 128-byte rows per store).  The median of three drops a
  // NaN; those results are computed again below.
  auto result = [&](int i, int j, int v) __attribute__((always_inline)) {
    const float r = ldexpf(fmaf(mixed[i][j][v], 1 / kLow, FINE ? total[FINE ? i : 0][FINE ? j : 0][v] : acc[i][j][v]), -exponent);
    acc[i][j][v] = r;
    finite = fmaf(r, 0.f, finite);
    return __builtin_amdgcn_fmed3f(r + bv[j], lowest, clamp.hi);
  };
  if (m0 + BM <= M && n0 + BN <= N) {  // scalar row addresses: the general form takes ten more vector instructions a value
    char* const first = reinterpret_cast<char*>(C + (size_t)(m0 + __builtin_amdgcn_readfirstlane(wm0)) * N + n0 + __builtin_amdgcn_readfirstlane(wn0));
    const unsigned off = 4u * (4u * (unsigned)h * (unsigned)N + (unsigned)li);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        char* const row = first + (size_t)(32 * i + 8 * (v / 4) + v % 4) * N * 4;
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<float*>(row + off + 128 * j) = result(i, j, v);
      }
  } else {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn0 + 32 * j + li;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = m0 + wm0 + 32 * i + 8 * (v / 4) + 4 * h + (v % 4);
          const float r = result(i, j, v);
          if (row < M && col < N) C[(size_t)row * N + col] = r;
        }
    }
  }
  // Values that the split does not carry (pair.h): results that are Inf or NaN, and small ones if it lost bits of an operand
  // of this workgroup, once more with the fp32 instructions,
  // over what was stored.
  bool again = finite != finite;
  float limit = 0.f;
  if (lost != 0) {
    limit = loss_limit(K, exponent, lost);
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
    // Up to eight results of a wavefront: a sum over its lanes for each (listed in LDS, where no tile is any more).
    constexpr int kFew = 8;
    int* const list = reinterpret_cast<int*>(lds_a) + 16 * __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    if (lane == 0) list[0] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int x = 0; x < TM * TN; ++x)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (wanted(acc[x / TN][x % TN][v], bv[x % TN])) {
          const int at = atomicAdd(list, 1);
          if (at < kFew) list[1 + at] = (16 * x + v) * 64 + lane;
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int few = __builtin_amdgcn_readfirstlane(*(volatile int*)list);
    if (few <= kFew) {
#pragma unroll 1
      for (int i = 0; i < few; ++i) {
        const int e = __builtin_amdgcn_readfirstlane(*(volatile int*)(list + 1 + i)), x = e / 1024, v = e / 64 % 16, l = e % 64;
        const int row = m0 + __builtin_amdgcn_readfirstlane(wm0) + 32 * (x / TN) + 8 * (v / 4) + 4 * (l / 32) + v % 4;
        const int col = n0 + __builtin_amdgcn_readfirstlane(wn0) + 32 * (x % TN) + l % 32;
        if (row >= M || col >= N) continue;
        const float* const ap = A + (A_KC ? (size_t)row * lda : (size_t)row);
        const float* const bp = B + (B_KC ? (size_t)col * ldb : (size_t)col);
        float sum = 0.f;
#pragma unroll 8
        for (int k = lane; k < K; k += 64) sum = fmaf(ap[A_KC ? (size_t)k : (size_t)k * lda], bp[B_KC ? (size_t)k : (size_t)k * ldb], sum);
#pragma unroll
        for (int m = 32; m > 0; m /= 2) sum += __shfl_xor(sum, m);
        if (lane == 0) C[(size_t)row * N + col] = apply_act(sum + (bias != nullptr ? bias[col] : 0.f), clamp);
      }
      return;
    }
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
      const float* const ap = A + (A_KC ? (size_t)row * lda : (size_t)row);
      const float* const bp = B + (B_KC ? (size_t)col * ldb : (size_t)col);
#pragma unroll 1
      for (int k = 8 * h; k - 8 * h < K; k += 16) {
        float fa[8], fb[8];
        fetch(ap + (A_KC ? (size_t)k : (size_t)k * lda), std::bool_constant<A_KC>{}, lda, K - k, fa);
        fetch(bp + (B_KC ? (size_t)k : (size_t)k * ldb), std::bool_constant<B_KC>{}, ldb, K - k, fb);
#pragma unroll
        for (int e = 0; e < 8; ++e) exact = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[e], fb[e], exact, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int out = m0 + wm0 + 32 * (block / TN) + 8 * (v / 4) + 4 * h + (v % 4);
        if (wanted(r[v], b) && out < M && n0 + wn0 + 32 * (block % TN) + li < N) C[(size_t)out * N + col] = apply_act(exact[v] + b, clamp);
      }
    }
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_KC, bool B_KC>
int launch_cfg(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, int act, hipStream_t stream) {
  constexpr int BK = 32;
  auto kern = gemm_pair_kernel<BM, BN, BK, WAVES_M, WAVES_N, A_KC, B_KC>;
  const int tiles_m = (m + BM - 1) / BM, tiles_n = (n + BN - 1) / BN;
  const long long total = (long long)batch * tiles_m * tiles_n;
  if (total > 0x7fffffffLL) return TFX_ERR_UNSUPPORTED;
  // how many k-slices lie inside K and (rows of no multiple of 4 elements) before a row-contiguous operand's last row; with fewer than
  // 4 rows / columns a quad reaches past more than one row, and with very long rows a slice past 32-bit offsets: none
  const bool whole = (A_KC || m % 4 == 0) && (B_KC || n % 4 == 0);
  int full = whole ? k / BK : (k - 1) / BK;
  if ((!A_KC && m < 4) || (!B_KC && n < 4) || (A_KC ? k : m) >= 1 << 23 || (B_KC ? k : n) >= 1 << 23) full = 0;
  hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(64 * WAVES_M * WAVES_N), 0, stream, a, b, c, bias, m, n, k, (k + BK - 1) / BK, full,
                     tiles_m, tiles_n, (int)total, (long long)m * k, (long long)n * k, (long long)m * n, act, n > m ? 1 : 0);
  return check_launch();
}

template <int BM, int BN, int WAVES_M, int WAVES_N>
int launch_layout(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, bool a_kc, bool b_kc, int act,
                  hipStream_t stream) {
  if (a_kc)
    return b_kc ? launch_cfg<BM, BN, WAVES_M, WAVES_N, true, true>(a, b, c, bias, batch, m, n, k, act, stream)
                : launch_cfg<BM, BN, WAVES_M, WAVES_N, true, false>(a, b, c, bias, batch, m, n, k, act, stream);
  return b_kc ? launch_cfg<BM, BN, WAVES_M, WAVES_N, false, true>(a, b, c, bias, batch, m, n, k, act, stream)
              : launch_cfg<BM, BN, WAVES_M, WAVES_N, false, false>(a, b, c, bias, batch, m, n, k, act, stream);
}

}  // namespace

int launch_gemm_pair(const float* a, const float* b, float* c, const float* bias, int batch, int m, int n, int k, bool a_kc, bool b_kc,
                     int act, hipStream_t stream, int tile) {
  return tile == 128 ? launch_layout<128, 128, 2, 2>(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream)
                     : launch_layout<64, 64, 1, 2>(a, b, c, bias, batch, m, n, k, a_kc, b_kc, act, stream);
}

}  // namespace tfx
