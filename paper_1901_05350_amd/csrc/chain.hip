// The small-map half of the batch-1 MobileNet v1 forward pass (Section 3.9, Table 1) as ONE kernel:
// the depthwise-separable blocks from the last 28 x 28 one (or the one after it) down to 7 x 7, the average pool, the fully
// connected layer and the softmax -- 20 dependent steps that, as 20 kernels of 3-6 us each, are
// bound by kernel boundaries and by each kernel's own start-up, not by their arithmetic.
//
// The kernel is persistent: 256 workgroups (one per CU) walk through the steps in order, and a step's
// work is cut into tasks that match the producers and consumers of the neighbouring steps:
//   depthwise task  = 16 consecutive output pixels x 32 channels (one output per thread),
//   pointwise task  = a 16-row x 16*TN-column tile of the pixel x channel GEMM, K split over the
//                     8 wavefronts, operands loaded straight into MFMA registers (the scheme of
//                     gemm_m16_direct_kernel), partial tiles added through LDS,
//   pool + fully connected task = 128 input channels x 128 classes, softmax = one task.
// There is no grid-wide barrier, and there are no flags.  Every step's output has memory of its own, which the first kernel of the pass
// fills with ones (chain_fill); a task writes each word of its output once, never as all ones (a NaN is stored as the one NaN
// 0x7fc00000), and a reader loads what it needs until no word of it is all ones.  What is read is what is waited for: no
// acknowledgement of the producer's stores, no barrier and no flag behind them, no second trip to memory behind a flag.  One full-width
// image of 224 x 224: the whole pass 91.1 us with a flag word for each task, 81.2 without, quarter width at 128 x 128 77.7 and 59.9.
// A pointwise task polls a word of each depthwise task first and loads its operand then: eight wavefronts' whole operands asked for
// again and again keep the memory busy (3/4 width at 192 x 192 86.3 us, 83.0 so).  Divisions of a step's critical path
// come from the host as multiplications (81.0 -> 78.3; quarter width 60.2 -> 55.2).  Tried and slower: filters fetched a step ahead, in
// front of a wait (loads return in order within a wavefront, so the polls return behind them: 90.4), the two kinds of tasks in
// workgroups of their own, two to a CU (82 - 90), offsets and filters of the next step computed before this one's wait (83 - 87).
//
// On binary16 storage (ChainParams<half_t>) a word is two channels: depthwise tasks have 64, a pointwise instruction takes 32 values of K,
// sums are floats and every layer rounds once.  The five launches in front (stem and block 1, which also fills; blocks 2 - 5) and
// this kernel, 38 us, take 63.3 us where 15 launches took 67.6 (of 3.4 us of host time each); 3/4 width 224 x 224 65.5 -> 58.8, half
// width 128 x 128 52.2 -> 46.3, quarter width 48.1 -> 42.7.
//
// Tiles of 16 or 32 columns: whichever takes fewer rounds of tasks.  With 32 from 160 such tasks on, some of 9 ... 13 row tiles, dealt to
// 8 XCDs, were two rounds: 3/4 width 192 x 192 80.9 -> 72.6 us, binary16 full width 192 x 192 67.8 -> 59.6.
//
// Visibility between workgroups on different XCDs (each XCD has its own L2) without cache write-back /
// invalidate instructions: every activation that one task writes and another reads moves through
// device-coherent accesses (the sc1 cache policy of agent-scope atomics: stores write through to
// the memory side, loads do not hit a stale line).  Filters and biases are read-only and use ordinary cached loads; they are
// fetched before the wait.
//
// No workgroup has to be resident for another one to end: a workgroup whose input does not come for kPatience polls (who has it to
// write is not running) leaves its tasks, and then computes every task of every step itself, in order, where each input is one that it
// has written before.  What is written twice is written with the same bits.  So any number of these kernels may run side by side --
// replays of captured passes on several streams, other processes -- and grids that keep each other's workgroups from the CUs end late,
// by 6 - 9 ms, but right.  (It costs nothing: one image, us, without and with, full width 224 x 224 78.5 / 78.5, 3/4 width 192 x 192 73.2 / 72.7,
// quarter width 128 x 128 55.1 / 54.4; binary16 62.9 / 62.95, 54.8 / 54.7, 42.6 / 42.1.)  The grid (256 workgroups, one per CU) is launched where
// all of it is resident at once (chain_grids), and launch_chain orders calls across streams such that no more of them run than the device
// holds: only replays of captured passes come to that.
//
// Every wait is bounded besides: a poll loop that still waits after kSpinLimit rounds (seconds; where a workgroup of the fully connected
// layer never gets to run) gives up and sets a failure word, and the softmax task then writes NaN to every output.
#include <algorithm>
#include <cstdlib>
#include <mutex>

#include "ragged.h"

namespace tfx {
namespace {

typedef _Float16 half_t;
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

constexpr int kChainThreads = 512;
constexpr int kChainWaves = kChainThreads / 64;
constexpr int kChainGrid = 256;
constexpr int kChainBlocks = 9;       // at most blocks 5 .. 13 of the network (0-based 4 .. 12)
constexpr int kFirstChainBlock = 4;   // a launch starts there or one block later (both read a 1/8-size map of 256 channels)
constexpr int kSpinLimit = 1 << 22;  // polls before a wait gives up (each poll is a memory round trip: seconds)
constexpr int kPatience = 4096;      // polls before a workgroup computes what it waits for itself (milliseconds)
constexpr int kFcSliceChannels = 128;  // input channels of the fully connected layer per task (2 to 8 slices)
constexpr int kFcColBlock = 128;      // classes per fully connected task
constexpr int kFcTasks = 64;          // at most: 8 slices x 8 blocks of classes
constexpr unsigned kEmpty = ~0u;       // a word of the chain's memory that no task has written yet
constexpr int kSc1 = 16;              // cache-policy operand of the buffer builtins: device-coherent access

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Tasks of a step with tiles_m x tiles_c tiles are dealt to workgroups so that a row tile's tasks fall on
// workgroups with the same id modulo 8, i.e. (workgroups are dealt to the 8 XCDs round robin) on one XCD -- or, with
// 1, 2 or 4 row tiles, on 8, 4 or 2 XCDs, so that no XCD stays idle: the exchange between a row tile's depthwise
// tasks and its pointwise tiles then stays inside an XCD's L2, which answers device-coherent accesses to lines it
// owns faster than the memory side does (measured: 1.3 against 1.8 us per dependent step).  Correctness does not
// depend on where workgroups run.  Workgroup w takes the virtual tasks vt = w, w + 256, ...; vt % 8 is the XCD.
struct TaskMap {
  int tiles_m, tiles_c, mode, shift, count;
  FastDiv by_c;  // division by tiles_c
};
TaskMap make_task_map(int tiles_m, int tiles_c) {
  TaskMap m{tiles_m, tiles_c, 2, 0, tiles_m * tiles_c, fast_div((unsigned)tiles_c)};  // mode 2: plain order
  if (tiles_m >= 8) {
    m.mode = 0, m.count = 8 * ((tiles_m + 7) / 8) * tiles_c;  // vt = r % 8 + 8 ((r / 8) tiles_c + c)
  } else if (tiles_m == 1 || tiles_m == 2 || tiles_m == 4) {
    const int f = 8 / tiles_m;  // XCD = r f + c % f, slot = c / f
    m.mode = 1, m.shift = f == 8 ? 3 : f == 4 ? 2 : 1, m.count = 8 * ((tiles_c + f - 1) / f);
  }
  return m;
}
__device__ __forceinline__ bool task_of(const TaskMap& m, int vt, int* r, int* c) {
  const int u = m.mode == 2 ? vt : vt / 8, by = (int)div_by((unsigned)u, m.by_c), rest = u - by * m.tiles_c;
  if (m.mode == 0) {
    *r = vt % 8 + 8 * by;
    *c = rest;
  } else if (m.mode == 1) {
    *r = (vt % 8) >> m.shift;
    *c = (u << m.shift) + (vt & ((1 << m.shift) - 1));
  } else {
    *r = by;
    *c = rest;
  }
  return *r < m.tiles_m && *c < m.tiles_c;
}

template <typename T>  // of the storage: float or half_t
struct ChainBlock {
  const T *dw_w, *dw_b, *pw_w, *pw_b;
  int in_hw, out_hw, stride, pad;  // square maps; pad = zero rows / columns before the image
  int cin, cout;
  int tn;                          // 16-column blocks per pointwise tile
  FastDiv by_hw;                   // division by out_hw
  TaskMap dw_map, pw_map;
  unsigned in_off, mid_off, out_off;  // element offsets in the chain workspace: input (0 for the first block, whose
                                   // input is a buffer of its own), depthwise output, pointwise output
};

template <typename T>
struct ChainParams {
  ChainBlock<T> blk[kChainBlocks];
  const T* in0;         // input of the first block (written by an earlier kernel)
  unsigned in0_bytes;
  void* act;            // chain workspace: every step's output
  unsigned act_bytes;
  int* failed;          // a wait has given up
  const T *fc_w, *fc_b;
  unsigned partial_at;  // byte offset in act: [feat / 128][classes] partial logits, floats
  T *probs, *logits;
  int classes, feat, last_hw;
  int spin_limit;       // polls before a wait gives up
  int patience;         // and before the workgroup does everything itself
  int nblocks;          // blocks in blk[]
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  // raw buffer (stride 0): an access at or past `bytes` returns 0 / is dropped by the hardware
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ unsigned ld_word(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, (int)byte_off, 0, kSc1);
}
__device__ __forceinline__ u32x4 ld_words4(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, kSc1);
}
// (all NaNs become one, which is not kEmpty)
__device__ __forceinline__ unsigned word_of(float v) { return v == v ? __float_as_uint(v) : 0x7fc00000u; }
__device__ __forceinline__ void st_f32(__amdgpu_buffer_rsrc_t r, unsigned byte_off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(word_of(v), r, (int)byte_off, 0, kSc1);
}
__device__ __forceinline__ void st_f32x2(__amdgpu_buffer_rsrc_t r, unsigned byte_off, float a, float b) {
  __builtin_amdgcn_raw_buffer_store_b64(u32x2{word_of(a), word_of(b)}, r, (int)byte_off, 0, kSc1);
}

// What bounds this wavefront's waits.
struct Waits {
  int* failed;     // a wait has given up (device memory)
  int spin_limit, patience;
  int* left;       // in LDS, set where this wavefront leaves a task because its input did not come
};

// Runs load(), which fetches what this lane needs and says whether any word of it is still empty, until no lane of the wavefront
// misses any; false: they did not come.  A wait that gives up sets the failure word.
template <typename F>
__device__ __forceinline__ bool load_written(Waits& waits, F load) {
  const int most = min(__builtin_amdgcn_readfirstlane(waits.patience), waits.spin_limit);
  int polls = most;
  bool missing;
  do {
    missing = __builtin_amdgcn_ballot_w64(load()) != 0;
    asm volatile("" ::: "memory");
  } while (missing && --polls >= 0);
  if (__builtin_expect(missing, 0)) {
    if (most >= waits.spin_limit) __hip_atomic_store(waits.failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    waits.patience = 0;  // the wavefront's other tasks are left at once
    *waits.left = 1;
  }
  return !missing;
}

// `word` is one of kChainWaves in LDS, a wavefront's own; behind a barrier: whether a wavefront's is `value`.
__device__ __forceinline__ bool any_wave(const int* word, int value) {
  return __builtin_amdgcn_ballot_w64(word[threadIdx.x % kChainWaves] == value) != 0;
}
// Whether a pointwise task's result v stands for a sum of words that have not come: they are empty, which as a value is a NaN.  (Nothing
// is looked up for any other result.)
__device__ __forceinline__ bool not_computed(float v, const int* left, int task) {
  return __builtin_amdgcn_ballot_w64(v != v) != 0 && any_wave(left, task) && v != v;
}

// ---- depthwise 3x3 + bias + ReLU6: 16 output pixels x 32 channels, one output per thread ----
// wait: the input comes from a task of this launch
__device__ __forceinline__ void dw_task(Waits& waits, const ChainBlock<float>& B, int r, int c, bool wait,
                                        __amdgpu_buffer_rsrc_t in, __amdgpu_buffer_rsrc_t act) {
  const int m_out = B.out_hw * B.out_hw;
  const int t = threadIdx.x, px = t / 32, ch = 32 * c + t % 32;
  // filter taps and bias first: they do not depend on anybody
  float w[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) w[k] = B.dw_w[k * B.cin + ch];
  const float bias = B.dw_b[ch];

  const int p = 16 * r + px;
  const bool live = p < m_out;
  const int oy = (int)div_by((unsigned)p, B.by_hw), ox = p - oy * B.out_hw;
  const int iy0 = oy * B.stride - B.pad, ix0 = ox * B.stride - B.pad;
  float v[9];
  unsigned off[9];
  bool ok[9];
#pragma unroll
  for (int kh = 0; kh < 3; ++kh)
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) {
      const int iy = iy0 + kh, ix = ix0 + kw;
      ok[kh * 3 + kw] = live && iy >= 0 && iy < B.in_hw && ix >= 0 && ix < B.in_hw;
      // a tap outside the image reads past the end of the buffer: the hardware returns 0, no branch
      off[kh * 3 + kw] = ok[kh * 3 + kw] ? (B.in_off + (unsigned)((iy * B.in_hw + ix) * B.cin + ch)) * 4u : 0x80000000u;
    }
  const bool have = load_written(waits, [&]() __attribute__((always_inline)) {
    unsigned most = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const unsigned w1 = ld_word(in, off[k]);
      v[k] = __uint_as_float(w1), most = max(most, w1);
    }
    return wait && most == kEmpty;
  });
  float acc = bias;
#pragma unroll
  for (int k = 0; k < 9; ++k) acc = ok[k] ? fmaf(v[k], w[k], acc) : acc;
  ActClamp clamp;
  clamp.on = true;
  clamp.hi = 6.0f;
  if (have && live) st_f32(act, (B.mid_off + (unsigned)(p * B.cin + ch)) * 4u, apply_act(acc, clamp));
}

// The same on halfs: 16 output pixels x 64 channels, two (a word) per thread, sums in fp32 and one rounding.
__device__ __forceinline__ unsigned half_bits(half_t v) { return v == v ? (unsigned)__builtin_bit_cast(unsigned short, v) : 0x7e00u; }
__device__ __forceinline__ unsigned word_of(float a, float b) { return half_bits((half_t)a) | half_bits((half_t)b) << 16; }
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void dw_task(Waits& waits, const ChainBlock<half_t>& B, int r, int c, bool wait,
                                        __amdgpu_buffer_rsrc_t in, __amdgpu_buffer_rsrc_t act) {
  const int m_out = B.out_hw * B.out_hw;
  const int t = threadIdx.x, px = t / 32, ch = 64 * c + 2 * (t % 32);
  unsigned w[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) w[k] = *reinterpret_cast<const unsigned*>(B.dw_w + k * B.cin + ch);
  const unsigned bias = *reinterpret_cast<const unsigned*>(B.dw_b + ch);

  const int p = 16 * r + px;
  const bool live = p < m_out;
  const int oy = (int)div_by((unsigned)p, B.by_hw), ox = p - oy * B.out_hw;
  const int iy0 = oy * B.stride - B.pad, ix0 = ox * B.stride - B.pad;
  unsigned v[9], off[9];
  bool ok[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int iy = iy0 + k / 3, ix = ix0 + k % 3;
    ok[k] = live && iy >= 0 && iy < B.in_hw && ix >= 0 && ix < B.in_hw;
    off[k] = ok[k] ? (B.in_off + (unsigned)((iy * B.in_hw + ix) * B.cin + ch)) * 2u : 0x80000000u;  // (past the end: 0)
  }
  const bool have = load_written(waits, [&]() __attribute__((always_inline)) {
    unsigned most = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) v[k] = ld_word(in, off[k]), most = max(most, v[k]);
    return wait && most == kEmpty;
  });
  const h2 b = __builtin_bit_cast(h2, bias);
  float acc[2] = {(float)b[0], (float)b[1]};
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const h2 x = __builtin_bit_cast(h2, v[k]), f = __builtin_bit_cast(h2, w[k]);
#pragma unroll
    for (int e = 0; e < 2; ++e) acc[e] = ok[k] ? fmaf((float)x[e], (float)f[e], acc[e]) : acc[e];
  }
  ActClamp clamp;
  clamp.on = true;
  clamp.hi = 6.0f;
  if (have && live)
    __builtin_amdgcn_raw_buffer_store_b32(word_of(apply_act(acc[0], clamp), apply_act(acc[1], clamp)), act,
                                          (int)((B.mid_off + (unsigned)(p * B.cin + ch)) * 2u), 0, kSc1);
}

// ---- pointwise 1x1 + bias + ReLU6: 16 x (16 TN) tile, K = WAVES x CHUNK split over the first WAVES 
// wavefronts (all 8 where K is a multiple of 128; 4 for the K = 64 and K = 192 of the narrower networks) ----
template <int CHUNK, int TN, int WAVES>
__device__ __forceinline__ void pw_task(Waits& waits, const ChainBlock<float>& B, int tile_m, int tile_n,
                                        __amdgpu_buffer_rsrc_t act, float* red, int* left, int task) {
  constexpr int G = CHUNK / 16;
  const int K = B.cin, N = B.cout, M = B.out_hw * B.out_hw;
  const int tid = threadIdx.x, wk = tid / 64, lane = tid % 64, li = lane % 16, q = lane / 16;
  const bool compute = tid < 64 * WAVES;
  const int m0 = 16 * tile_m, n0 = 16 * TN * tile_n;

  // filter columns and bias before the wait (ordinary cached loads)
  const float* bp = B.pw_w + (size_t)(wk * CHUNK + 4 * q) * N + n0 + TN * li;
  float b[G][4][TN];
  if (compute) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float* p = bp + (size_t)(16 * g + s) * N;
        if constexpr (TN == 2) {
          const float2 t2 = *reinterpret_cast<const float2*>(p);
          b[g][s][0] = t2.x;
          b[g][s][1] = t2.y;
        } else {
          b[g][s][0] = *p;
        }
      }
  }
  // epilogue thread e < 256 owns register v = e / 64 of lane l = e % 64: row 4 (l / 16) + v, columns TN (l % 16) ...
  const int ev = tid / 64, el = tid % 64;
  const int erow = m0 + 4 * (el / 16) + ev, ecol = n0 + TN * (el % 16);
  float ebias[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) ebias[j] = tid < 256 ? B.pw_b[ecol + j] : 0.f;

  if (compute) {
    const int arow = min(m0 + li, M - 1);  // rows past M repeat the last one (they feed outputs that are not stored)
    const unsigned a_off = (B.mid_off + (unsigned)(arow * K + wk * CHUNK + 4 * q)) * 4u;
    u32x4 a[G];
    {  // a word of each depthwise task first: eight wavefronts' whole operands, asked for again and again, keep the memory busy
      const unsigned last = (B.mid_off + (unsigned)(min(m0 + 15, M - 1) * K + wk * CHUNK + 32 * (li % ((CHUNK + 31) / 32)))) * 4u;
      (void)load_written(waits, [&]() __attribute__((always_inline)) { return ld_word(act, last) == kEmpty; });
    }
    const bool have = load_written(waits, [&]() __attribute__((always_inline)) {
      unsigned most = 0;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        a[g] = ld_words4(act, a_off + 64u * g);
        most = max(max(max(a[g][0], a[g][1]), max(a[g][2], a[g][3])), most);
      }
      return most == kEmpty;
    });
    if (!have) left[wk] = task;

    floatx4 acc[2][TN];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[c][j][v] = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[s & 1][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[g][s]), b[g][s][j], acc[s & 1][j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[((wk * TN + j) * 4 + v) * 64 + lane] = acc[0][j][v] + acc[1][j][v];
  }
  __syncthreads();
  if (tid < 256) {
    ActClamp clamp;
    clamp.on = true;
    clamp.hi = 6.0f;
    float o[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float sum = ebias[j];
#pragma unroll
      for (int w = 0; w < WAVES; ++w) sum += red[((w * TN + j) * 4 + ev) * 64 + el];
      o[j] = apply_act(sum, clamp);
    }
    if (not_computed(o[0], left, task) || erow >= M) return;
    const unsigned off = (B.out_off + (unsigned)(erow * N + ecol)) * 4u;
    if constexpr (TN == 2) st_f32x2(act, off, o[0], o[1]);
    else st_f32(act, off, o[0]);
  }
}

// The same on halfs, 32 values of K an instruction.  A filter value is one of a lane's eight of consecutive rows: words of two columns
// (single halfs with TN == 1) come from eight rows and are put together in registers.
template <int CHUNK, int TN, int WAVES>
__device__ __forceinline__ void pw_task(Waits& waits, const ChainBlock<half_t>& B, int tile_m, int tile_n,
                                        __amdgpu_buffer_rsrc_t act, float* red, int* left, int task) {
  constexpr int G = CHUNK / 32;
  const int K = B.cin, N = B.cout, M = B.out_hw * B.out_hw;
  const int tid = threadIdx.x, wk = tid / 64, lane = tid % 64, li = lane % 16, q = lane / 16;
  const bool compute = tid < 64 * WAVES;
  const int m0 = 16 * tile_m, n0 = 16 * TN * tile_n;

  const half_t* bp = B.pw_w + (size_t)(wk * CHUNK + 8 * q) * N + n0 + TN * li;
  unsigned raw[G][8];
  if (compute) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const half_t* p = bp + (size_t)(32 * g + s) * N;
        if constexpr (TN == 2) raw[g][s] = *reinterpret_cast<const unsigned*>(p);
        else raw[g][s] = *reinterpret_cast<const unsigned short*>(p);
      }
  }
  const int ev = tid / 64, el = tid % 64;
  const int erow = m0 + 4 * (el / 16) + ev, ecol = n0 + TN * (el % 16);
  float ebias[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) ebias[j] = tid < 256 ? (float)B.pw_b[ecol + j] : 0.f;

  if (compute) {
    const int arow = min(m0 + li, M - 1);
    const unsigned a_off = (B.mid_off + (unsigned)(arow * K + wk * CHUNK + 8 * q)) * 2u;
    u32x4 a[G];
    {  // (a word of each depthwise task first, as above)
      const unsigned last = (B.mid_off + (unsigned)(min(m0 + 15, M - 1) * K + wk * CHUNK + 32 * (li % G))) * 2u;
      (void)load_written(waits, [&]() __attribute__((always_inline)) { return ld_word(act, last) == kEmpty; });
    }
    const bool have = load_written(waits, [&]() __attribute__((always_inline)) {
      unsigned most = 0;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        a[g] = ld_words4(act, a_off + 64u * g);
        most = max(max(max(a[g][0], a[g][1]), max(a[g][2], a[g][3])), most);
      }
      return most == kEmpty;
    });
    if (!have) left[wk] = task;

    floatx4 acc[2][TN] = {};
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        u32x4 b;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          b[i] = __builtin_amdgcn_perm(raw[g][2 * i + 1], raw[g][2 * i], j == 0 ? 0x05040100u : 0x07060302u);
        acc[g & 1][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a[g]), __builtin_bit_cast(h8, b), acc[g & 1][j], 0, 0, 0);
      }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[((wk * TN + j) * 4 + v) * 64 + lane] = acc[0][j][v] + acc[1][j][v];
  }
  __syncthreads();
  if (tid < 256) {
    ActClamp clamp;
    clamp.on = true;
    clamp.hi = 6.0f;
    float o[2];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float sum = ebias[j];
#pragma unroll
      for (int w = 0; w < WAVES; ++w) sum += red[((w * TN + j) * 4 + ev) * 64 + el];
      o[j] = apply_act(sum, clamp);
    }
    // (TN == 1: the next lane's column, for the even ones; a word is written whole)
    if constexpr (TN == 1) o[1] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(o[0]), 0xb1, 0xf, 0xf, true));
    if (!not_computed(o[0], left, task) && erow < M && (TN == 2 || el % 2 == 0))
      __builtin_amdgcn_raw_buffer_store_b32(word_of(o[0], o[1]), act, (int)((B.out_off + (unsigned)(erow * N + ecol)) * 2u), 0, kSc1);
  }
}

__device__ __forceinline__ float block_sum_or_max(float v, bool is_max, float* scratch) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float o = __shfl_xor(v, off, 64);
    v = is_max ? fmaxf(v, o) : v + o;
  }
  __syncthreads();
  if (threadIdx.x % 64 == 0) scratch[threadIdx.x / 64] = v;
  __syncthreads();
  float r = scratch[0];
#pragma unroll
  for (int i = 1; i < kChainWaves; ++i) r = is_max ? fmaxf(r, scratch[i]) : r + scratch[i];
  return r;
}

// The pointwise task for a layer of K input channels: the K split, and 32-column tiles only below K = 1024.
template <typename T, int K>
__device__ __forceinline__ void pw_task_for(Waits& waits, const ChainBlock<T>& B, int r, int c,
                                            __amdgpu_buffer_rsrc_t act, float* red, int* left, int task) {
  constexpr int STEP = sizeof(T) == 2 ? 32 : 16;  // a wavefront takes whole steps
  constexpr int WAVES = K % (8 * STEP) == 0 ? 8 : sizeof(T) == 2 && K % (6 * STEP) == 0 ? 6 : K % (4 * STEP) == 0 ? 4 : 2;
  constexpr int CHUNK = K / WAVES;
  static_assert(CHUNK % STEP == 0 && CHUNK <= 128, "a wavefront takes whole steps of K");
  if constexpr (K < 1024) {
    if (B.tn == 2) return pw_task<CHUNK, 2, WAVES>(waits, B, r, c, act, red, left, task);
  }
  pw_task<CHUNK, 1, WAVES>(waits, B, r, c, act, red, left, task);
}

// Four weights of the fully connected layer as they are stored.
template <typename T>
struct FcWeights;
template <>
struct FcWeights<float> {
  typedef float4 V;
  static __device__ __forceinline__ float get(const V& v, int e) { return (&v.x)[e]; }
};
template <>
struct FcWeights<half_t> {
  typedef _Float16 V __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ float get(const V& v, int e) { return (float)v[e]; }
};

// Q = width multiplier in quarters: the chained blocks have 64 Q, 128 Q and 256 Q input channels, the fully
// connected layer 256 Q = 2 Q slices of 128.
template <typename T, int Q>
__global__ __launch_bounds__(kChainThreads) void mobilenet_chain_kernel(const ChainParams<T> P) {
  constexpr int kSlices = 2 * Q;
  constexpr bool kHalf = sizeof(T) == 2;
  // 2 x 16 KB: split-K partial tiles, of one task and the next (between a task's reads and the writes of the task after the next lies
  // the barrier of the next); reused by the tail
  __shared__ float red2[2][kChainWaves * 2 * 4 * 64];
  // Each wavefront's own: whether it has left a task of the steps, of the last one, and by turn the number of a pointwise task that it left.
  __shared__ int left[4][kChainWaves];
  const int wg = blockIdx.x, tid = threadIdx.x;
  if (tid % 64 < 4) left[tid % 64][tid / 64] = 0;
  Waits waits{P.failed, P.spin_limit, P.patience, &left[0][tid / 64]};
  {
    // The block descriptors are read at every block change, on the critical path, and the first touch of a line of
    // the kernel argument segment misses the scalar cache: touch every line now.
    typedef __attribute__((address_space(4))) const int* KernargInts;
    KernargInts karg = (KernargInts)__builtin_amdgcn_kernarg_segment_ptr();
    int warm = 0;
#pragma unroll
    for (int i = 0; i < (int)sizeof(ChainParams<T>) / 4; i += 16) warm += karg[i];
    asm volatile("" ::"s"(warm));
  }
  const __amdgpu_buffer_rsrc_t in0 = make_rsrc(P.in0, P.in0_bytes);
  const __amdgpu_buffer_rsrc_t act = make_rsrc(P.act, P.act_bytes);

  // this workgroup's slice of the fully connected weights (128 input channels x 128 classes, 32 values per
  // thread), fetched now: nothing in the kernel depends on it for the next 50 us
  const int fc_tasks_c = (P.classes + kFcColBlock - 1) / kFcColBlock;
  const int fc_tasks = kSlices * fc_tasks_c;
  constexpr int kper = 128;  // input channels per task, 8 per thread
  typedef typename FcWeights<T>::V Weights;
  Weights fw[8] = {};
  const bool fvec = P.classes % 4 == 0;
  auto load_fc = [&](int task, Weights (&dst)[8]) {
    const int ks = task / fc_tasks_c, cb = task % fc_tasks_c;
    const int col = kFcColBlock * cb + 4 * (tid % 32), k0 = kper * ks + 8 * (tid / 32);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const T* p = P.fc_w + (size_t)(k0 + i) * P.classes + col;
      if (fvec && col + 3 < P.classes) {
        dst[i] = *reinterpret_cast<const Weights*>(p);
      } else {
        dst[i] = Weights{col < P.classes ? p[0] : (T)0.f, col + 1 < P.classes ? p[1] : (T)0.f, col + 2 < P.classes ? p[2] : (T)0.f,
                         col + 3 < P.classes ? p[3] : (T)0.f};
      }
    }
  };
  if (wg < fc_tasks) load_fc(wg, fw);
  // tasks first, first + stride, ... of every step
  int count = 0;
  auto steps = [&](int first, int stride) __attribute__((always_inline)) {
    for (int bi = 0; bi < P.nblocks; ++bi) {
      const ChainBlock<T>& B = P.blk[bi];
      const TaskMap &dw_map = B.dw_map, &pw_map = B.pw_map;
      for (int vt = first; vt < dw_map.count; vt += stride) {
        int r, c;
        if (task_of(dw_map, vt, &r, &c)) dw_task(waits, B, r, c, bi > 0, bi == 0 ? in0 : act, act);
      }
      for (int vt = first; vt < pw_map.count; vt += stride) {
        int r, c;
        if (!task_of(pw_map, vt, &r, &c)) continue;
        ++count;
        const int turn = count % 2;
        float* const red = red2[turn];
        if (B.cin == 64 * Q) pw_task_for<T, 64 * Q>(waits, B, r, c, act, red, left[2 + turn], count);
        else if (B.cin == 128 * Q) pw_task_for<T, 128 * Q>(waits, B, r, c, act, red, left[2 + turn], count);
        else pw_task_for<T, 256 * Q>(waits, B, r, c, act, red, left[2 + turn], count);
      }
    }
  };

  // ---- average pool + fully connected: task (ks, cb) = 128 input channels x 128 classes ----
  const ChainBlock<T>& L = P.blk[P.nblocks - 1];
  const int hw2 = P.last_hw * P.last_hw;
  float* const red = red2[0];
  // own: after its own steps, of which a wavefront may have left one; false: then, or where the last step's words do not come
  auto fully_connected = [&](bool own) __attribute__((always_inline)) {
    waits.left = &left[1][tid / 64];
    __syncthreads();
    if (own && any_wave(left[0], 1)) return false;
    if (wg < fc_tasks) {
      const int ks = wg / fc_tasks_c, cb = wg % fc_tasks_c;
      float* pooled = red;             // [128]
      float* psum = red + 128;         // [4][128], halfs: [8][128]
      float* fsum = red + 128 + 1024;  // [16][128]
      constexpr int PG = kHalf ? 8 : 4, PX = 64 / PG, WORDS = kChainThreads / PG;
      {
        // thread (pixel group pg of PG, word of WORDS: a channel, halfs: two) sums pixels pg, pg + PG, ... (at most 64 pixels)
        const int word = tid % WORDS, pg = tid / WORDS, chn = (kHalf ? 2 : 1) * word;
        unsigned x[PX];
        (void)load_written(waits, [&]() __attribute__((always_inline)) {
          unsigned most = 0;
#pragma unroll
          for (int i = 0; i < PX; ++i) {
            const int p = pg + PG * i;
            x[i] = ld_word(act, p < hw2 ? (L.out_off + (unsigned)(p * P.feat + kper * ks + chn)) * (unsigned)sizeof(T) : 0x80000000u);
            most = max(most, x[i]);
          }
          return most == kEmpty;
        });
        float s[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < PX; ++i) {
          if constexpr (kHalf) {
            const h2 v = __builtin_bit_cast(h2, x[i]);
            s[0] += (float)v[0], s[1] += (float)v[1];
          } else {
            s[0] += __uint_as_float(x[i]);
          }
        }
        psum[pg * 128 + chn] = s[0];
        if constexpr (kHalf) psum[pg * 128 + chn + 1] = s[1];
      }
      __syncthreads();
      if (tid < 128) {
        float s = psum[tid];
#pragma unroll
        for (int i = 1; i < PG; ++i) s += psum[128 * i + tid];
        pooled[tid] = (float)(T)(s / (float)hw2);  // (the pooled vector is a tensor of the storage type)
      }
      __syncthreads();
      {
        const int kq = tid / 32, c4 = tid % 32;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float pv = pooled[8 * kq + i];
          s.x = fmaf(pv, FcWeights<T>::get(fw[i], 0), s.x);
          s.y = fmaf(pv, FcWeights<T>::get(fw[i], 1), s.y);
          s.z = fmaf(pv, FcWeights<T>::get(fw[i], 2), s.z);
          s.w = fmaf(pv, FcWeights<T>::get(fw[i], 3), s.w);
        }
        *reinterpret_cast<float4*>(fsum + kq * 128 + 4 * c4) = s;
      }
      __syncthreads();
      const bool some_left = own && any_wave(left[1], 1);
      if (tid < kFcColBlock) {
        float s = 0.f;
#pragma unroll
        for (int g = 0; g < 16; ++g) s += fsum[g * 128 + tid];
        const int col = kFcColBlock * cb + tid;
        if (col < P.classes && !some_left) st_f32(act, P.partial_at + (unsigned)(ks * P.classes + col) * 4u, s);
      }
      __syncthreads();
      if (some_left) return false;
    }
    return true;
  };

  steps(wg, kChainGrid);
  if (!fully_connected(true)) {  // an input did not come: every task
    waits.patience = 0x7fffffff;
    steps(0, 1);
    if (wg < fc_tasks) load_fc(wg, fw);
    (void)fully_connected(false);
  }

  // ---- bias + softmax: one task, two classes per thread ----
  if (wg == 0) {
    waits.patience = 0x7fffffff;  // (what it waits for is left to nobody: its workgroups end without it)
    float l[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = tid + kChainThreads * h;
      const bool in = j < P.classes;
      float part[kSlices];
      (void)load_written(waits, [&]() __attribute__((always_inline)) {
        unsigned most = 0;
#pragma unroll
        for (int s = 0; s < kSlices; ++s) {
          const unsigned word = ld_word(act, in ? P.partial_at + (unsigned)(s * P.classes + j) * 4u : 0x80000000u);
          part[s] = __uint_as_float(word), most = max(most, word);
        }
        return most == kEmpty;
      });
      float v = in ? (float)P.fc_b[j] : 0.f;
#pragma unroll
      for (int s = 0; s < kSlices; ++s) v += part[s];
      l[h] = in ? (float)(T)v : -INFINITY;  // (halfs: the softmax is taken of the stored logits)
    }
    const bool failed = __hip_atomic_load(P.failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    const float mx = block_sum_or_max(fmaxf(l[0], l[1]), true, red);
    float e[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) e[h] = tid + kChainThreads * h < P.classes ? __expf(l[h] - mx) : 0.f;
    const float sum = block_sum_or_max(e[0] + e[1], false, red + 16);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = tid + kChainThreads * h;
      if (j < P.classes) {
        const float nan = __uint_as_float(0x7fc00000u);
        if (P.logits) P.logits[j] = (T)(failed ? nan : l[h]);
        P.probs[j] = (T)(failed ? nan : e[h] / sum);
      }
    }
  }
}

}  // namespace

bool chain_supported(int image_size, int width_quarters, int classes, long long batch) {
  // the 1/8-size map of 64 q channels is what the first chained block reads; channel counts 64 q / 128 q / 256 q
  return batch == 1 && width_quarters >= 1 && width_quarters <= 4 && image_size >= 32 && image_size <= 256 &&
         classes >= 1 && classes <= 1024;
}

namespace {
template <typename T>
using ChainKernel = void (*)(const ChainParams<T>);
template <typename T>
ChainKernel<T> chain_kernel(int width_quarters) {
  switch (width_quarters) {
    case 1: return mobilenet_chain_kernel<T, 1>;
    case 2: return mobilenet_chain_kernel<T, 2>;
    case 3: return mobilenet_chain_kernel<T, 3>;
    default: return mobilenet_chain_kernel<T, 4>;
  }
}
}  // namespace

// How many grids of the chain kernel are resident at once on the current device, at most 2 (looked up once per device).
int chain_grids(int width_quarters, bool half) {
  static std::atomic<int> states[8][64];  // 0 unknown, else one more than the grids
  int dev = 0;
  if (width_quarters < 1 || width_quarters > 4 || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  std::atomic<int>* const state = states[width_quarters - 1 + (half ? 4 : 0)];
  const int s = state[dev].load(std::memory_order_acquire);
  if (s) return s - 1;
  int cus = 0, per_cu = 0;
  const void* const kernel = half ? reinterpret_cast<const void*>(chain_kernel<half_t>(width_quarters)) : reinterpret_cast<const void*>(chain_kernel<float>(width_quarters));
  const bool ok = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                  hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kChainThreads, 0) == hipSuccess;
  const int grids = !ok ? 0 : (int)std::min(2ll, (long long)cus * per_cu / kChainGrid);
  state[dev].store(1 + grids, std::memory_order_release);
  return grids;
}

namespace {
constexpr int kNetChannels[13] = {64, 128, 128, 256, 256, 512, 512, 512, 512, 512, 512, 1024, 1024};
constexpr int kNetStrides[13] = {1, 2, 1, 2, 1, 2, 1, 1, 1, 1, 1, 2, 1};

// Bytes of the chained part for an input map of in_hw x in_hw x 64 q (the output of block 4) at width q / 4.
template <typename T>
size_t chain_layout(int in_hw, int classes, int q, ChainParams<T>* P, int first) {
  constexpr int kTaskChannels = 128 / (int)sizeof(T);  // of a depthwise task
  size_t off = 0;
  const int nblocks = 13 - first;
  int hw = in_hw, cin = kNetChannels[first - 1] * q / 4;
  size_t prev_out = 0;
  for (int bi = 0; bi < nblocks; ++bi) {
    const int net = first + bi, s = kNetStrides[net], cout = kNetChannels[net] * q / 4;
    const int out_hw = (hw + s - 1) / s;
    const int need = (out_hw - 1) * s + 3 - hw;
    const int pad = need > 0 ? need / 2 : 0;
    const int m = out_hw * out_hw, tiles_m = (m + 15) / 16;
    // 32-column tiles where 16-column ones take more rounds of tasks (never for K = 1024: 32 values of K per lane)
    auto rounds = [&](int columns) { return (make_task_map(tiles_m, cout / columns).count + kChainGrid - 1) / kChainGrid; };
    const int tn = cin < 1024 && rounds(16) > rounds(32) ? 2 : 1;
    if (P) {
      ChainBlock<T>& B = P->blk[bi];
      B.in_hw = hw, B.out_hw = out_hw, B.stride = s, B.pad = pad, B.cin = cin, B.cout = cout, B.tn = tn;
      B.by_hw = fast_div((unsigned)out_hw);
      B.dw_map = make_task_map(tiles_m, cin / kTaskChannels), B.pw_map = make_task_map(tiles_m, cout / (16 * tn));
      B.in_off = (unsigned)prev_out;
      B.mid_off = (unsigned)off;
      B.out_off = (unsigned)(off + (size_t)m * cin);
    }
    prev_out = off + (size_t)m * cin;
    off += (size_t)m * cin + (size_t)m * cout;
    hw = out_hw, cin = cout;
  }
  const int slices = cin / kFcSliceChannels;
  if (P) {
    P->partial_at = (unsigned)(off * sizeof(T));
    P->last_hw = hw;
    P->feat = cin;
    P->classes = classes;
    P->nblocks = nblocks;
  }
  return off * sizeof(T) + (size_t)slices * classes * sizeof(float);
}
}  // namespace

// The chain's memory: flag words -- the failure word, then those of the launch that runs blocks 2 - 4 as stages (block.hip) --, then
// every step's output.
namespace {
size_t flag_region(int image_size) {
  const int half = (image_size + 1) / 2;
  return (size_t)(1 + block_chain_flag_words(half, half)) * block_chain_flag_stride() * sizeof(int);
}
int eighth_of(int image_size) {
  const int half = (image_size + 1) / 2, quarter = (half + 1) / 2;
  return (quarter + 1) / 2;
}
}  // namespace
ChainFill chain_fill(int image_size, int classes, int width_quarters, int first_block, void* chain_ws) {
  return ChainFill{static_cast<char*>(chain_ws) + flag_region(image_size),
                   (chain_layout<float>(eighth_of(image_size), classes, width_quarters, nullptr, first_block) + 255) / 256 * 256};
}
ChainFill chain_fill_f16(int image_size, int classes, int width_quarters, int first_block, void* chain_ws) {
  return ChainFill{static_cast<char*>(chain_ws) + 256,  // (the failure word)
                   (chain_layout<half_t>(eighth_of(image_size), classes, width_quarters, nullptr, first_block) + 255) / 256 * 256};
}
// (laid out for the longer chain; a launch that starts one block later uses a part of it)
size_t chain_workspace_bytes(int image_size, int classes, int width_quarters) {
  return flag_region(image_size) + chain_fill(image_size, classes, width_quarters, kFirstChainBlock, nullptr).bytes;
}
size_t chain_workspace_bytes_f16(int image_size, int classes, int width_quarters) {
  return 256 + chain_fill_f16(image_size, classes, width_quarters, kFirstChainBlock, nullptr).bytes;
}
int chain_flag_words(int image_size) {
  const int half = (image_size + 1) / 2;
  return 1 + block_chain_flag_words(half, half);
}
int chain_spin_limit() {
  // Test hook: TFX_CHAIN_SPIN_LIMIT=<n> makes every wait give up after n polls, which exercises the failure
  // path (all outputs NaN, the kernels still run to their end) without any workgroup actually missing.
  if (const char* e = getenv("TFX_CHAIN_SPIN_LIMIT")) {
    const long v = strtol(e, nullptr, 10);
    if (v >= 1 && v <= kSpinLimit) return (int)v;
  }
  return kSpinLimit;
}

int chain_workgroups() {
  // Test hook: TFX_CHAIN_WORKGROUPS=<n> leaves out the workgroups from the nth on (those of the fully connected layer are the first
  // 64), as if they never got to run.
  if (const char* e = getenv("TFX_CHAIN_WORKGROUPS")) {
    const long v = strtol(e, nullptr, 10);
    if (v >= kFcTasks && v <= kChainGrid) return (int)v;
  }
  return kChainGrid;
}

namespace {
// Kernels of waiting workgroups of one process are ordered across streams such that all that run are resident, on two tracks per
// device: the kernels of one track never overlap.  One of which two grids are resident at once takes one track -- that of its stream if
// there is one, else the two in turn --, any other one both.  For each track the last stream is remembered; a launch on
// another stream first records an event behind everything queued on that stream and makes the new stream wait for it.  Launches that
// stay on one stream, and of the former kind those of two streams, pay nothing.  One binary16 image, us each on 1, 2 and 4 streams: full width
// 224 x 224 62.8, 38.8, 51, with one track 62.7, 51.1, 58.6, as launches that do not wait 68.7, 53, 53; quarter width 128 x 128 44, 25, 48;
// 43.7, 47, 46.5; 56, 56, 54.  (With more than two streams some share a hardware queue, in which a wait holds up both.)
// A stream that is being captured into a graph is left alone: an event of another stream cannot be recorded into the capture.  Replays of
// such passes, full width 224 x 224: 67.6, 39.9, 40, as launches 73.3, 42.8, 40.  (Those of the fp32 pass at full width, whose launch of blocks
// 2 - 4 has workgroups that do need each other to run, are the caller's to order.)
struct ChainOrder {
  std::mutex lock;
  hipStream_t last[64][2];
  hipEvent_t event[64];
  bool launched[64][2], have_event[64];
  int turn[64];
};
ChainOrder g_order;

void order_after_other_streams(int dev, hipStream_t stream, bool one_track) {
  hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &capturing) != hipSuccess || capturing != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return;
  }
  bool* const launched = g_order.launched[dev];
  hipStream_t* const last = g_order.last[dev];
  int first = 0, end = 2;
  if (one_track) {
    for (first = 0; first < 2 && !(launched[first] && last[first] == stream);) ++first;
    if (first == 2) first = g_order.turn[dev] ^= 1;
    end = first + 1;
  }
  for (int i = first; i < end; ++i) {
    if (launched[i] && last[i] != stream) {
      if (!g_order.have_event[dev])
        g_order.have_event[dev] = hipEventCreateWithFlags(&g_order.event[dev], hipEventDisableTiming) == hipSuccess;
      // a stream that has been destroyed since is refused by the runtime: nothing of it can still be running
      if (g_order.have_event[dev] && hipEventRecord(g_order.event[dev], last[i]) == hipSuccess)
        (void)hipStreamWaitEvent(stream, g_order.event[dev], 0);
      (void)hipGetLastError();
    }
    last[i] = stream;
    launched[i] = true;
  }
}
}  // namespace

// Runs fn(arg) -- which enqueues a kernel whose workgroups wait for each other -- once `stream` has been ordered behind
// the last such kernels of other streams.
int launch_ordered(hipStream_t stream, int (*fn)(void*), void* arg) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return TFX_ERR_LAUNCH;
  std::lock_guard<std::mutex> guard(g_order.lock);
  order_after_other_streams(dev, stream, false);
  return fn(arg);
}

namespace {
template <typename T, typename W>
int launch_chain_of(const T* in0, int image_size, const W* w, void* chain_ws, const ChainFill& fill, T* probs, T* logits, int classes,
                    int width_quarters, hipStream_t stream, int (*before)(void*), void* before_arg, int first_block) {
  if (first_block != kFirstChainBlock && first_block != kFirstChainBlock + 1) return TFX_ERR_ARG;
  if (width_quarters < 1 || width_quarters > 4) return TFX_ERR_ARG;
  ChainParams<T> P{};
  const int in_hw = eighth_of(image_size);
  const size_t used = chain_layout<T>(in_hw, classes, width_quarters, &P, first_block);
  auto t = [](const auto* p) { return reinterpret_cast<const T*>(p); };
  for (int bi = 0; bi < P.nblocks; ++bi) {
    const int net = first_block + bi;
    P.blk[bi].dw_w = t(w->dw_w[net]);
    P.blk[bi].dw_b = t(w->dw_b[net]);
    P.blk[bi].pw_w = t(w->pw_w[net]);
    P.blk[bi].pw_b = t(w->pw_b[net]);
  }
  P.in0 = in0;
  P.in0_bytes = (unsigned)((size_t)in_hw * in_hw * (kNetChannels[first_block - 1] * width_quarters / 4) * sizeof(T));
  P.failed = static_cast<int*>(chain_ws);
  P.act = fill.at;
  P.act_bytes = (unsigned)used;
  P.fc_w = t(w->fc_w);
  P.fc_b = t(w->fc_b);
  P.probs = probs;
  P.logits = logits;
  P.spin_limit = chain_spin_limit();
  P.patience = kPatience;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return TFX_ERR_LAUNCH;
  std::lock_guard<std::mutex> guard(g_order.lock);
  order_after_other_streams(dev, stream, before == nullptr && chain_grids(width_quarters, sizeof(T) == 2) >= 2);
  // a launch of waiting workgroups that belongs in front of this one (blocks 2 - 4 as stages, block.hip) is enqueued
  // under the same lock, so that the pair is ordered against other streams' pairs as one
  if (before != nullptr) {
    const int rc = before(before_arg);
    if (rc != TFX_OK) return rc;
  }
  hipLaunchKernelGGL(chain_kernel<T>(width_quarters), dim3(chain_workgroups()), dim3(kChainThreads), 0, stream, P);
  return check_launch();
}
}  // namespace

int launch_chain(const float* in0, int image_size, const tfx_mobilenet_v1_weights* w, void* chain_ws, float* probs, float* logits,
                 int classes, int width_quarters, hipStream_t stream, int (*before)(void*), void* before_arg, int first_block) {
  return launch_chain_of<float>(in0, image_size, w, chain_ws, chain_fill(image_size, classes, width_quarters, first_block, chain_ws),
                                probs, logits, classes, width_quarters, stream, before, before_arg, first_block);
}

int launch_chain_f16(const uint16_t* in0, int image_size, const tfx_mobilenet_v1_weights_f16* w, void* chain_ws, uint16_t* probs,
                     uint16_t* logits, int classes, int width_quarters, int first_block, hipStream_t stream) {
  return launch_chain_of<half_t>(reinterpret_cast<const half_t*>(in0), image_size, w, chain_ws,
                                 chain_fill_f16(image_size, classes, width_quarters, first_block, chain_ws),
                                 reinterpret_cast<half_t*>(probs), reinterpret_cast<half_t*>(logits), classes, width_quarters, stream,
                                 nullptr, nullptr, first_block);
}

}  // namespace tfx
