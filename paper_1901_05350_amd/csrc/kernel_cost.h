#ifndef TFX_KERNEL_COST_H_
#define TFX_KERNEL_COST_H_

namespace tfx {

// Which kernel: the one that a model of their times says is fastest.  A kernel of bm x bn tiles gives
// c = batch x tiles / 256 of them to a CU (a whole number of rounds while there are few), each of which walks through k:
//   us = fixed + per_k k + c (per_tile + per_tile_k k)
// per_k is the memory round trips of a chain that nothing hides, per_tile_k what k costs the CU.  Fitted to the measured
// times of 226 products and 190 convolutions of either storage type (sizes 16 ... 4096, channels 3 ... 512; mean error
// 4 - 18 %); over these its choice costs 2 - 4 % on average against the fastest kernel of each.
//
// Those sizes are bound by their contraction.  For fp32 products of k < 128, which their output bounds, gemm.hip has
// constants of its own (and the two functions below), fitted to 1000 products of k = 1 ... 127 (2^12 ... 2^26 outputs, batch
// 1 ... 2000, every layout; rms error 6 - 11 % near the choice): there the choice costs 1.8 % on average against the fastest
// kernel, more than 10 % for one product in 14 and at most 28 %; with the constants of long contractions it cost 24 % on
// average and up to 5.2 times.  What makes the difference is that a kernel whose wavefronts split k does not get faster
// below a step for each of them (16 x 2048 x 2048 x 16: 32 x 32 tiles 202 us, 128 x 128 80, gemm_thin.hip 58).
//
// `resident`: the tiled kernels keep 2 (128 x 128) or 4 (64 x 64) tiles on a CU at once, which hide each other's waits.
// The c of a round then grows slowly from its first tile, and the first tile of the next round costs a whole one: of
// 128 x 128 tiles 256 take 1, 308 1.4, 400 1.8, 512 2.3, and 560 as much as 700, 3.65 (measured on 110 products and 57
// convolutions of 100 - 4000 tiles; with the plain count 1947 x 2200 x 3862 went to 64 x 64 tiles for 351 us, now 233).
struct KernelCost {
  int bm, bn;
  double fixed, per_k, per_tile, per_tile_k;
  int resident = 0;
  double us(long long batch, long long m, long long n, double k) const {
    const double tiles = (double)(batch * ((m + bm - 1) / bm) * ((n + bn - 1) / bn)) / 256.;
    double c = tiles <= 2. ? (tiles <= 1. ? 1. : 2.) : tiles + .5;
    if (resident != 0) {
      const bool two = resident == 2;
      const double rounds = (double)(long long)(tiles / resident), rest = tiles - rounds * resident;
      c = rounds * (two ? 2.45 : 4.8);
      if (rest > 0.) c += (rest <= 1. ? 1. : 1. + (two ? 1.3 : .87) * (rest - 1.)) + (rounds == 0. ? 0. : two ? .2 : .6);
    }
    return fixed + per_k * k + c * (per_tile + per_tile_k * k);
  }
};

// us = fixed + per_k k + c (per_tile + per_tile_k k) + per_output x 1e6 outputs, where c is 1 up to a tile for each of the 256 CUs
// and then grows by `share` for a further tile of a CU, of which `round` counts as soon as any CU has it; `odd` operands cost the
// loads `per_odd` of their share each.
struct PipeCost {
  int bm, bn;
  double fixed, per_tile, per_tile_k, round, share, per_odd, per_output, per_k = 0.;
  double us(long long batch, long long m, long long n, int k, int odd) const {
    const double tiles = (double)(batch * ((m + bm - 1) / bm) * ((n + bn - 1) / bn)) / 256., up = (double)(long long)(tiles + .999999);
    const double c = tiles <= 1. ? 1. : 1. + share * (round * up + (1. - round) * tiles - 1.);
    return fixed + per_k * k + c * (per_tile + per_tile_k * k * (1. + per_odd * odd)) + per_output * 1e-6 * (double)(batch * m * n);
  }
};

// gemm_deep.hip: two column blocks per workgroup once single ones are more than one for each CU, where a few CUs would have
// two and the rest wait (halfs: 137 x 1376 x 520, 297 or 153 workgroups, 8.9 and 6.0 us; 376 x 3504 x 168 15.2 and 9.1); a
// few more of those of 4 wavefronts, up to 8 k-steps, run side by side (floats, 128 x 120 x 600, 304 or 152: 3.1 and 3.3).
inline bool deep_two_columns(long long rows, long long n, int steps) {
  return n % 2 == 0 && n > 16 && rows * ((n + 15) / 16) > (steps <= 8 ? 320 : 256);
}

// gemm_deep.hip on floats, k < 128.
inline double shallow_deep_us(long long batch, long long m, long long n, int k) {
  const long long rows = batch * ((m + 15) / 16), wide = rows * ((n + 31) / 32);
  const bool two = deep_two_columns(rows, n, (k + 15) / 16);
  const double c = (double)(two ? wide : rows * ((n + 15) / 16)) / 256.;
  return 3.09 + .0025 * k + (c > 1. ? c : 1.) * (two ? .299 + .0029 * k : .208 + .0017 * k);
}

// gemm_thin.hip on floats, k <= 32: B into registers once per wavefront (4096 of them at a time), then the speed of
// writing C, whose rows of no multiple of 4 elements are written in pieces of lines; with two k-steps a wavefront of few
// tiles shows more of its loads' latency.
inline double thin_us(long long batch, long long m, long long n, int k) {
  const int tn = n <= 32 ? 1 : 2, steps = k <= 16 ? 1 : 2;
  const double chains = (double)(batch * ((n + 32 * tn - 1) / (32 * tn))), tiles = (double)((m + 31) / 32);
  const double waves = chains >= 4096. ? 1. : 4096. / chains, per_wave = tiles > waves ? tiles / waves : 1.;
  const double outputs = 1e-6 * (double)(batch * m * n), padded = 1e-6 * chains * tiles * 1024. * tn;
  return 2.8 + .45 * tn * steps * (chains > 4096. ? chains / 4096. : 1.) +
         outputs * (.375 + (n % 4 != 0 ? .166 * steps : 0.)) + padded * (steps == 1 ? .53 : .58 + .33 / per_wave);
}

// Whether gemm_thin.hip is the fastest for a 1x1 convolution with a stride (floats) or a product of one batch with A stored
// [M,K] (halfs): from how many outputs on its start is paid back.  Measured on 1x1 convolutions of 100 ... 250 000 rows:
// floats, 8 -> 16 channels, 200704 rows 25 -> 8 us; 40 -> 152, 248292 rows 145 -> 80; 48 -> 24, 1700 rows 3.5 -> 5.3 (not
// taken); 48 -> 128, 200000 rows 46 us with 128 x 128 tiles, 61 here; halfs, 11 -> 22, 207936 rows 33 -> 7.  With many
// columns a wavefront has few rows for the B that it loads: halfs, 4096 x 4096 outputs, k = 32 / 64 / 128: 16 / 20 / 28
// us here, 13.6 / 13.8 / 15.8 with tiles (2048 x 2048 x 32: 6.5 and 7.4); 64 columns from k = 48 on likewise (100000 rows,
// B stored [N,K]: 10.9 and 8.9; 128 columns 22.5 and 25.9).
inline bool thin_pays(long long m, long long n, int k, bool half) {
  const long long outputs = m * n;
  if (!half) return k <= 16 ? outputs >= 400000 : k <= 32 && outputs >= 1000000;
  if (k <= 16) return n <= 2048 && outputs >= (n <= 32 ? 400000 : 1000000);
  if (k <= 32) return n <= 2048 && outputs >= 1300000;
  return outputs >= 3000000 && (n <= 32 ? k <= 64 : k <= 48 && n > 64 && n <= 512);
}

}  // namespace tfx

#endif  // TFX_KERNEL_COST_H_
