#ifndef TFX_KERNEL_COST_H_
#define TFX_KERNEL_COST_H_

namespace tfx {

// Which kernel: the one that a model of their times says is fastest.  A kernel of bm x bn tiles gives
// c = batch x tiles / 256 of them to a CU (a whole number of rounds while there are few), each of which walks through k:
//   us = fixed + per_k k + c (per_tile + per_tile_k k)
// per_k is the memory round trips of a chain that nothing hides, per_tile_k what k costs the CU.  Fitted to the measured
// times of 226 products and 190 convolutions of either storage type (sizes 16 ... 4096, channels 3 ... 512; mean error
// 4 - 18 %); over these its choice costs 2 - 4 % against the fastest kernel of each.
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

// Whether gemm_thin.hip is the fastest: from how many outputs on its start (B into registers, longer with k) is paid back.
// Measured on 1x1 convolutions of 100 ... 250 000 rows: floats, 8 -> 16 channels, 200704 rows 25 -> 8 us, 40 -> 152, 248292
// rows 145 -> 80; 48 -> 24, 1700 rows 3.5 -> 5.3 (not taken); halfs, 11 -> 22, 207936 rows 33 -> 7.
inline bool thin_pays(long long m, long long n, int k, bool half) {
  const long long outputs = m * n;
  if (!half) return k <= 16 ? outputs >= 400000 : k <= 32 ? outputs >= 1000000 : k <= 48 && outputs >= 20000000;
  if (k <= 16) return outputs >= (n <= 32 ? 400000 : 1000000);
  return k <= 32 ? outputs >= 1300000 : k <= 64 ? outputs >= 3000000 : k <= 128 && outputs >= 10000000;
}

}  // namespace tfx

#endif  // TFX_KERNEL_COST_H_
