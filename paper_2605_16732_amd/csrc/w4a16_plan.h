// Host side of the W4A16 GEMM: which of its kernels runs a layer.  Plain C++: a host test compares the choice with measured
// times (tests/golden/w4a16_kernel_times.txt).
#pragma once

#include <initializer_list>

namespace dirotq {
namespace w16 {

// Channels per workgroup of the stream over the weights at 9 to 32 tokens: 48 where 32 would leave some CUs a second workgroup
// and 48 do not.
inline int few_channels(int N, int cus) { return (N + 31) / 32 > cus && (N + 47) / 48 <= cus ? 48 : 32; }

// The tiles with nj (1, 2, 4 or 5) token tiles per workgroup, us: a first round of workgroups, further ones (with one or two
// token tiles they overlap it: two workgroups fit a CU), per step of 128 channels and per step for every CU's worth of
// workgroups (power, memory).  Groups of 32 apart: their scale sweep is twice as long.  Fitted to 1428 measured layers
// (nj = 4 and 5: 600), 2 to 3.5% off (root mean square).
inline double tile_us(long M, long N, long K, int g, int nj, int cus) {
  struct Cost { double first, round, round_step, step, full; };
  static constexpr Cost kCost[2][4] = {
      {{3.23, 1.30, 0.36, 0.49, 0.03}, {3.46, 1.81, 0.50, 0.58, 0.09}, {6.00, 4.49, 0.79, 0.66, 0.34}, {7.15, 5.41, 0.77, 0.68, 0.57}},
      {{3.59, 1.41, 0.41, 0.61, 0.05}, {3.62, 2.61, 0.78, 0.77, 0.06}, {6.19, 4.53, 0.85, 0.84, 0.45}, {7.49, 5.10, 1.13, 1.03, 0.44}}};
  const Cost& c = kCost[g == 32][nj < 4 ? nj - 1 : nj - 2];
  const long wgs = ((M + 32 * nj - 1) / (32 * nj)) * ((N + 127) / 128);
  const double more = (double)((wgs + cus - 1) / cus - 1), steps = (double)((K + 127) / 128);
  return c.first + c.round * more + steps * (c.round_step * more + c.step + c.full * (double)wgs / cus);
}
// The cheapest: on average 0.03% and at most 2.9% above the best of 602 layers, 0.10% and at most 4.9% of 140 that were not in the
// fit.  N = 1152, K = 4608, us with 1 | 2 | 4 | 5 token tiles: 512 tokens 22.5 | 25.7 | 34.9 | 40.1, 1024: 33.1 | 26.2 |
// 35.0 | 40.2, 2048: 48.1 | 40.9 | 35.5 | 40.2, 4096: 78.0 | 67.9 | 76.1 | 48.8.
inline int token_tiles(long M, long N, long K, int g, int cus) {
  int nj = 5;
  double us = tile_us(M, N, K, g, nj, cus);
  for (int c : {4, 2, 1}) {
    const double t = tile_us(M, N, K, g, c, cus);
    // (grids of 512 threads stay below 2^32)
    if (t <= us && (M + 32 * c - 1) / (32 * c) * ((N + 127) / 128) <= 1L << 22) us = t, nj = c;
  }
  return nj;
}

// 33 to 64 tokens: two launches of the kernel for up to 32 are faster where K is long (the tiles walk it with one workgroup
// per 128 channels, the stream with one per 32) and its workgroups make one round.  Workgroups of 48 channels: only with
// groups of 32, the shortest second launches and the longest K (N = 9216, K = 12288, two launches | tiles, us: 33 tokens 59.9
// | 63.7, 48: 70.8 | 63.9; groups of 64, 33 tokens 50.3 | 51.0).  Both launches together, us, and per panel of 512 channels,
// by the second one's tokens (more than 8, up to 8) and the channels of a workgroup (32, 48); on average 0.04% and at most 4%
// above the better one of 826 layers, 0.09% and 4% of 120 that were not in the fit.  Two launches | tiles, us, K x N: 1152 x
// 1152, 48 tokens 8.8 | 7.6; 4608 x 1152, 33 tokens 15.7 | 21.1, 48: 17.8 | 21.0; groups of 32, 48: 21.7 | 25.9; 12288 x 3072,
// 48: 40.1 | 50.8; 3072 x 9216, 48: 19.4 | 15.6.
inline bool two_few_launches(int M, int N, int K, int g, int cus) {
  const int channels = few_channels(N, cus);
  if (M <= 32 || M > 64 || (N + channels - 1) / channels > cus) return false;
  struct Cost { double both, panel; };
  static constexpr Cost kCost[2][2][2] = {{{{4.45, 1.58}, {6.05, 2.26}}, {{4.06, 1.33}, {5.55, 1.96}}},
                                          {{{4.21, 2.04}, {7.25, 2.66}}, {{3.81, 1.72}, {4.34, 2.48}}}};
  const Cost& c = kCost[g == 32][M <= 40][channels == 48];
  return c.both + c.panel * (double)((K + 511) / 512) < tile_us(M, N, K, g, token_tiles(M, N, K, g, cus), cus);
}

}  // namespace w16
}  // namespace dirotq
