// Host side of the W4A16 GEMM: which of its kernels runs a layer.  Plain C++: a host test compares the choice with measured
// times (tests/golden/w4a16_kernel_times.txt).
#pragma once

#include <initializer_list>

namespace dirotq {
namespace w16 {

// Token tiles per workgroup: the cheapest of 1, 2, 4 and 5, by rounds of workgroups over the CUs times a round's time
// per step of 128 channels (0.45, 0.63, 1.15 and 1.40 us: a larger tile costs less per output, 0.45 against 0.28 per 32 x
// 128, a smaller one leaves less of the last round empty).  N = 1152, K = 4608, us with 1 | 2 | 4 | 5 token tiles:
// 512 tokens 23.1 | 27.3 | 41.5 | 50.3, 2048: 50.3 | 44.6 | 42.8 | 50.2, 4096: 78.6 | 68.2 | 84.3 | 55.4.
inline long tile_rounds(long M, long N, int nj, int cus) {
  const long wgs = ((M + 32 * nj - 1) / (32 * nj)) * ((N + 127) / 128);
  return (wgs + cus - 1) / cus;
}
inline int token_tiles(long M, long N, long K, int cus) {
  const double step_us[6] = {0, 0.45, 0.63, 0, 1.15, 1.40};
  auto us = [&](int nj) { return 4.0 + step_us[nj] * (double)((K + 127) / 128) * (double)tile_rounds(M, N, nj, cus); };
  int nj = 1;
  for (int c : {2, 4, 5})
    if (us(c) < us(nj)) nj = c;
  return nj;
}

// 33 to 64 tokens: two launches of the few-token kernel are faster where K is long (the tiles walk it with one workgroup per
// 128 channels, the stream with one per 32) and its workgroups fit one round.  Fitted to 264 measured layers (within 7%): two
// launches 4.4 us and 1.5 (second one up to 8 tokens) or 1.8 us per 512 channels and round, groups of 32 1.8 or 2.15; the
// tiles 3.7 us and 0.49 us per 128 channels, groups of 32 4.0 and 0.62 (their scale sweep is twice as long).  Two launches
// | tiles, us: 1152 x 1152, 48 tokens 9.7 | 8.1; 4608 x 1152, 33 tokens 17.9 | 21.5, 48: 20.5 | 21.5; groups of 32, 48:
// 23.3 | 26.3; 3072 x 9216 28.1 | 15.7; 12288 x 3072 49.2 | 51.0.
inline bool two_few_launches(int M, int N, int K, int g, int cus) {
  if (M <= 32 || M > 64) return false;
  const int nj = token_tiles(M, N, K, cus);
  const double chunks = (K + 511) / 512, steps = (K + 127) / 128, few_rounds = (double)(((N + 31) / 32 + cus - 1) / cus);
  const double few = 4.4 + (g == 32 ? (M <= 40 ? 1.8 : 2.15) : (M <= 40 ? 1.5 : 1.8)) * chunks * few_rounds;
  const double tile_steps = steps * (double)tile_rounds(M, N, nj, cus) * (nj == 1 ? 1.0 : 1.4);
  return few < (g == 32 ? 4.0 + 0.62 * tile_steps : 3.7 + 0.49 * tile_steps);
}

}  // namespace w16
}  // namespace dirotq
