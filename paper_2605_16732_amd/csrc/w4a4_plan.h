// Host side of kernel B: which of its schedules runs a W4A4 layer.  Plain C++: a host test compares the choice with measured
// times of all schedules (tests/golden/w4a4_schedule_times.txt).
#pragma once

#include "pipe_plan.h"

namespace dirotq {

enum class W4A4Schedule { kTile, kWs, kSkinny32, kSkinny64, kPipe, kDense };

struct W4A4Plan {
  W4A4Schedule schedule = W4A4Schedule::kTile;
  long big_tokens = 0;                       // (kPipe: see w4a4_pipe_plan)
  // whether kernel A writes the symmetric activation codes of a whole layer in field form (pipe_unpack.h) for it
  bool reads_fields() const { return schedule == W4A4Schedule::kTile || schedule == W4A4Schedule::kPipe; }
};

namespace w4a4_plan {

// 128 x 128 tiles of a launch, at most: its grid (512 threads a tile) stays below 2^32 threads.  Layers with 4-bit channels that
// have more go to the persistent kernels, others in several launches (slab_tokens).
constexpr long MOST_TILES = 1L << 22;

inline long tiles(long M, long N, long m, long n) { return ((M + m - 1) / m) * ((N + n - 1) / n); }
inline double rounds(long work, long slots) { return (double)((work + slots - 1) / slots); }

// Costs in microseconds of the schedules: k = 1024 4-bit channels, q = 128 16-bit ones.  Fitted to what kernel B adds to
// kernel A in whole layers (graph replay over three sets of weights and activations; K = 640 ... 12288, N = 320 ... 12288, all
// group sizes): the split-K forms to 7250 layers of up to 9000 tokens with r up to 256, the 128 x 128 tiles to 1260 with the
// field form and r up to 2048, the persistent kernels to 650 of those (3 to 6% off, root mean square).  The last two stand times
// 1.03 and 1.02 (groups of 32, wave-specialised: 1.07), which is what the split-K forms' costs are above the
// present times: only the comparisons matter.  The numbers that depend on the kind of code stand as {groups of 64, 128, 32
// symmetric; the same asymmetric}; ragged: rows of y that do not begin at multiples of 8 (persistent kernels: 8 or 16, tile:
// 16) bytes are stored in smaller pieces, down to single values.
struct Cost {
  double k, q;
  int kind, cus;
  Cost(int K, int r, int g, bool asym, int cus)
      : k((K - r) / 1024.0), q(r / 128.0), kind((g == 64 ? 0 : g == 128 ? 1 : 2) + (asym ? 3 : 0)), cus(cus) {}
  // 64 x 64 outputs, one workgroup per CU (128 KB of LDS)
  double skinny64(long M, long N) const {
    static constexpr double K[6] = {2.07, 2.10, 3.40, 2.80, 3.35, 5.52};
    const long T = tiles(M, N, 64, 64);
    const double ragged = N % 4 ? 0.93 : 0.0;
    return 2.10 + rounds(T, cus) * (1.41 + ragged + 0.66 * q + K[kind] * k) + (double)T / cus * (2.82 + 0.09 * k + 0.42 * q);
  }
  // 32 x 32 outputs, two workgroups per CU (registers)
  double skinny32(long M, long N) const {
    static constexpr double K[6] = {0.69, 0.68, 1.60, 0.75, 0.72, 1.67}, T1[6] = {0.44, 0.46, 0.51, 0.53, 0.54, 0.83};
    const long T = tiles(M, N, 32, 32);
    const double ragged = N % 4 ? 0.46 : 0.0;
    return 2.31 + 0.56 * k + rounds(T, 2L * cus) * (0.40 * q + K[kind] * k) +
           (double)T / cus * (0.70 + ragged + T1[kind] * k + 0.32 * q);
  }
  // 128 x 128 tiles, one per CU (LDS, registers)
  double tile(long M, long N) const {
    static constexpr double K[6] = {4.81, 4.69, 8.13, 5.89, 5.95, 9.93};
    const long T = tiles(M, N, 128, 128);
    const double ragged = N % 8 ? 1.39 : 0.0;
    return 3.01 + rounds(T, cus) * (3.36 + ragged + 1.16 * q + K[kind] * k) + (double)T / cus * (1.41 + 0.92 * k);
  }
  // Large layers: outputs of a 256 x 256 tile for every CU, as a measure for rows that are stored value by value
  double outputs(long M, long N) const { return (double)M * (double)N / (65536.0 * cus); }
  // 256 x 128 tiles of the wave-specialised kernel
  double ws(long M, long N) const {
    static constexpr double K[6] = {9.85, 9.66, 0.0, 12.74, 11.89, 28.84};
    const double ragged = N % 4 ? 40.26 : N % 8 ? 8.66 : 0.0;
    return 5.77 + rounds(tiles(M, N, 128, 256), cus) * (4.44 + 2.61 * q + K[kind] * k) + ragged * outputs(M, N);
  }
  // the pipelined kernel, whose plan takes the time of `large` 256 x 256 tiles
  double pipe(double large, long M, long N) const {
    static constexpr double K[3] = {17.33, 17.30, 28.00}, Q[3] = {5.39, 5.39, 7.85};
    const double ragged = N % 4 ? 42.22 : N % 8 ? 7.77 : 0.0;
    return 4.61 + large * (5.92 + Q[kind] * q + K[kind] * k) + ragged * outputs(M, N);
  }
};

// Tokens of a launch of the 128 x 128 tiles: as many whole tiles as MOST_TILES allows
inline long slab_tokens(long N) { return MOST_TILES / ((N + 127) / 128) * 128; }

}  // namespace w4a4_plan

// Large layers, from 128 tiles of 256 x 128 on: the cheapest of the pipelined kernel (symmetric; persistent workgroups, 256 x 256
// and 256 x 128 tiles), the wave-specialised one (256 x 128; not symmetric groups of 32) and the 128 x 128 tiles.  What kernel B
// takes, us, pipelined | wave-specialised | tiles: M = 4096, N = 3072, K = 1152 28 | 35 | 33; M = 4096, K = 3072, N = 1152 41 | 36 |
// 41, N = 6144 (1.5 rounds of 256 x 256 tiles) 134 | 118 | 132; N = 4026, K = 1536, whose rows are stored value by value, 74 | 78
// | 57; M = 10814, K = 3072, N = 2263, asymmetric - | 209 | 177.  500 layers that were not in the fit: on average 0.12% above the
// best of the three (symmetric at most 4%, asymmetric 14%, next 4%).
// Below: the cheapest of the split-K kernels (few tokens; 32 x 32 or 64 x 64 outputs per workgroup) and the 128 x 128 tiles:
// 0.29% above the best of 1206 layers (mean).  150 layers of either kind with r = 320 to 2048: 0.17%.  big_tokens: see
// w4a4_pipe_plan.
inline W4A4Schedule w4a4_choose(int M, int N, int K, int r, int g, bool asym, int cus, long& big_tokens) {
  using namespace w4a4_plan;
  big_tokens = 0;
  if (K - r <= 0) return tiles(M, N, 128, 128) > cus ? W4A4Schedule::kDense : W4A4Schedule::kTile;   // (see dense_gemm_kernel)
  const Cost cost(K, r, g, asym, cus);
  const double c128 = cost.tile(M, N);
  const long half_tiles = tiles(M, N, 128, 256);
  if (half_tiles >= 128) {
    double persistent = asym || g != 32 ? cost.ws(M, N) : 0.0;
    W4A4Schedule sch = W4A4Schedule::kWs;
    if (!asym) {
      const double plan = w4a4_pipe_plan(M, N, cus, big_tokens);
      // (groups of 32: half-size tiles only, and no wave-specialised form)
      const double c = cost.pipe(g == 32 ? pipe::HALF * rounds(half_tiles, cus < 8 ? 8 : cus / 8 * 8) : plan, M, N);
      if (g == 32 || c <= persistent) persistent = c, sch = W4A4Schedule::kPipe;
    }
    return c128 < persistent && tiles(M, N, 128, 128) <= MOST_TILES ? W4A4Schedule::kTile : sch;
  }
  const double c32 = cost.skinny32(M, N), c64 = cost.skinny64(M, N);
  if (c32 <= c64 && c32 <= c128) return W4A4Schedule::kSkinny32;
  return c64 <= c128 ? W4A4Schedule::kSkinny64 : W4A4Schedule::kTile;
}

}  // namespace dirotq
