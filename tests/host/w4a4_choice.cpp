// Host check of the W4A4 schedule choice (w4a4_plan.h) against measured times: reads the table given as argument and prints,
// for the choices on 256 CUs, how far they are from the best schedule of each row, and whether every grid of the 128 x 128
// tiles stays below 2^32 threads.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "w4a4_plan.h"

using namespace dirotq;

struct Sum {
  int n = 0, over5 = 0;
  double excess = 0, worst = 1;
  void add(double t, double best, const char* row) {
    const double x = t / best;
    n++, excess += x - 1, over5 += x > 1.05;
    if (x > worst) worst = x;
    if (x > 1.2) std::printf("%.2f: %s", x, row);
  }
  void print(const char* name) const { std::printf("%s: rows %d mean_excess %.5f over5 %d worst %.3f\n", name, n, excess / n, over5, worst); }
};

int main(int, char** argv) {
  char line[256];
  Sum small, large;
  FILE* f = std::fopen(argv[1], "r");
  if (!f) return 1;
  while (std::fgets(line, sizeof line, f)) {
    int M, N, K, r, g, asym;
    char c[5][16];
    if (line[0] == '#' || std::sscanf(line, "%d %d %d %d %d %d %15s %15s %15s %15s %15s", &M, &N, &K, &r, &g, &asym, c[0], c[1], c[2], c[3], c[4]) != 11) continue;
    double t[5], best = 1e30;
    for (int i = 0; i < 5; i++) {
      t[i] = std::strcmp(c[i], "-") ? std::atof(c[i]) : 1e30;
      if (t[i] < best) best = t[i];
    }
    long big = 0;
    const W4A4Schedule s = w4a4_choose(M, N, K, r, g, asym, 256, big);
    const int i = s == W4A4Schedule::kSkinny32 ? 0 : s == W4A4Schedule::kSkinny64 ? 1 : s == W4A4Schedule::kTile ? 2 : s == W4A4Schedule::kWs ? 3 : 4;
    (i < 3 ? small : large).add(t[i], best, line);
  }
  std::fclose(f);
  small.print("split_k_or_tiles");
  large.print("persistent");
  // the largest outputs that the shape rules admit, narrow and wide, with and without 4-bit channels
  int big = 0;
  for (long N : {1L, 33L, 129L, 6001L, 8065L, 12288L, 1L << 20, 1L << 24})
    for (long K : {32L, 640L, 12288L})
      for (int g : {32, 64})
        for (int kind = 0; kind < 3; kind++) {            // symmetric, asymmetric, 16-bit channels only
          const long M = std::min(1L << 24, (1L << 30) / ((N + 127) / 128) * 128);
          long split = 0;
          const W4A4Schedule s = w4a4_choose((int)M, (int)N, (int)K, kind == 2 ? (int)K : 0, g, kind == 1, 256, split);
          if (s != W4A4Schedule::kTile && s != W4A4Schedule::kDense) continue;
          const long slab = w4a4_plan::slab_tokens(N), tokens = kind == 2 ? std::min(M, slab) : M;
          big += slab < 128 || slab % 128 != 0 || (kind == 2) != (s == W4A4Schedule::kDense) ||
                 (s == W4A4Schedule::kTile ? 512 : 256) * w4a4_plan::tiles(tokens, N, 128, 128) >= 1L << 32;
        }
  std::printf("w4a4_grids: rows 0 mean_excess 0 over5 %d worst 1\n", big);
  return 0;
}
