// Host check of the W4A16 kernel choice at 33 to 64 tokens (w4a16_plan.h) against measured times: reads the table given as
// argument and prints, for the choices on 256 CUs, how far they are from the better one of each row.
#include <cstdio>

#include "w4a16_plan.h"

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
  Sum sum;
  FILE* f = std::fopen(argv[1], "r");
  if (!f) return 1;
  while (std::fgets(line, sizeof line, f)) {
    int M, N, K, g;
    double few, tiles;
    if (line[0] == '#' || std::sscanf(line, "%d %d %d %d %lf %lf", &M, &N, &K, &g, &few, &tiles) != 6) continue;
    sum.add(w16::two_few_launches(M, N, K, g, 256) ? few : tiles, few < tiles ? few : tiles, line);
  }
  std::fclose(f);
  sum.print("two_few_or_tiles");
  return 0;
}
