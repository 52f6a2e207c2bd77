// Host check of the split of tokens between the two tile sizes of the pipelined W4A4 kernel (pipe_plan.h): the same plan
// as the walk over every split of the last two rounds, and few splits looked at.
#include <cstdio>

#include "pipe_plan.h"

using namespace dirotq;

static double every_split(int M, int N, int cus, long& big_tokens) {
  const uint32_t wpx = (uint32_t)std::max(1, cus / 8);
  const long n_nt = (N + 255) / 256, n_big = (M + 255) / 256, lo = std::max(1L, n_big - 2 - 16L * wpx / n_nt);
  long best_t = n_big;
  double best = pipe::split_at(n_big, M, n_nt, wpx);
  for (long t = n_big - 1; t >= 0; t = t > lo ? t - 1 : t ? 0 : -1) {
    const double c = pipe::split_at(t, M, n_nt, wpx);
    if (c < best) best = c, best_t = t;
  }
  big_tokens = std::min(best_t * 256, (long)M);
  return best;
}

int main() {
  long failures = 0, n = 0;
  uint64_t state = 1;
  auto next = [&](uint32_t below) { return (uint32_t)((state = state * 6364136223846793005ull + 1442695040888963407ull) >> 33) % below; };
  auto check = [&](int M, int N, int cus) {
    long a = -1, b = -1;
    const double ta = w4a4_pipe_plan(M, N, cus, a), tb = every_split(M, N, cus, b);
    n++;
    if ((a != b || ta != tb) && failures++ < 10) std::printf("M=%d N=%d cus=%d: %ld (%g), every split: %ld (%g)\n", M, N, cus, a, ta, b, tb);
  };
  for (int cus : {1, 8, 80, 256, 304})
    for (int N = 1; N <= 4200; N += N < 64 ? 63 : 128)
      for (int M = 1; M <= 70000; M += 1 + next(900)) check(M, N, cus);
  for (int i = 0; i < 20000; i++) check(1 + next(1 << 24), 1 + next(1 << (8 + next(9))), 256);
  std::printf("%ld failure(s) of %ld\n", failures, n);
  return failures != 0;
}
