// Host side of the pipelined kernel B (w4a4_gemm_pipe.hip): how a layer's tokens are split between its two tile sizes.
// Plain C++: a host test compares it with the walk over every split.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace dirotq {

namespace pipe {

constexpr int TNW = 256;                     // output channels per workgroup tile (4 waves of 64)

// Time of a 256 x 128 tile, in units of a 256 x 256 one: median of 189 layers of more than three rounds of small tiles,
// all in large or all in small ones, with the field form
constexpr double HALF = 0.65;

// Time of the workgroup that has most to do with `big` 256 x 256 tiles and `small` 256 x 128 ones, in units of a large
// tile, a small one takes HALF (field form, M = 8192, K = 3072, N = 9216: 4.5 rounds 310 us, 9 small ones 377), and a workgroup that has both kinds drains and refills its
// pipeline once in between.  Per XCD (wpx workgroups) the large tiles are dealt to the slots 0, 1, ... in turn, the small
// ones to the slots from the other end.
inline double most(long big, long small, uint32_t wpx) {
  constexpr double PHASE = 0.04;
  const uint32_t b = (uint32_t)((big + 7) / 8), h = (uint32_t)((small + 7) / 8);
  const uint32_t bq = b / wpx, br = b % wpx, hq = h / wpx, hr = h % wpx;
  auto time = [&](uint32_t nb, uint32_t nh) { return nb + HALF * nh + (nb && nh ? PHASE : 0.0); };
  if (br + hr > wpx) return time(bq + 1, hq + 1);
  return std::max(time(bq, hq), std::max(br ? time(bq + 1, hq) : 0.0, hr ? time(bq, hq + 1) : 0.0));
}
// ... with the first `t` runs of 256 tokens in large tiles
inline double split_at(long t, int M, long n_nt, uint32_t wpx) {
  return most(t * n_nt, t * 256 < M ? ((M - t * 256 + 127) / 128) * n_nt : 0, wpx);
}

}  // namespace pipe

// Where the tokens are split, so that the workgroup with the most work has least of it.  N = 12288, M = 4608 (3.375 tiles of
// 256 x 256 per CU): 248 us with three rounds of large tiles and one of small ones, 266 us with large ones only, 307 us
// with small ones only.  big_tokens: how many of the first tokens go to the large tiles; returns the time in their units.
inline double w4a4_pipe_plan(int M, int N, int cus, long& big_tokens) {
  const uint32_t wpx = (uint32_t)std::max(1, cus / 8);
  const long n_nt = (N + pipe::TNW - 1) / pipe::TNW;
  // (only a split within the last two rounds of large tiles, or none at all, can be the best one)
  const long n_big = (M + 255) / 256, lo = std::max(1L, n_big - 2 - 16L * wpx / n_nt);
  long best_t = n_big;
  double best = pipe::split_at(n_big, M, n_nt, wpx);
  // downwards over the splits that put another large tile less on an XCD: between them only the small ones grow (with
  // N <= 256 every eighth split: 66 instead of 514 on 256 CUs)
  for (long t = n_big; t > 0;) {
    const long down = n_nt >= 8 ? t - 1 : 8 * (((uint32_t)(t * n_nt) + 7) / 8 - 1) / (uint32_t)n_nt;
    t = down >= lo ? down : 0;
    const double c = pipe::split_at(t, M, n_nt, wpx);
    if (c < best) {
      best = c;
      best_t = t;
    }
  }
  big_tokens = std::min(best_t * 256, (long)M);
  return best;
}

}  // namespace dirotq
