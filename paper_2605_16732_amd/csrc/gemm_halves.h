// Shared by the W4A16 tile kernel and the medium W4A8 one: 128 output channels x 32 NJ tokens per workgroup, eight waves: four of 32
// channels, twice, for the even and the odd stages of 64 channels of K (two waves per SIMD hide each other's latencies
// without decoding a weight twice).  D[token][n] orientation: accumulator v of lane (h, c) holds token 8 (v / 4) + 4 h +
// v % 4 of its tile and the wave's channel c.
#pragma once

#include "dirotq_internal.h"

namespace dirotq {
namespace halves {

constexpr int TN_ = 128, NT = 512, NBUF = 3;             // (a ring of three stages for each half of the waves)
constexpr int W_BYTES = TN_ * 32, S_BYTES = 4 * 256;     // of a stage: packed codes of 64 channels; scales per wave
constexpr int slot_bytes(int x_row, int nj) { return 32 * nj * x_row + W_BYTES + S_BYTES; }
// (the exchange at the end takes 16 KB per token tile)
constexpr int smem_bytes(int x_row, int nj) {
  const int ring = 2 * NBUF * slot_bytes(x_row, nj);
  return ring > nj * 16384 ? ring : nj * 16384;
}

// Workgroup -> tile: an XCD walks a contiguous run of tiles, four output tiles per token tile (operands stay in its L2).
__device__ __forceinline__ bool tile_of(int n_mt, int n_nt, int per_xcd, int tm, int& m0, int& n0) {
  constexpr int GN = 4;
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= n_mt * n_nt) return false;
  const int grp = logical / (GN * n_mt), in_grp = logical % (GN * n_mt), gn = min(n_nt - grp * GN, GN);
  n0 = (grp * GN + in_grp % gn) * TN_;
  m0 = in_grp / gn * tm;
  return true;
}

// The weight scales (fp16 [group][N]) of a wave's 32 (48: DWORDS = 28) channels from nw on: a copy brings a window of dwords
// that begins at the dword of the first one; with two groups the upper half of the lanes fetches the second one's.
struct ScaleRows {
  const unsigned char* base;
  size_t last;                                           // byte offset of the dword of the last scale
  int N, nw;
  __device__ __forceinline__ size_t at(int g) const { return ((size_t)g * N + nw) * 2 & ~(size_t)3; }
  template <bool TWO, int DWORDS = 20>
  __device__ __forceinline__ void copy(uint32_t lds, int g0, int g1) const {
    const int l = threadIdx.x & 63;
    const size_t e0 = at(g0);
    uint32_t v = min(TWO ? l & 31 : l, DWORDS - 1) * 4;
    if (TWO && l >= 32) v += (uint32_t)(at(g1) - e0);
    copy4_to_lds(lds, min(v, (uint32_t)min(last - e0, (size_t)0x7ffffffc)), base + e0);
  }
  __device__ __forceinline__ float read(const unsigned char* p, int g, int c) const {
    return f16_bits_to_f32(*(const uint16_t*)(p + ((((size_t)g * N + nw) & 1) + c) * 2));
  }
};

// The two halves exchange their sums (token tile j is finished by half j & 1), add the bias and store.
template <bool OUT_F32, int NJ>
__device__ __forceinline__ void finish(f32x16 (&acc)[NJ], unsigned char* smem, int kh, int w, int m0, int n0,
                                       const uint16_t* __restrict__ bias, int M, int N, void* __restrict__ y) {
  const int l = threadIdx.x & 63, h = l >> 5, c = l & 31;
  __syncthreads();
  float4* xch = (float4*)smem;
#pragma unroll
  for (int j = 0; j < NJ; j++)
    if ((j & 1) != kh)
#pragma unroll
      for (int q = 0; q < 4; q++)
        xch[((j * 4 + w) * 4 + q) * 64 + l] = make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
  __syncthreads();
  // two channels of a token in one dword: neighbouring lanes exchange, the even one stores token v, the odd one v + 1
  const int n = n0 + 32 * w + c;
  const float bn = bias && n < N ? bf16_bits_to_f32(bias[n]) : 0.0f;
  const bool pairs = !OUT_F32 && (N & 1) == 0, odd = l & 1;
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    if ((j & 1) != kh) continue;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const float4 o = xch[((j * 4 + w) * 4 + q) * 64 + l];
      acc[j][4 * q] += o.x;
      acc[j][4 * q + 1] += o.y;
      acc[j][4 * q + 2] += o.z;
      acc[j][4 * q + 3] += o.w;
    }
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const int m = m0 + j * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
      const float y0 = bias ? acc[j][v] + bn : acc[j][v], y1 = bias ? acc[j][v + 1] + bn : acc[j][v + 1];
      if (pairs) {
        const float got = __shfl_xor(odd ? y0 : y1, 1);
        const uint32_t d = f32x2_to_bf16x2_bits(odd ? got : y0, odd ? y1 : got);
        if (n < N && m + odd < M) *(uint32_t*)((uint16_t*)y + (size_t)(m + odd) * N + (n - odd)) = d;
      } else if (n < N) {
#pragma unroll
        for (int e = 0; e < 2; e++)
          if (m + e < M) {
            const float o = e ? y1 : y0;
            if (OUT_F32) ((float*)y)[(size_t)(m + e) * N + n] = o;
            else ((uint16_t*)y)[(size_t)(m + e) * N + n] = f32_to_bf16_bits(o);
          }
      }
    }
  }
}

}  // namespace halves
}  // namespace dirotq
