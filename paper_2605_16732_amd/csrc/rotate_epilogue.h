// Epilogue of kernel A's waves whose accumulators are CI x TI tiles of 32 channels x 32 tokens (32x32 MFMA layout: a lane owns one
// token and 4 consecutive channels per register quad, so a tile's maximum is in-lane work and one exchange within the lane
// pair): the split at r, the per-group quantizer and the packing, all in registers.  QM as in rotate_quantize.hip.  Virtual
// channels: the 16-bit part, then the 4-bit part from r_pad on; cl0: the wave's first 4-bit channel (negative: the split
// point lies inside the wave's channels).
#pragma once

#include "pipe_unpack.h"

namespace dirotq {
namespace rq {

// Absolute maximum (QM 1: maximum and minimum) of each tile's 32 channels
template <int QM, int CI, int TI>
__device__ __forceinline__ void tile_extremes(const f32x16 (&acc)[CI][TI], float (&tmax)[TI][CI], float (&tmin)[TI][CI]) {
#pragma unroll
  for (int j = 0; j < TI; j++)
#pragma unroll
    for (int i = 0; i < CI; i++) {
      if constexpr (QM == 1) {
        float lo = acc[i][j][0], hi = acc[i][j][0];
#pragma unroll
        for (int v = 1; v < 16; v++) {
          lo = fminf(lo, acc[i][j][v]);
          hi = fmaxf(hi, acc[i][j][v]);
        }
        tmin[j][i] = fminf(lo, __shfl_xor(lo, 32));
        tmax[j][i] = fmaxf(hi, __shfl_xor(hi, 32));
      } else {
        float a = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; v++) a = fmaxf(a, fabsf(acc[i][j][v]));
        tmax[j][i] = fmaxf(a, __shfl_xor(a, 32));
        tmin[j][i] = 0.0f;
      }
    }
}

// ... then of each group of g channels, as far as the wave holds it
template <int CI, int TI>
__device__ __forceinline__ void group_extremes(int g, float (&tmax)[TI][CI], float (&tmin)[TI][CI]) {
#pragma unroll
  for (int half = 1; half < CI; half *= 2)
    if (g >= 64 * half)
#pragma unroll
      for (int j = 0; j < TI; j++)
#pragma unroll
        for (int i = 0; i < CI; i += 2 * half) {
          const float hi = fmaxf(tmax[j][i], tmax[j][i + half]), lo = fminf(tmin[j][i], tmin[j][i + half]);
#pragma unroll
          for (int k = 0; k < 2 * half; k++) {
            tmax[j][i + k] = hi;
            tmin[j][i + k] = lo;
          }
        }
}

// 16-bit part: 4 consecutive channels per register quad -> one 8-byte store
template <int CI, int TI>
__device__ __forceinline__ void store_bf16(const f32x16 (&acc)[CI][TI], int vb, int tok_base, int M, int r, uint16_t* xh) {
  const int l = threadIdx.x & 63, h = l >> 5;
#pragma unroll
  for (int j = 0; j < TI; j++) {
    const int m = tok_base + j * 32 + (l & 31);
#pragma unroll
    for (int i = 0; i < CI; i++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int c = vb + i * 32 + 8 * q + 4 * h;
        if (c < r && m < M) {
          uint2 o;
          o.x = f32_to_bf16_bits(acc[i][j][4 * q]) | ((uint32_t)f32_to_bf16_bits(acc[i][j][4 * q + 1]) << 16);
          o.y = f32_to_bf16_bits(acc[i][j][4 * q + 2]) | ((uint32_t)f32_to_bf16_bits(acc[i][j][4 * q + 3]) << 16);
          *(uint2*)(xh + (size_t)m * r + c) = o;
        }
      }
  }
}

// QM 2, waves past the 16-bit part (which here ends on 128 channels): the channels as fp32, in 16-byte stores.  amax: the
// wave's absolute maximum over them for each token; a lane's maximum is taken beside the stores and exchanged once (an exchange
// for each tile, all before the first store: M = 896, K = 3072 with the per-token quantizer 32.1 against 31.7 us)
template <int CI, int TI>
__device__ __forceinline__ void store_f32(const f32x16 (&acc)[CI][TI], int cl0, int tok_base, int M, int KL, float* xf, float (&amax)[TI]) {
  const int l = threadIdx.x & 63, h = l >> 5;
#pragma unroll
  for (int j = 0; j < TI; j++) {
    const int m = tok_base + j * 32 + (l & 31);
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < CI; i++) {
      const int cl = cl0 + i * 32;
      if (cl < KL) {
#pragma unroll
        for (int v = 0; v < 16; v++) a = fmaxf(a, fabsf(acc[i][j][v]));
        if (m < M)
#pragma unroll
          for (int q = 0; q < 4; q++)
            *(float4*)(xf + (size_t)m * KL + cl + 8 * q + 4 * h) =
                make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
      }
    }
    amax[j] = fmaxf(a, __shfl_xor(a, 32));
  }
}

// 4-bit part: the codes (nibbles, or in field form) and scales (and zero-points) of the groups
template <int QM, int CI, int TI>
__device__ __forceinline__ void store_low(const f32x16 (&acc)[CI][TI], const float (&tmax)[TI][CI], const float (&tmin)[TI][CI], int cl0,
                                          int tok_base, int M, int KL, int g, uint8_t* xl, uint16_t* sx, uint16_t* zx, int sx_ld, bool fields) {
  constexpr bool ASYM = QM == 1;
  const int l = threadIdx.x & 63, h = l >> 5;
  const size_t xl_ld = (size_t)KL / 2;
  const int gi_tiles = g >> 5, g_log2 = 31 - __builtin_clz(g);   // 32-channel MFMA tiles per group: 1, 2, 4
#pragma unroll
  for (int j = 0; j < TI; j++) {
    const int m = tok_base + j * 32 + (l & 31);
#pragma unroll
    for (int i = 0; i < CI; i++) {
      const int cl = cl0 + i * 32;                          // first 4-bit channel of this tile
      const bool valid = cl >= 0 && cl < KL && m < M;
      uint16_t sbits, zbits = 0;
      float sf, zf = 0.0f;
      if constexpr (ASYM) {
        zf = group_zero(tmin[j][i], zbits);
        sf = group_scale_asym(tmin[j][i], tmax[j][i], sbits);
      } else {
        sf = group_scale(tmax[j][i], sbits);
      }
      const float inv = group_inv(sf);
      if (valid && h == 0 && ((cl >> 5) & (gi_tiles - 1)) == 0) {
        sx[(size_t)(cl >> g_log2) * sx_ld + m] = sbits;
        if constexpr (ASYM) zx[(size_t)(cl >> g_log2) * sx_ld + m] = zbits;
      }
      // this lane's 16 codes: quad q covers channels cl + 8q + 4h .. +3 -> one 16-bit piece, two pieces a dword
      float v0[8], v1[8];
#pragma unroll
      for (int v = 0; v < 8; v++) {
        v0[v] = acc[i][j][v];
        v1[v] = acc[i][j][8 + v];
      }
      const uint32_t P0 = quant_pack8<ASYM>(v0, zf, inv), P1 = quant_pack8<ASYM>(v1, zf, inv);
      // lane h=0 keeps dwords 0,1 of the tile's 16 bytes, lane h=1 dwords 2,3
      const uint32_t recv = __shfl_xor(h ? P0 : P1, 32);
      const uint32_t lo = h ? recv : P0, hi = h ? P1 : recv;
      uint2 o;
      o.x = (lo & 0xFFFFu) | (hi << 16);
      o.y = (lo >> 16) | (hi & 0xFFFF0000u);
      if (!ASYM && fields) o = pipe::to_fields_pair(o, h);
      if (valid) *(uint2*)(xl + (size_t)m * xl_ld + cl / 2 + 8 * h) = o;
    }
  }
}

}  // namespace rq
}  // namespace dirotq
