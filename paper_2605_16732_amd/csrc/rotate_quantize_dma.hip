// Kernel A, tiles fed by global-to-LDS copies: x_hat = x Q with the split / per-group quantize / pack fused behind it
// (rotation/split equation of Section 4.2 and the quantizer of Section 3 of the paper); the same sums as
// rotate_quantize.hip, of which this is the form for launches of about one round of workgroups.
//
// Staging through registers stores every byte to LDS with ds_write, and those instructions share the LDS port with the
// operand reads (four waves reading and four storing: 80 and 56 bytes per clock; reading beside copies: 124 and 64, what each
// reaches alone).  A workgroup holds 64 x 32 or 64 x 64 outputs per wave, two or three waves per SIMD (a copy holds its wave
// up for about 75 clocks; another one feeds the matrix pipe meanwhile), and any multiple of 32 tokens, so that a launch can be
// cut into one full round.  A ring of three or four stages of 64 channels; within a stage the operands of the next 16 channels
// are read while those of the last are multiplied, copies sit behind the MFMAs, and the barrier that opens the next
// stage comes before the last 16 channels' MFMAs.  (All copies, then all reads, then all MFMAs of a stage, which the barrier
// makes every wave do at the same time: 38.5 instead of 35.3 us for M = 1000, K = 3072 in 128 x 160 tiles.)
//
// Bound: the copies (28 clocks per KB and CU in this pattern) and reads, 0.70 us a stage of 128 x 160, 0.72 to 0.95 of 128 x
// 256.  Measured against the best tiling through registers, us: K = 1152, M = 4096 21.7 -> 16.6, M = 7003 30.7 -> 22.3; K =
// 3072, M = 1500 44.1 -> 39.0; K = 2080, M = 1999 (stages of 32 channels there) 35.4 -> 26.7.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "rotate_epilogue.h"

namespace dirotq {

namespace dma {

constexpr int CI = 2;                                                 // 32-channel MFMA tiles of a wave
// wave tile: 64 channels x 32 TI tokens; workgroup: WC x WT waves
template <int TI, int WC, int WT>
struct Tile {
  static constexpr int C = 32 * CI * WC, T = 32 * TI * WT, NW = WC * WT, NT = NW * 64;
  static constexpr int ROWB = 128, STAGE = (C + T) * ROWB;           // 64 channels of a row
  static constexpr int COPIES = (C + T) / 8;                         // 1-KB copies of a stage: 8 rows each
  static constexpr int MOST = (COPIES + NW - 1) / NW, FULL = COPIES - (MOST - 1) * NW;   // per wave; waves that have MOST
  static constexpr int NBUF = std::min(160 * 1024 / STAGE, 4), SMEM = NBUF * STAGE;
  static_assert(NBUF >= 3 && NW * TI * 32 * 2 * 4 <= SMEM, "LDS");
};

__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

template <int TI, int WC, int WT, int QM>
__global__ __launch_bounds__(WC* WT * 64, (WC * WT + 3) / 4) void rotate_quantize_dma_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ Qt, int M, int K, int r, int g,
    uint16_t* __restrict__ xh, uint8_t* __restrict__ xl, uint16_t* __restrict__ sx, uint16_t* __restrict__ zx,
    float* __restrict__ xf, float* __restrict__ pmax, int r_pad, int Kv, int n_ct, int n_tt, int per_xcd, int sx_ld,
    bool fields) {
  using F = Tile<TI, WC, WT>;
  constexpr bool ASYM = QM == 1;
  constexpr int NBUF = F::NBUF;
  extern __shared__ __align__(16) unsigned char smem[];
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= n_ct * n_tt) return;
  constexpr int GC = 4;
  const int grp = logical / (GC * n_tt), in_grp = logical % (GC * n_tt), gc = min(n_ct - grp * GC, GC);
  const int v0 = (grp * GC + in_grp % gc) * F::C, m0 = in_grp / gc * F::T;
  const int t = threadIdx.x, l = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wc = w % WC, wt = w / WC;

  auto channel = [&](int v) { return max(v < r_pad ? min(v, r - 1) : min(r + (v - r_pad), K - 1), 0); };
  const int c0 = channel(v0);
  // copy i of this wave fills rows 8 (w + i NW) .. + 7
  uint32_t voff[F::MOST];
  const int piece = (l & 7) ^ swz(l >> 3), piece2 = piece ^ 4;        // (of even and odd copies: row / 8's parity is bit 2 of swz)
#pragma unroll
  for (int i = 0; i < F::MOST; i++) {
    const int k = w + i * F::NW, row = 8 * k + (l >> 3);
    const int gr = row < F::C ? channel(v0 + row) - c0 : min(m0 + row - F::C, M - 1) - m0;
    voff[i] = (uint32_t)gr * (uint32_t)(2 * K) + (k & 1 ? piece2 : piece) * 16;
  }
  const unsigned char* qbase = (const unsigned char*)(Qt + (size_t)c0 * K);
  const unsigned char* xbase = (const unsigned char*)(x + (size_t)m0 * K);
  const uint32_t ring = lds_address(smem) + w * 1024;
  const int nk = (K + 63) / 64;
  const bool half_last = (K & 63) != 0;
  const bool most = w < F::FULL;                                      // (this wave has MOST copies a stage)
  // part p of PARTS of this wave's copies of stage s
  constexpr int PARTS = 3;
  auto issue = [&](int s, int slot, int p) {
    const bool cut = half_last && s == nk - 1;                        // (the upper half lies past the row's end: the lower one again)
#pragma unroll
    for (int i = p * F::MOST / PARTS; i < (p + 1) * F::MOST / PARTS; i++) {
      if (i == F::MOST - 1 && F::FULL < F::NW && !most) break;
      const int k = w + i * F::NW;
      const uint32_t o = voff[i] - (cut && ((k & 1 ? piece2 : piece) & 4) ? 64u : 0u);
      copy_to_lds(ring + slot + i * (F::NW * 1024), o, (8 * k < F::C ? qbase : xbase) + (size_t)s * 128);
    }
  };
  auto wait_stage = [&](auto behind) {                                // until only the copies of `behind` later stages are in flight
    constexpr int B = decltype(behind)::value;
    if (F::FULL == F::NW || most) wait_copies<B * F::MOST>();
    else wait_copies<B * (F::MOST - 1)>();
  };

  f32x16 acc[CI][TI];
#pragma unroll
  for (int i = 0; i < CI; i++)
#pragma unroll
    for (int j = 0; j < TI; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;

#pragma unroll
  for (int n = 0; n < NBUF - 1; n++)
    if (n < nk)
#pragma unroll
      for (int p = 0; p < PARTS; p++) issue(n, n * F::STAGE, p);
  const int lrow = l & 31, h = l >> 5, sw = swz(lrow);
  const int offA = (wc * (32 * CI) + lrow) * 128, offB = (F::C + wt * (32 * TI) + lrow) * 128;
  bf16x8 a[2][CI], b[2][TI];
  auto fetch = [&](int slot, int ks) {
    const unsigned char* sp = smem + slot;
    const int at = ((2 * ks + h) ^ sw) << 4;
#pragma unroll
    for (int j = 0; j < TI; j++) b[ks & 1][j] = *(const bf16x8*)(sp + offB + j * (32 * 128) + at);
#pragma unroll
    for (int i = 0; i < CI; i++) a[ks & 1][i] = *(const bf16x8*)(sp + offA + i * (32 * 128) + at);
  };
  // stage s has landed (all waves' copies) and all waves have read stage s - 1
  auto enter = [&](int s) {
    const int behind = min(NBUF - 2, nk - 1 - s);
    if (behind <= 0) wait_stage(std::integral_constant<int, 0>{});
    else if (behind == 1) wait_stage(std::integral_constant<int, 1>{});
    else wait_stage(std::integral_constant<int, 2>{});
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  enter(0);
  fetch(0, 0);
  int cur = 0, fill = (NBUF - 1) * F::STAGE;
  for (int s = 0; s < nk; s++) {
    const int nxt = cur + F::STAGE == NBUF * F::STAGE ? 0 : cur + F::STAGE;
    const bool more = s + NBUF - 1 < nk, half = half_last && s == nk - 1;
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      if (ks < 3) {
        fetch(cur, ks + 1);
      } else if (s + 1 < nk) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // (stage s is read)
        enter(s + 1);
        fetch(nxt, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (ks < 2 || !half)
#pragma unroll
        for (int i = 0; i < CI; i++)
#pragma unroll
          for (int j = 0; j < TI; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks & 1][i], b[ks & 1][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (ks < PARTS && more) issue(s + NBUF - 1, fill, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
    fill = cur;
    cur = nxt;
  }

  // ---- epilogue ----
  const int vb = v0 + wc * (32 * CI), tok_base = m0 + wt * (32 * TI);
  if constexpr (QM == 2) {
    float amax[TI] = {};
    if (vb < r_pad)
      rq::store_bf16(acc, vb, tok_base, M, r, xh);
    else
      rq::store_f32(acc, vb - r_pad, tok_base, M, K - r, xf, amax);
    // a maximum covers 128 channels, two waves: the first one takes the second's
    __syncthreads();                                                // (the ring is done with)
    float* ex = (float*)smem;                                       // [wave][token tile][32 tokens]
#pragma unroll
    for (int j = 0; j < TI; j++)
      if (h == 0) ex[(w * TI + j) * 32 + lrow] = amax[j];
    __syncthreads();
    if (h != 0 || vb < r_pad || vb >= Kv || ((vb - r_pad) & 127) != 0) return;
#pragma unroll
    for (int j = 0; j < TI; j++) {
      const int m = tok_base + j * 32 + lrow;
      if (m < M) pmax[(size_t)((vb - r_pad) >> 7) * sx_ld + m] = fmaxf(amax[j], ex[((w ^ 1) * TI + j) * 32 + lrow]);
    }
    return;
  } else {
    float tm[TI][CI], tn[TI][CI];
    rq::tile_extremes<QM>(acc, tm, tn);
    rq::group_extremes(g, tm, tn);
    if (g == 128) {                                                 // extremes over 128 channels: two waves'
      __syncthreads();                                              // (the ring is done with)
      float* ex = (float*)smem;                                     // [wave][token tile][max | min][32 tokens]
#pragma unroll
      for (int j = 0; j < TI; j++) {
        if (h == 0) ex[((w * TI + j) * 2) * 32 + lrow] = tm[j][0];
        if (ASYM && h == 0) ex[((w * TI + j) * 2 + 1) * 32 + lrow] = tn[j][0];
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < TI; j++) {
        const float om = ex[(((w ^ 1) * TI + j) * 2) * 32 + lrow];
        tm[j][0] = tm[j][1] = fmaxf(tm[j][0], om);
        if constexpr (ASYM) {
          const float on = ex[(((w ^ 1) * TI + j) * 2 + 1) * 32 + lrow];
          tn[j][0] = tn[j][1] = fminf(tn[j][0], on);
        }
      }
    }
    if (vb >= Kv) return;
    if (vb < r_pad) {
      rq::store_bf16(acc, vb, tok_base, M, r, xh);
      if (vb + 32 * CI <= r_pad) return;
    }
    rq::store_low<QM>(acc, tm, tn, vb - r_pad, tok_base, M, K - r, g, xl, sx, zx, sx_ld, fields);
  }
}

template <int TI, int WC, int WT, int QM>
static int launch_one(const uint16_t* x, const uint16_t* Qt, int M, int K, int r, int g, const RqOut& o, int r_pad, int Kv,
                      hipStream_t s, int sx_ld) {
  using F = Tile<TI, WC, WT>;
  const int n_ct = (Kv + F::C - 1) / F::C, n_tt = (M + F::T - 1) / F::T;
  const int per_xcd = (int)(((long)n_ct * n_tt + 7) / 8);
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)rotate_quantize_dma_kernel<TI, WC, WT, QM>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, F::SMEM);
    if (e != hipSuccess) return hip_failed(e);
    attr_done.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((rotate_quantize_dma_kernel<TI, WC, WT, QM>), dim3(per_xcd * 8), dim3(F::NT), F::SMEM, s, x, Qt, M, K,
                     r, g, o.xh, o.xl, o.sx, o.zx, o.xf, o.pmax, r_pad, Kv, n_ct, n_tt, per_xcd, sx_ld, o.fields);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

template <int TI, int WC, int WT>
static int launch_tile(const uint16_t* x, const uint16_t* Qt, int M, int K, int r, int g, const RqOut& o, int r_pad, int Kv,
                       hipStream_t s, int sx_ld) {
  if (o.xf) return launch_one<TI, WC, WT, 2>(x, Qt, M, K, r, g, o, r_pad, Kv, s, sx_ld);
  if (o.zx) return launch_one<TI, WC, WT, 1>(x, Qt, M, K, r, g, o, r_pad, Kv, s, sx_ld);
  return launch_one<TI, WC, WT, 0>(x, Qt, M, K, r, g, o, r_pad, Kv, s, sx_ld);
}

}  // namespace dma

int launch_rotate_quantize_dma(const uint16_t* x, const uint16_t* Qt, int M, int K, int r, int g, const RqOut& o, int r_pad,
                               int Kv, int channels, int tokens, hipStream_t s, int sx_ld) {
  if (channels == 256) return dma::launch_tile<2, 4, 2>(x, Qt, M, K, r, g, o, r_pad, Kv, s, sx_ld);
  switch (tokens) {
    case 128: return dma::launch_tile<1, 2, 4>(x, Qt, M, K, r, g, o, r_pad, Kv, s, sx_ld);
    case 160: return dma::launch_tile<1, 2, 5>(x, Qt, M, K, r, g, o, r_pad, Kv, s, sx_ld);
    case 192: return dma::launch_tile<1, 2, 6>(x, Qt, M, K, r, g, o, r_pad, Kv, s, sx_ld);
    default: return dma::launch_tile<2, 2, 4>(x, Qt, M, K, r, g, o, r_pad, Kv, s, sx_ld);
  }
}

}  // namespace dirotq
