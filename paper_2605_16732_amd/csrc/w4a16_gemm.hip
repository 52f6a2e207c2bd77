// W4A16 layers: 16-bit activations against 4-bit per-group weights, no rotation (the paper's
// appendix on quantization details keeps the input activations of some layers in 16 bits):
//   y[m,n] = sum_j s_w[n,j] * sum_{k in group j} x[m,k] q_w[n,k]   (+ bias[n]).
//
// A 4-bit code is a small integer and therefore an exact bf16 number, so the group sums run on
// the bf16 matrix pipe with nothing rounded before the fp32 accumulator; the per-group weight
// scale is applied afterwards, by one fma per accumulator and group.
//
// Up to 32 tokens a stream over the packed weights (one kernel up to 8, one beyond), then MFMA tiles (launch_w4a16_gemm).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include <cstdlib>
#include <cstring>

#include "gemm_halves.h"
#include "w4a16_plan.h"

namespace dirotq {

// ---- tiles (the layout of gemm_halves.h) ------------------------------------------------------------------------------
// All staging is copies global -> LDS (activations, packed codes, scales; a ring of three stages for each half, two in
// flight, one barrier per stage), so the waves issue nothing but operand reads, the decode, MFMAs and the scale sweep.
// A wave decodes the codes of its own 32 rows in registers, for its NJ token tiles: nibble -> fp8 subnormal byte -> bf16
// by the scaled conversion instruction (scale 2^9, exact), 12 instructions per 8 codes.
// D[token][n] orientation: a lane owns an output channel, so the group's scale is a per-lane number and one fma per
// accumulator and group applies it (no scale-product MFMA).
// Bound: not the matrix pipe alone (32 cycles x 4 per 32 x 32 tile and stage, 43 % of the time at NJ = 5) but with it the
// sweep and decode on the VALU and 28 KB of LDS traffic per 128 x 32 tile and stage (operand reads 16 KB, copies).  The
// kernel it replaces (128 x 128 tiles, two workgroups per CU) decoded into LDS, whose writes run at a quarter of the rate
// of reads, and had one stage of loads in flight.  Graph replay on one layer's weights, that kernel -> this one, us: 4096 x 4608 ->
// 1152 (M x K -> N) 111 -> 53 (now 51: 850 TFLOP/s), 512 tokens 87 -> 23; 4096 x 3072 -> 12288 454 -> 355 (now 344); 256 x 3072 -> 3072 51 -> 17.
namespace w16 {

using namespace halves;

// 8 sign-magnitude nibbles of a dword -> 8 bf16 numbers in channel order
__device__ __forceinline__ bf16x8 decode(uint32_t p) {
  uint32_t e, o;
  unpack8(p, e, o);
  const uint32_t lo = __builtin_amdgcn_perm(o, e, 0x05010400u), hi = __builtin_amdgcn_perm(o, e, 0x07030602u);
  uint4 r;                                               // bytes [s 0000 mmm] = m 2^-9 as fp8, times 2^9
  r.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.0f, false));
  r.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.0f, true));
  r.z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.0f, false));
  r.w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.0f, true));
  return __builtin_bit_cast(bf16x8, r);
}

template <int GS, bool OUT_F32, int NJ>
__global__ __launch_bounds__(NT, 1) void w4a16_large_kernel(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ wq, const uint16_t* __restrict__ sw,
    const uint16_t* __restrict__ bias, int M, int N, int K, void* __restrict__ y, int n_mt, int n_nt, int per_xcd) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int GPS = GS == 32 ? 2 : 1;                  // groups per stage
  constexpr int TM_ = 32 * NJ, X_BYTES = TM_ * 128, SLOT = slot_bytes(128, NJ);
  constexpr int COPIES = NJ + 2;                         // per wave and stage: activations, codes, scales
  // The copies of a stage sit behind the MFMAs of its token tiles (a copy holds its wave up for about 75 clocks, and with
  // all of them at the barrier all waves wait at once).  At the barrier -> spread, four layers' weights in turn, us: M = 4096, K =
  // 4608, N = 1152 56.3 -> 53.7, 2048 tokens 43.5 -> 38.0, K = 3072, N = 12288 397 -> 386; with a single token tile they come
  // first (M = 256, N = K = 3072 16.2, spread 17.2).
  constexpr bool SPREAD = NJ > 1;
  // With 4 or 5 token tiles each MFMA is followed by what the VALU can do beside it (32 cycles): four fma of the last tile's sweep,
  // across stages too, and a piece of the next stage's decode, whose codes and scales the wave has copied itself, so that
  // no barrier has to open them.  A tile's MFMAs, then the sweep, and the decode in front of a stage -> this, us: M = 4096, K =
  // 4608, N = 1152 53.0 -> 51.2, 2048 tokens 38.3 -> 36.7, K = 3072, N = 12288 360 -> 352; groups of 32, 2048 tokens 47.5 -> 46.6
  // (5 tiles: too many registers, equal).  Waves of 64 channels x half the tokens, which read half as much from LDS and decode
  // twice as much: 53.3 to 57.5 us for the first of these layers.
  // 1 and 2 tiles keep the plain order: the next stage's codes and scales may come in behind the first tile only, beside which the
  // last stage's scales are still in use, and their decode needs a further tile.
  constexpr bool FLOW = NJ >= 4 && !(GS == 32 && NJ == 5);
  int m0, n0;
  if (!tile_of(n_mt, n_nt, per_xcd, TM_, m0, n0)) return;
  const int t = threadIdx.x, l = t & 63, h = l >> 5, c = l & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), w = wave & 3, kh = wave >> 2;
  const int G = K / GS, nst = (K + 63) / 64, steps = (nst + 1) / 2;
  const bool short_last = GS == 32 && (K & 63) != 0;     // the last stage holds one 32-channel group

  // ---- copies of a stage by this wave: token rows 8 NJ w .. 8 NJ w + 8 NJ - 1 (8 rows per copy; 16-byte piece p of row `row` at
  // slot p ^ ((row >> 1) & 7)), the packed codes of its 32 weight rows (half p of row `row` at p ^ ((row >> 3) & 1)), and
  // their scales
  uint32_t vo_x[NJ];
#pragma unroll
  for (int i = 0; i < NJ; i++) {
    const int row = 8 * NJ * w + 8 * i + (l >> 3), piece = (l & 7) ^ ((row >> 1) & 7);
    vo_x[i] = (uint32_t)(min(m0 + row, M - 1) - m0) * (uint32_t)(2 * K) + piece * 16;
  }
  const int w_row = l >> 1, w_half = (l & 1) ^ ((w_row >> 3) & 1);
  const uint32_t vo_w = (uint32_t)(min(n0 + 32 * w + w_row, N - 1) - n0) * (uint32_t)(K / 2) + w_half * 16;
  const int nw = min(n0 + 32 * w, N - 1);                // first channel of the wave (past the edge: nothing is stored)
  const unsigned char *xb = (const unsigned char*)(x + (size_t)m0 * K), *wb = wq + (size_t)n0 * (K / 2);
  const uint32_t ring = lds_address(smem) + kh * (NBUF * SLOT);
  const ScaleRows scales = {(const unsigned char*)sw, ((size_t)G * N * 2 - 1) & ~(size_t)3, N, nw};
  auto group = [&](int s, int jj) { return min(GS == 32 ? 2 * s + jj : GS == 128 ? s >> 1 : s, G - 1); };
  // copies first .. end - 1 of a stage: activations (below NJ), codes, scales (past the last stage: that one again, unused)
  auto issue = [&](int s, int slot, int first, int end) {
    s = min(s, nst - 1);
    const uint32_t at = ring + slot;
    const bool cut = short_last && s == nst - 1;         // (the missing upper half: the lower one again)
#pragma unroll
    for (int i = 0; i < NJ; i++)
      if (i >= first && i < end) {
        const int row = 8 * NJ * w + 8 * i + (l >> 3), piece = (l & 7) ^ ((row >> 1) & 7);
        copy_to_lds(at + (8 * NJ * w + 8 * i) * 128, vo_x[i] - (cut && piece >= 4 ? 64u : 0u), xb + (size_t)s * 128);
      }
    if (NJ >= first && NJ < end) copy_to_lds(at + X_BYTES + w * 1024, vo_w - (cut && w_half ? 16u : 0u), wb + (size_t)s * 32);
    if (end == COPIES) scales.copy<GS == 32>(at + X_BYTES + W_BYTES + w * 256, group(s, 0), group(s, GPS - 1));
  };

  f32x16 acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; j++)
#pragma unroll
    for (int v = 0; v < 16; v++) acc[j][v] = 0.0f;
  // operand reads: k-step ks of lane half h is 16-byte piece 4 h + ks (8 channels) of a token row, dword ks of its half of
  // a weight row; groups of 32, which must not mix the halves: piece 2 ks + h, dword 2 ks + h of the whole row
  const int swx = (c >> 1) & 7, swz = (c >> 3) & 1;      // (tile bases are multiples of 32 rows)
  int ln_x[4];
#pragma unroll
  for (int ks = 0; ks < 4; ks++) ln_x[ks] = c * 128 + (((GS == 32 ? 2 * ks + h : 4 * h + ks) ^ swx) << 4);
  issue(kh, 0, 0, COPIES);
  issue(2 + kh, SLOT, 0, COPIES);
  int cur = 0;
  if constexpr (FLOW) {
    constexpr int SUBS = NJ * GPS, KS = 4 / GPS;         // groups of a stage's tiles, MFMAs of each
    constexpr int CODES_AT = NJ / 2 - 1, SLOTS = (NJ - 1 - CODES_AT) * 4;
    // (fetch_codes replaces the scales of the stage before, whose last tile is swept beside tile 0)
    static_assert(CODES_AT >= 1 && SLOTS >= 4, "codes and scales of the next stage come behind tile 0 and are decoded behind them");
    float fa[NJ][16];                                    // (value by value, so that they are accumulated in place)
#pragma unroll
    for (int j = 0; j < NJ; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) fa[j][e] = 0.0f;
    uint32_t p[4];
    bf16x8 a[2][4], b[2][4];
    f32x16 I[2];
    float sc[2][GPS];
#pragma unroll
    for (int v = 0; v < 16; v++) I[1][v] = 0.0f;         // (the tile before the first one)
#pragma unroll
    for (int jj = 0; jj < GPS; jj++) sc[1][jj] = 0.0f;
    auto fetch_codes = [&](int s, int slot, auto to) {
      const unsigned char *sp = smem + kh * (NBUF * SLOT) + slot + X_BYTES, *wp = sp + w * 1024 + c * 32;
      if constexpr (GS == 32) {
        const uint4 lo = *(const uint4*)(wp + (swz << 4)), hi = *(const uint4*)(wp + ((1 ^ swz) << 4));
        p[0] = h ? lo.y : lo.x;
        p[1] = h ? lo.w : lo.z;
        p[2] = h ? hi.y : hi.x;
        p[3] = h ? hi.w : hi.z;
      } else {
        const uint4 v = *(const uint4*)(wp + ((h ^ swz) << 4));
        p[0] = v.x, p[1] = v.y, p[2] = v.z, p[3] = v.w;
      }
#pragma unroll
      for (int jj = 0; jj < GPS; jj++) sc[to][jj] = scales.read(sp + W_BYTES + w * 256 + jj * 128, group(min(s, nst - 1), jj), c);
    };
    auto fetch_a = [&](int j) {
      const unsigned char* sp = smem + kh * (NBUF * SLOT) + cur;
#pragma unroll
      for (int ks = 0; ks < 4; ks++) a[j & 1][ks] = *(const bf16x8*)(sp + ln_x[ks] + j * (32 * 128));
    };
    auto stage = [&](int s, auto P_) {
      constexpr int P = decltype(P_)::value;
      int nxt = cur + SLOT, fill = cur + 2 * SLOT;
      if (nxt >= 3 * SLOT) nxt -= 3 * SLOT;
      if (fill >= 3 * SLOT) fill -= 3 * SLOT;
      const bool half_stage = short_last && s == nst - 1;
      fetch_a(0);
#pragma unroll
      for (int v = 0; v < SUBS; v++) {
        const int j = v / GPS, jj = v % GPS;
        const int now = (P * SUBS + v) & 1, pv = (v + SUBS - 1) % SUBS, pj = pv / GPS, pjj = pv % GPS;
        if (jj == 0 && j == CODES_AT) {                  // (the wave's own copies: no barrier)
          wait_copies<CODES_AT * COPIES / NJ>();
          fetch_codes(s + 2, nxt, std::integral_constant<int, P ^ 1>{});
        }
        if (jj == 0 && j + 1 < NJ) fetch_a(j + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < KS; k++) {
          const int ks = jj * KS + k;
          if (k == 0) {
            f32x16 z;
#pragma unroll
            for (int e = 0; e < 16; e++) z[e] = 0.0f;
            I[now] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j & 1][ks], b[P][ks], z, 0, 0, 0);
          } else {
            I[now] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j & 1][ks], b[P][ks], I[now], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (pjj == 0 || v == 0 || !half_stage)         // (not 0 x: an infinity would become a NaN)
#pragma unroll
            for (int e = k * 16 / KS; e < (k + 1) * 16 / KS; e++) {
              fa[pj][e] = fmaf(I[now ^ 1][e], sc[v == 0 ? P ^ 1 : P][pjj], fa[pj][e]);
              asm volatile("" : "+v"(fa[pj][e]));
            }
          if (j > CODES_AT) {
            const int slot = (j - CODES_AT - 1) * 4 + ks;
#pragma unroll
            for (int q = slot * 4 / SLOTS; q < (slot + 1) * 4 / SLOTS; q++) b[P ^ 1][q] = decode(p[q]);
          }
          if (k == KS - 1 && jj == GPS - 1) issue(s + 4, fill, j * COPIES / NJ, (j + 1) * COPIES / NJ);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      cur = nxt;
    };
    wait_copies<COPIES>();
    fetch_codes(kh, 0, std::integral_constant<int, 0>{});
#pragma unroll
    for (int ks = 0; ks < 4; ks++) b[0][ks] = decode(p[ks]);
    int s = kh;
    auto enter = [&]() {                                 // this wave's copies of stage s have landed, and (barrier) all waves';
      wait_copies<COPIES>();                             // stage s - 2 has been read by all of them
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    auto last = [&](auto P_) {                           // the last tile of the last stage
      constexpr int P = decltype(P_)::value;
      if (GPS == 1 || !short_last || s - 2 != nst - 1)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          fa[NJ - 1][e] = fmaf(I[(P * SUBS + SUBS - 1) & 1][e], sc[P][GPS - 1], fa[NJ - 1][e]);
          asm volatile("" : "+v"(fa[NJ - 1][e]));
        }
    };
    const int mine = (nst - kh + 1) / 2;                 // stages of this half
    for (int i = 1; i < mine; i += 2) {
      enter();
      stage(s, std::integral_constant<int, 0>{});
      s += 2;
      enter();
      stage(s, std::integral_constant<int, 1>{});
      s += 2;
    }
    if (mine & 1) {
      enter();
      stage(s, std::integral_constant<int, 0>{});
      s += 2;
      last(std::integral_constant<int, 0>{});
    } else if (mine) {
      last(std::integral_constant<int, 1>{});
    }
#pragma unroll
    for (int j = 0; j < NJ; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[j][e] = fa[j][e];
    if (mine < steps) __builtin_amdgcn_s_barrier();      // (an odd number of stages: the other half has the last one)
  } else {
    for (int step = 0; step < steps; step++) {
      const int s = 2 * step + kh;
      wait_copies<COPIES>();                               // this wave's copies of stage s have landed, and (barrier) all
      __builtin_amdgcn_s_barrier();                        // waves'; stage s - 2 has been read by all of them
      asm volatile("" ::: "memory");
      int fill = cur + 2 * SLOT;
      if (fill >= 3 * SLOT) fill -= 3 * SLOT;
      if constexpr (!SPREAD) issue(s + 4, fill, 0, COPIES);
      if (s >= nst) break;                                 // (an odd number of stages: the other half has the last one)
      const bool half_stage = short_last && s == nst - 1;
      const unsigned char* sp = smem + kh * (NBUF * SLOT) + cur;
      const unsigned char* sc_p = sp + X_BYTES + W_BYTES + w * 256;
      float sc[GPS];
#pragma unroll
      for (int jj = 0; jj < GPS; jj++) sc[jj] = scales.read(sc_p + jj * 128, group(s, jj), c);
      const unsigned char* wp = sp + X_BYTES + w * 1024 + c * 32;
      bf16x8 b[4];
      if constexpr (GS == 32) {
        const uint4 lo = *(const uint4*)(wp + (swz << 4)), hi = *(const uint4*)(wp + ((1 ^ swz) << 4));
        b[0] = decode(h ? lo.y : lo.x);
        b[1] = decode(h ? lo.w : lo.z);
        b[2] = decode(h ? hi.y : hi.x);
        b[3] = decode(h ? hi.w : hi.z);
      } else {
        const uint4 p = *(const uint4*)(wp + ((h ^ swz) << 4));
        b[0] = decode(p.x);
        b[1] = decode(p.y);
        b[2] = decode(p.z);
        b[3] = decode(p.w);
      }
      bf16x8 a[2][4];
#pragma unroll
      for (int ks = 0; ks < 4; ks++) a[0][ks] = *(const bf16x8*)(sp + ln_x[ks]);
      f32x16 I[2][GPS];
#pragma unroll
      for (int j = 0; j <= NJ; j++) {
        if (j < NJ - 1)
#pragma unroll
          for (int ks = 0; ks < 4; ks++) a[(j + 1) & 1][ks] = *(const bf16x8*)(sp + ln_x[ks] + (j + 1) * (32 * 128));
        if (j < NJ) {
#pragma unroll
          for (int jj = 0; jj < GPS; jj++) {
            f32x16 z;
#pragma unroll
            for (int v = 0; v < 16; v++) z[v] = 0.0f;
#pragma unroll
            for (int ks = jj * (4 / GPS); ks < (jj + 1) * (4 / GPS); ks++)
              z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j & 1][ks], b[ks], z, 0, 0, 0);
            I[j & 1][jj] = z;
          }
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (SPREAD) {                          // a share of the copies of stage s + 4
            issue(s + 4, fill, j * COPIES / NJ, (j + 1) * COPIES / NJ);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (j > 0) {
#pragma unroll
          for (int jj = 0; jj < GPS; jj++)
            if (jj == 0 || !half_stage)                    // (not 0 x: an infinity would become a NaN)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[j - 1][v] = fmaf(I[(j - 1) & 1][jj][v], sc[jj], acc[j - 1][v]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      cur = cur + SLOT >= 3 * SLOT ? 0 : cur + SLOT;
    }
  }
  wait_copies<0>();                                      // (nothing may land in LDS after the workgroup has ended)

  finish<OUT_F32, NJ>(acc, smem, kh, w, m0, n0, bias, M, N, y);
}

template <int GS, bool OUT_F32, int NJ>
static int launch_large_one(const uint16_t* x, const void* blob, const uint16_t* bias, int M, int N, int K, void* y,
                        hipStream_t s) {
  const BlobLayout L = blob_layout(N, K, 0, GS);
  const char* bp = (const char*)blob;
  constexpr int TM_ = 32 * NJ, SMEM = smem_bytes(128, NJ);
  const int n_mt = (M + TM_ - 1) / TM_, n_nt = (N + TN_ - 1) / TN_;
  const long n_blocks = (long)n_mt * n_nt;
  const int per_xcd = (int)((n_blocks + 7) / 8);
  // (idempotent: two threads racing here would both set the same attribute)
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)w4a16_large_kernel<GS, OUT_F32, NJ>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return hip_failed(e);
    attr_done.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((w4a16_large_kernel<GS, OUT_F32, NJ>), dim3(per_xcd * 8), dim3(NT), SMEM, s, x,
                     (const uint8_t*)(bp + L.off_codes), (const uint16_t*)(bp + L.off_sw), bias, M, N, K, y, n_mt, n_nt,
                     per_xcd);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

template <int GS, bool OUT_F32>
static int launch_large(const uint16_t* x, const void* blob, const uint16_t* bias, int M, int N, int K, void* y, int nj,
                        hipStream_t s) {
  switch (nj) {
    case 1: return launch_large_one<GS, OUT_F32, 1>(x, blob, bias, M, N, K, y, s);
    case 2: return launch_large_one<GS, OUT_F32, 2>(x, blob, bias, M, N, K, y, s);
    case 4: return launch_large_one<GS, OUT_F32, 4>(x, blob, bias, M, N, K, y, s);
    default: return launch_large_one<GS, OUT_F32, 5>(x, blob, bias, M, N, K, y, s);
  }
}

}  // namespace w16

// ---- up to 8 tokens: every weight is used once, so the kernel is a stream over the packed weights.
// One workgroup (8 waves) = 32 output channels.  K is walked in chunks of 1024 channels:
// the chunk's codes (32 rows x 512 B), activations (8 rows x 2 KB)
// and scales go through registers into one of two LDS buffers, every thread loading consecutive 16-byte
// pieces of a row, while the waves multiply the previous chunk (wave w takes scale groups w, w + 8, ...).
// Orientation D[token][n]: the activations are the row operand of the 32x32x16 MFMA (tokens padded to 32 by
// re-reading the last one), a lane owns one output channel, so the group's weight scale is a per-lane
// scalar; lane half h holds channels [h GS/2, (h + 1) GS/2) of the group.  LDS rows are padded by 16 bytes
// so that the 32 lanes of an operand read hit different banks.  Within each run of 8 channels both
// operands are kept in the order c0 c2 c4 c6 c1 c3 c5 c7 (the activations are permuted once when they
// are staged), which saves the last round of byte permutes of the weight decode.  The 8 waves' partial
// sums are added through LDS in wave order.
// Bound: the decode and the staging beside it, not the stream: a second or third chunk in flight makes it slower (four layers' weights
// in turn, one token, K = 3072, N = 9216: 8.4 -> 8.8, 9.4 us).  Activation rows past M are not stored to LDS (8.4 -> 8.15) and the
// decode is the scaled conversion instead of byte tables (8.15 -> 7.6).  Both, us: K = 12288, N = 3072 16.4 -> 14.4; 3072,
// 3072 5.6 -> 5.1; 6144, 12288 13.9 -> 12.4; 8 tokens, 3072, 9216 8.6 -> 8.1.
struct Eight {
  static constexpr int MT = 8, KC = 1024;           // token capacity, channels per chunk
  static constexpr int WROW = KC / 2 + 16;          // bytes per LDS row of codes
  static constexpr int XROW = KC * 2 + 16;          // bytes per LDS row of activations
  static constexpr int CODES_B = 32 * WROW;
  static constexpr int X_B = MT * XROW;
  static constexpr int NV = MT / 2;                 // accumulator registers that hold real tokens (of 16)
  static constexpr int buf_bytes(int gs) { return CODES_B + X_B + (KC / gs) * 32 * 2; }
  static constexpr int smem_bytes(int gs) { return 2 * buf_bytes(gs) > 8 * NV * 256 ? 2 * buf_bytes(gs) : 8 * NV * 256; }
};

// 8 sign-magnitude nibbles -> bf16 in the order c0 c2 c4 c6 c1 c3 c5 c7 (10 instructions)
__device__ __forceinline__ uint4 nibbles_to_bf16_eo(uint32_t p) {
  uint32_t e, o;
  unpack8(p, e, o);
  uint4 r;                                               // bytes [s 0000 mmm] = m 2^-9 as fp8, times 2^9
  r.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(e, 512.0f, false));   // c0, c2
  r.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(e, 512.0f, true));    // c4, c6
  r.z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(o, 512.0f, false));   // c1, c3
  r.w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(o, 512.0f, true));    // c5, c7
  return r;
}

template <int GS, bool OUT_F32>
__global__ __launch_bounds__(512) void w4a16_eight_kernel(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ wq, const uint16_t* __restrict__ sw,
    const uint16_t* __restrict__ bias, int M, int N, int K, void* __restrict__ y, int sw_shift) {
  static_assert(GS == 32 || GS == 64, "scale granularity");
  using F = Eight;
  constexpr int MT = F::MT, KC = F::KC, STEPS = GS / 16, GPC = KC / GS, BUF = F::buf_bytes(GS), NV = F::NV;
  constexpr int CPT = KC / 512;                 // 16-byte code pieces per thread and chunk (32 rows x KC/32 pieces)
  constexpr int XPT = MT * (KC / 8) / 512;      // 16-byte activation pieces per thread and chunk
  constexpr int SPT = (GPC * 32 + 511) / 512;   // scales per thread and chunk
  extern __shared__ __align__(16) unsigned char smem[];
  const int t = threadIdx.x, l = t & 63, w = t >> 6, h = l >> 5, c = l & 31;
  const int n0 = blockIdx.x * 32, n = n0 + c;
  const int mrow = min(c, M - 1);
  const int nch = (K + KC - 1) / KC;

  // staging roles of this thread within a chunk: piece index t + 512 i over (row, 16-byte piece of the row)
  int crow[CPT], cpiece[CPT], xrow[XPT], xpiece[XPT];
  const uint8_t* gc[CPT];
  const uint16_t* gx[XPT];
#pragma unroll
  for (int i = 0; i < CPT; i++) {
    const int idx = t + 512 * i;
    crow[i] = idx / (KC / 32), cpiece[i] = idx % (KC / 32);
    gc[i] = wq + (size_t)min(n0 + crow[i], N - 1) * (K / 2) + cpiece[i] * 16;
  }
#pragma unroll
  for (int i = 0; i < XPT; i++) {
    const int idx = t + 512 * i;
    xrow[i] = idx / (KC / 8), xpiece[i] = idx % (KC / 8);
    gx[i] = x + (size_t)min(xrow[i], M - 1) * K + xpiece[i] * 8;
  }
  const uint16_t* gsc = sw + min(n0 + (t & 31), N - 1);       // scale (group (t + 512 i) / 32, channel t % 32)

  uint4 rc[CPT], rx[XPT];
  uint32_t rs[SPT] = {};
  auto gload = [&](int ch) {
    const int k0 = ch * KC;
#pragma unroll
    for (int i = 0; i < CPT; i++)
      rc[i] = k0 + cpiece[i] * 32 < K ? *(const uint4*)(gc[i] + k0 / 2) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < XPT; i++)
      rx[i] = (k0 + xpiece[i] * 8 < K && xrow[i] < M) ? *(const uint4*)(gx[i] + k0) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < SPT; i++) {
      const int sg = (t + 512 * i) >> 5, j = ch * GPC + sg;
      if (sg < GPC && j < K / GS) rs[i] = gsc[(size_t)(j >> sw_shift) * N];
    }
  };
  auto sstore = [&](int buf) {
    unsigned char* sb = smem + buf * BUF;
#pragma unroll
    for (int i = 0; i < CPT; i++) *(uint4*)(sb + crow[i] * F::WROW + cpiece[i] * 16) = rc[i];
#pragma unroll
    for (int i = 0; i < XPT; i++) {
      if (__builtin_amdgcn_readfirstlane(xrow[i]) >= M) continue;   // (nobody reads it; a wave's pieces are of one row)
      uint4 v;                                            // c0c1 c2c3 c4c5 c6c7 -> c0c2 c4c6 c1c3 c5c7
      v.x = __builtin_amdgcn_perm(rx[i].y, rx[i].x, 0x05040100u);
      v.y = __builtin_amdgcn_perm(rx[i].w, rx[i].z, 0x05040100u);
      v.z = __builtin_amdgcn_perm(rx[i].y, rx[i].x, 0x07060302u);
      v.w = __builtin_amdgcn_perm(rx[i].w, rx[i].z, 0x07060302u);
      *(uint4*)(sb + F::CODES_B + xrow[i] * F::XROW + xpiece[i] * 16) = v;
    }
#pragma unroll
    for (int i = 0; i < SPT; i++) {
      const int sg = (t + 512 * i) >> 5;
      if (sg < GPC) ((uint16_t*)(sb + F::CODES_B + F::X_B))[sg * 32 + (t & 31)] = (uint16_t)rs[i];
    }
  };

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; v++) acc[v] = 0.0f;

  gload(0);
  sstore(0);
  __syncthreads();
  for (int ch = 0; ch < nch; ch++) {
    const bool more = ch + 1 < nch;
    if (more) gload(ch + 1);                              // in flight while this chunk is multiplied
    const unsigned char* sb = smem + (ch & 1) * BUF;
    const int groups = min(GPC, (K - ch * KC) / GS);
    for (int gi = w; gi < groups; gi += 8) {
      uint32_t cw[STEPS];
      if constexpr (GS == 64) {
        const uint4 v = *(const uint4*)(sb + c * F::WROW + gi * 32 + h * 16);
        cw[0] = v.x, cw[1] = v.y, cw[2] = v.z, cw[3] = v.w;
      } else {
        const uint2 v = *(const uint2*)(sb + c * F::WROW + gi * 16 + h * 8);
        cw[0] = v.x, cw[1] = v.y;
      }
      const unsigned char* xs = sb + F::CODES_B + mrow * F::XROW + (gi * GS + h * (GS / 2)) * 2;
      f32x16 z;
#pragma unroll
      for (int v = 0; v < 16; v++) z[v] = 0.0f;
#pragma unroll
      for (int s2 = 0; s2 < STEPS; s2++) {
        const bf16x8 xa = *(const bf16x8*)(xs + s2 * 16);
        const uint4 wv = nibbles_to_bf16_eo(cw[s2]);
        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa, __builtin_bit_cast(bf16x8, wv), z, 0, 0, 0);
      }
      const float sf = f16_bits_to_f32(((const uint16_t*)(sb + F::CODES_B + F::X_B))[gi * 32 + c]);
      // accumulator register v holds token 8 (v / 4) + 4 h + v % 4: the first NV cover tokens 0 .. MT-1
#pragma unroll
      for (int v = 0; v < NV; v++) acc[v] = fmaf(z[v], sf, acc[v]);
    }
    if (more) sstore((ch + 1) & 1);
    __syncthreads();
  }
  // partial sums of the 8 waves, added in wave order: red[wave][register][lane]
  float* red = (float*)smem;
#pragma unroll
  for (int v = 0; v < NV; v++) red[(w * NV + v) * 64 + l] = acc[v];
  __syncthreads();
  const int m = 4 * h + w;                                // wave w < 4: register w, tokens w and 4 + w
  if (n < N && w < NV && m < M) {
    const float b = bias ? bf16_bits_to_f32(bias[n]) : 0.0f;
    float r = red[w * 64 + l];
#pragma unroll
    for (int p2 = 1; p2 < 8; p2++) r += red[(p2 * NV + w) * 64 + l];
    r += b;
    if (OUT_F32) ((float*)y)[(size_t)m * N + n] = r;
    else ((uint16_t*)y)[(size_t)m * N + n] = f32_to_bf16_bits(r);
  }
}

template <int GS, bool OUT_F32>
static int launch_eight(const uint16_t* x, const void* blob, const uint16_t* bias, int M, int N, int K, int g, void* y,
                        hipStream_t s) {
  const BlobLayout L = blob_layout(N, K, 0, g);
  const char* bp = (const char*)blob;
  constexpr int SMEM = Eight::smem_bytes(GS);
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)w4a16_eight_kernel<GS, OUT_F32>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return hip_failed(e);
    attr_done.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((w4a16_eight_kernel<GS, OUT_F32>), dim3((N + 31) / 32), dim3(512), SMEM, s, x,
                     (const uint8_t*)(bp + L.off_codes), (const uint16_t*)(bp + L.off_sw), bias, M, N, K, y,
                     g == 2 * GS ? 1 : 0);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

// ---- 9 to 32 tokens: the same stream.  One workgroup (8 waves) = 32 output channels, or 48 (a second MFMA tile of which 16
// lanes are real) where 32 leave some CUs two workgroups and 48 do not (32 tokens, K = 3072, N = 9216 on 256 CUs: 13.9 ->
// 10.7 us).  K is walked in panels of 512 channels: codes, activations and scales come by global-to-LDS copies of whole
// lines into a ring of up to four panels, all of them in flight from the start, and the waves multiply a panel's scale
// groups in turn (wave w takes groups w, w + 8, ...).  Orientation as above.  The 8 waves' partial sums are added through LDS
// in wave order.
// Bound: launch (1.7 us), the copies, one memory latency and the decode.  Through registers into two buffers, with the next
// panel's 32 to 64 KB in flight, -> now, us, one layer's weights again and again | four layers' in turn: K = 3072, N = 9216: 12
// tokens 13.7 -> 9.4 | 14.4 -> 10.1, 32: 14.7 -> 9.7 | 15.9 -> 10.3; N = 3072, 16: 7.6 -> 6.9 | 7.8 -> 7.0; K = 12288, N = 3072,
// 20 tokens 23.8 -> 20.4 | 24.3 -> 20.6.  Of this 0.2 to 0.3 us came from leaving out copies of codes and scales that nobody read.
template <int NCH>
struct Few {
  static constexpr int KC = 512;                          // channels per panel
  static constexpr int CROW = KC / 2, XROW = KC * 2;      // bytes per row of codes and of activations
  static constexpr int CT = (NCH + 31) / 32;              // column tiles
  // Copies per panel: codes, 4 rows each, and scales, of one or two groups, by the last waves; every wave has as many.
  // (48 channels and groups of 32: four waves would be one short; they copy the last row again, which is 3% faster than
  // counting two kinds of waves or splitting the scales: 32 tokens, K = 3072, N = 9216 12.1 against 12.5 us.)
  static constexpr int codes(int gs) { return NCH == 48 && gs == 32 ? 16 : NCH * CROW / 1024; }
  static constexpr int per_copy(int gs) { return NCH == 32 && gs == 64 ? 1 : 2; }
  static constexpr int sc(int gs) { return KC / gs / per_copy(gs); }
  static constexpr int share(int gs) { return (codes(gs) + sc(gs)) / 8; } // copies of codes and scales of a wave
  static constexpr int scales_at(int gs) { return codes(gs) * 1024; }
  static constexpr int x_at(int gs) { return scales_at(gs) + sc(gs) * 256; }
  static constexpr int panel_bytes(int gs, int xc) { return x_at(gs) + xc * 8192; }
};

// XC: copies of activations per wave and panel (8 rows by all waves)
template <int GS, bool OUT_F32, int NCH, int XC>
__global__ __launch_bounds__(512) void w4a16_few_kernel(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ wq, const uint16_t* __restrict__ sw,
    const uint16_t* __restrict__ bias, int M, int N, int K, void* __restrict__ y, int sw_shift, int nbuf) {
  static_assert(GS == 32 || GS == 64, "scale granularity");
  using F = Few<NCH>;
  constexpr int CT = F::CT;
  constexpr int KC = F::KC, STEPS = GS / 16, GPC = KC / GS, NV = 16, PANEL = F::panel_bytes(GS, XC), SC = F::sc(GS);
  constexpr int CPP = F::CROW / 16, XPP = F::XROW / 16;   // 16-byte pieces per row
  constexpr int CODES = F::codes(GS), SHARE = F::share(GS), PER_COPY = F::per_copy(GS);
  static_assert(SC <= 8 && (CODES + SC) % 8 == 0, "shares of the waves");
  extern __shared__ __align__(16) unsigned char smem[];
  const int t = threadIdx.x, l = t & 63, h = l >> 5, c = l & 31;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n0 = blockIdx.x * NCH;
  const int np = (K + KC - 1) / KC, G = K / GS;           // (stored groups hold GS << sw_shift channels)
  const uint32_t lds = lds_address(smem);
  const halves::ScaleRows scales = {(const unsigned char*)sw, ((size_t)(((G - 1) >> sw_shift) + 1) * N * 2 - 1) & ~(size_t)3, N, n0};
  const unsigned char* wb = wq + (size_t)n0 * (K / 2);
  // Panel p into the ring slot at `at`.  Piece q of code row `row` sits at q ^ (row & 15), of activation row `row` at q ^ (row &
  // 7): rows that are read together start in different banks.  What lies past the end of a row, past the last row or
  // the last group is read from inside, unused.
  const bool has_x = w * XC * 1024 < M * F::XROW;           // (this wave's copies of activations are of real rows)
  auto wait_panel = [&](auto behind) {                    // until only the copies of `behind` later panels are in flight
    constexpr int B = decltype(behind)::value;
    if (has_x) wait_copies<B * (SHARE + XC)>();
    else wait_copies<B * SHARE>();
  };
  auto issue = [&](int p, uint32_t at) {
    const int last = (K - p * KC) / 32 - 1;               // last piece of codes in this panel's rows (may be past its end)
#pragma unroll
    for (int i = 0; i < (CODES + 7) / 8; i++) {
      const int k = CODES % 8 == 0 ? w * (CODES / 8) + i : w + 8 * i, row = (k * 64 + l) / CPP, q = l % CPP ^ (row & 15);
      if (CODES % 8 == 0 || k < CODES)
        copy_to_lds(lds + at + k * 1024, (uint32_t)min(min(row, NCH - 1), N - 1 - n0) * (uint32_t)(K / 2) + min(q, last) * 16, wb + (size_t)p * F::CROW);
    }
    if (SC == 8 || w >= 8 - SC) {
      const int k = w - (8 - SC), g0 = min(p * GPC + PER_COPY * k, G - 1), g1 = min(p * GPC + PER_COPY * k + 1, G - 1);
      scales.copy<PER_COPY == 2, NCH == 32 ? 20 : 28>(lds + at + F::scales_at(GS) + k * 256, g0 >> sw_shift, g1 >> sw_shift);
    }
    const int xlast = 4 * last + 3;
    if (!has_x) return;
#pragma unroll
    for (int i = 0; i < XC; i++) {
      const int f = (w * XC + i) * 64 + l, row = f / XPP, q = (f % XPP) ^ (row & 7);
      copy_to_lds(lds + at + F::x_at(GS) + (w * XC + i) * 1024, (uint32_t)min(row, M - 1) * (uint32_t)(2 * K) + min(q, xlast) * 16,
                  (const unsigned char*)x + (size_t)p * F::XROW);
    }
  };
  f32x16 acc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ct++)
#pragma unroll
    for (int v = 0; v < 16; v++) acc[ct][v] = 0.0f;
  for (int p = 0; p < nbuf; p++)
    if (p < np) issue(p, p * PANEL);
  const int mrow = min(c, M - 1);
  int cur = 0;
  for (int p = 0; p < np; p++) {
    // this wave's copies of panel p have landed, and (barrier) all waves'; panel p - 1 has been read by all of them
    const int behind = min(np - 1 - p, p == 0 ? nbuf - 1 : nbuf - 2);
    if (behind <= 0) wait_panel(std::integral_constant<int, 0>{});
    else if (behind == 1) wait_panel(std::integral_constant<int, 1>{});
    else if (behind == 2) wait_panel(std::integral_constant<int, 2>{});
    else wait_panel(std::integral_constant<int, 3>{});
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (p > 0 && p - 1 + nbuf < np) issue(p - 1 + nbuf, (cur == 0 ? nbuf - 1 : cur - 1) * PANEL);
    const unsigned char* sb = smem + cur * PANEL;
    const int groups = min(GPC, (K - p * KC) / GS);
    for (int gi = w; gi < groups; gi += 8) {
      const unsigned char* xs = sb + F::x_at(GS) + mrow * F::XROW;
      bf16x8 xa[STEPS];
#pragma unroll
      for (int s2 = 0; s2 < STEPS; s2++) xa[s2] = *(const bf16x8*)(xs + (((gi * (GS / 8) + h * (GS / 16) + s2) ^ (mrow & 7)) << 4));
      const int j = (p * GPC + gi) >> sw_shift;
#pragma unroll
      for (int ct = 0; ct < CT; ct++) {
        const int row = ct * 32 + (ct + 1 == CT && NCH % 32 != 0 ? c & 15 : c);   // (lanes past the last channel: one of the others)
        uint32_t cw[STEPS];
        if constexpr (GS == 64) {
          const uint4 v = *(const uint4*)(sb + row * F::CROW + (((2 * gi + h) ^ (row & 15)) << 4));
          cw[0] = v.x, cw[1] = v.y, cw[2] = v.z, cw[3] = v.w;
        } else {
          const uint2 v = *(const uint2*)(sb + row * F::CROW + ((gi ^ (row & 15)) << 4) + 8 * h);
          cw[0] = v.x, cw[1] = v.y;
        }
        f32x16 z;
#pragma unroll
        for (int v = 0; v < 16; v++) z[v] = 0.0f;
#pragma unroll
        for (int s2 = 0; s2 < STEPS; s2++) z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[s2], w16::decode(cw[s2]), z, 0, 0, 0);
        const float sf = scales.read(sb + F::scales_at(GS) + (PER_COPY == 2 ? (gi >> 1) * 256 + (gi & 1) * 128 : gi * 256), j, row);
        // accumulator register v holds token 8 (v / 4) + 4 h + v % 4
#pragma unroll
        for (int v = 0; v < NV; v++) acc[ct][v] = fmaf(z[v], sf, acc[ct][v]);
      }
    }
    cur = cur + 1 == nbuf ? 0 : cur + 1;
  }
  // partial sums of the 8 waves, added in wave order: red[wave][register][lane]
  constexpr int RPW = NV / 8;                             // registers finished by each wave
  float* red = (float*)smem;
#pragma unroll
  for (int ct = 0; ct < CT; ct++) {
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NV; v++) red[(w * NV + v) * 64 + l] = acc[ct][v];
    __syncthreads();
    const int n = n0 + ct * 32 + c;
    if (n < N && ct * 32 + c < NCH) {
      const float b = bias ? bf16_bits_to_f32(bias[n]) : 0.0f;
#pragma unroll
      for (int e = 0; e < RPW; e++) {
        const int v = w * RPW + e, m = 8 * (v >> 2) + 4 * h + (v & 3);
        if (m < M) {
          float r = red[v * 64 + l];
#pragma unroll
          for (int p2 = 1; p2 < 8; p2++) r += red[(p2 * NV + v) * 64 + l];
          r += b;
          if (OUT_F32) ((float*)y)[(size_t)m * N + n] = r;
          else ((uint16_t*)y)[(size_t)m * N + n] = f32_to_bf16_bits(r);
        }
      }
    }
  }
}

template <int GS, bool OUT_F32, int NCH, int XC>
static int launch_few16(const uint16_t* x, const void* blob, const uint16_t* bias, int M, int N, int K, int g, void* y, int cus,
                        hipStream_t s) {
  const BlobLayout L = blob_layout(N, K, 0, g);
  const char* bp = (const char*)blob;
  constexpr int KC = Few<NCH>::KC, PANEL = Few<NCH>::panel_bytes(GS, XC), RED = 8 * 16 * 256;
  static_assert(2 * PANEL >= RED && 2 * PANEL <= 160 * 1024, "LDS");
  // up to four panels; more than one workgroup per CU: as many as leave room for two, at least two
  const int wgs = (N + NCH - 1) / NCH;
  int nbuf = std::min(4, 160 * 1024 / PANEL);
  if (wgs > cus) nbuf = std::min(nbuf, std::max(2, 80 * 1024 / PANEL));
  nbuf = std::max(2, std::min(nbuf, (K + KC - 1) / KC));
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)w4a16_few_kernel<GS, OUT_F32, NCH, XC>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, std::min(4, 160 * 1024 / PANEL) * PANEL);
    if (e != hipSuccess) return hip_failed(e);
    attr_done.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((w4a16_few_kernel<GS, OUT_F32, NCH, XC>), dim3(wgs), dim3(512), nbuf * PANEL, s, x,
                     (const uint8_t*)(bp + L.off_codes), (const uint16_t*)(bp + L.off_sw), bias, M, N, K, y,
                     g == 2 * GS ? 1 : 0, nbuf);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

template <int GS, bool OUT_F32>
static int launch_few(const uint16_t* x, const void* blob, const uint16_t* bias, int M, int N, int K, int g, void* y, int cus,
                      hipStream_t s) {
  const bool wide = w16::few_channels(N, cus) == 48;
#define DIROTQ_FEW16(XC)                                                                  \
  return wide ? launch_few16<GS, OUT_F32, 48, XC>(x, blob, bias, M, N, K, g, y, cus, s)   \
              : launch_few16<GS, OUT_F32, 32, XC>(x, blob, bias, M, N, K, g, y, cus, s)
  if (M <= 8) return launch_eight<GS, OUT_F32>(x, blob, bias, M, N, K, g, y, s);
  if (M <= 16) DIROTQ_FEW16(2);
  DIROTQ_FEW16(4);
#undef DIROTQ_FEW16
}

int launch_w4a16_gemm(const uint16_t* x, const void* blob, const uint16_t* bias, int M, int N, int K, int g, void* y,
                      int y_dtype, hipStream_t s) {
  int dev = 0, cus = 256;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return hip_failed(e);
  auto few = [&](const uint16_t* xs, void* ys, int Ms) -> int {   // up to 32 tokens
    if (g == 32)
      return y_dtype ? launch_few<32, true>(xs, blob, bias, Ms, N, K, g, ys, cus, s)
                     : launch_few<32, false>(xs, blob, bias, Ms, N, K, g, ys, cus, s);
    return y_dtype ? launch_few<64, true>(xs, blob, bias, Ms, N, K, g, ys, cus, s)
                   : launch_few<64, false>(xs, blob, bias, Ms, N, K, g, ys, cus, s);
  };
  // few tokens: the weight stream, not the matrix pipe, is the bound
  if (M <= 32) return few(x, y, M);
  int nj = w16::token_tiles(M, N, K, g, cus);
  bool two_few = w16::two_few_launches(M, N, K, g, cus);
  // DIROTQ_W4A16_KERNEL=few (33 to 64 tokens) / tile / tile1 / tile2 / tile4 / tile5 in the environment forces one of the two,
  // the tiles with the rule's or that number of token tiles per workgroup (the tests use it to run all on the same inputs)
  if (const char* f = getenv("DIROTQ_W4A16_KERNEL")) {
    if (!strcmp(f, "few")) two_few = M <= 64;
    if (!strncmp(f, "tile", 4)) two_few = false;
    for (int c : {1, 2, 4, 5})
      if (!strncmp(f, "tile", 4) && f[4] == '0' + c && !f[5]) nj = c;
  }
  if (two_few) {
    const int st = few(x, y, 32);
    return st ? st : few(x + (size_t)32 * K, (char*)y + (size_t)32 * N * (y_dtype ? 4 : 2), M - 32);
  }
  switch (g) {
    case 32: return y_dtype ? w16::launch_large<32, true>(x, blob, bias, M, N, K, y, nj, s)
                            : w16::launch_large<32, false>(x, blob, bias, M, N, K, y, nj, s);
    case 64: return y_dtype ? w16::launch_large<64, true>(x, blob, bias, M, N, K, y, nj, s)
                            : w16::launch_large<64, false>(x, blob, bias, M, N, K, y, nj, s);
    case 128: return y_dtype ? w16::launch_large<128, true>(x, blob, bias, M, N, K, y, nj, s)
                             : w16::launch_large<128, false>(x, blob, bias, M, N, K, y, nj, s);
  }
  return DIROTQ_ERR_UNSUPPORTED;
}

}  // namespace dirotq
