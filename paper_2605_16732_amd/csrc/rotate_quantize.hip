// Kernel A: online rotation x_hat = x Q (bf16 MFMA, fp32 accumulate) with the
// split / per-group quantize / pack fused into the GEMM epilogue (rotation/split
// equation of Section 4.2 and the quantizer of Section 3 of the paper).
//
// Orientation.  The product is computed transposed, D[channel][token] =
// sum_k Qt[channel][k] x[token][k]: both operands stream K-contiguous rows, and in the
// 32x32 MFMA accumulator layout a lane then owns ONE token and 4 consecutive rotated
// channels per register quad.  A wave computes 128 channels x 32 tokens (64 with the 16x16 MFMA), so every
// quantization group (32, 64 or 128 channels of one token) lives in one lane pair
// (l, l^32): the absmax is an in-lane max plus one cross-lane exchange, the codes are
// packed in registers, and nothing is staged through LDS after the main loop.
//
// Channel tiling.  Waves own 128 "virtual" channels: the bf16 part [0, r), then the 4-bit part
// [r, K) from virtual channel r_pad on, placed so that groups never straddle a wave: r_pad = r when
// r is a multiple of the group size (the wave that holds the split point then stores both kinds),
// else r rounded up to 128.
//
// Main loop.  Operand tiles are staged HBM -> registers -> LDS (two LDS stages) with an
// XOR swizzle applied on the global side, so that the 16-byte MFMA operand reads of 16
// consecutive rows are bank-conflict free.  While stage kt is multiplied, the registers
// holding stage kt+1 (loaded during stage kt-1) are written to the other LDS stage and
// refilled with stage kt+2; every store/load pair sits between MFMAs.  (With one or two waves of
// 128 x 64 outputs per SIMD this beats global_load_lds, which holds its wave up longer than a register load plus
// an LDS store; more and smaller waves turn it round: rotate_quantize_dma.hip.)  A last stage of 32 channels
// (K = 32 mod 64) gets zeros for its upper half; stages of 32 channels throughout, us: M = 4608, K = 3104 112 against 86;
// M = 32768, K = 1184 130 against 108; M = 3000, K = 6176 312 against 243.
#include <atomic>

#include "rotate_epilogue.h"

namespace dirotq {

// KSP = 2: the workgroup holds two such sets of waves, each with LDS stages of its own, and each walks one half of
// K; the halves' accumulators are added through LDS before the epilogue (small launches: half as long a chain of
// stage latencies).
template <int WGC, int WGT, int MI, int KSP = 1>
struct RQ {
  static constexpr int BK = 64;                            // channels per stage
  static constexpr int WAVE_C = 128, WAVE_T = MI == 32 ? 32 : 64;   // wave tile: channels x tokens (the small launches, with the
                                                           // 32x32 MFMA: half the arithmetic per wave and stage)
  static constexpr int TC = WGC * WAVE_C, TT = WGT * WAVE_T;
  static constexpr int NW = WGC * WGT, NT = NW * KSP * 64; // waves per k-part, threads per workgroup
  static constexpr int ROWB = BK * 2;                      // bytes per LDS row
  static constexpr int CPR = ROWB / 16;                    // 16-B chunks per row
  static constexpr int STAGE_BYTES = (TC + TT) * ROWB;
  static constexpr int IPW = (TC + TT) * CPR / 64 / NW;    // 16-B loads per lane per stage
  static constexpr int KS = BK / 16;                       // MFMA k-steps per stage
  static constexpr int PP = IPW / KS;                      // store/load pairs per k-step
  static constexpr int SMEM = KSP * 2 * STAGE_BYTES;
  // register budget: two waves per SIMD unless LDS (160 KB per CU) admits only one 4-wave workgroup
  static constexpr int WAVES_PER_SIMD = (NW * KSP <= 4 && 2 * SMEM > 160 * 1024) ? 1 : 2;
  static_assert(KSP == 1 || (KSP == 2 && SMEM >= NW * 64 * (WAVE_C * WAVE_T / 64) * 4), "the second part's accumulators pass through the stage buffers");
  static_assert((TC + TT) * CPR % (64 * NW) == 0, "loads must divide evenly over waves");
  static_assert(IPW % KS == 0 && PP >= 1 && PP <= 4, "store/load pairs are spread over the 4 MFMA rows of a k-step");

  // chunk c of row `row` is stored in 16-B slot c ^ swz(row)
  // (LDS has 64 banks: a 16-byte read is served 16 lanes per cycle, so 16 consecutive rows
  // must land in 16 different 16-byte slots of a 256-byte bank line: row&1 picks the half line,
  // (row>>1)&7 permutes the 8 chunks)
  __device__ static __forceinline__ int swz(int row) { return (row >> 1) & 7; }
};

// what a last stage of 32 channels (K = 32 mod 64) has in the place of its upper half
static __device__ const uint4 kZeros = {0, 0, 0, 0};

// QM selects what happens to the channels [r, K): 0 = symmetric 4-bit per-group quantizer,
// 1 = asymmetric one (zero-point min, 16 unsigned levels; zx receives the zero-points, laid out
// like sx), 2 = no quantizer here: the fp32 values go to xf [M][K-r] and the absolute maximum of
// every 128-channel wave tile to pmax [ceil((K-r)/128)][M] (per-token 8-bit quantization needs the
// maximum over all channels of a token, which no single workgroup sees).
template <int WGC, int WGT, int MI, int QM, int KSP, bool TAIL>
__global__ __launch_bounds__(WGC* WGT* KSP * 64, (RQ<WGC, WGT, MI, KSP>::WAVES_PER_SIMD)) void rotate_quantize_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ Qt, int M, int K, int r, int g,
    uint16_t* __restrict__ xh, uint8_t* __restrict__ xl, uint16_t* __restrict__ sx, uint16_t* __restrict__ zx,
    float* __restrict__ xf, float* __restrict__ pmax, int r_pad, int Kv, int n_ct, int n_tt, int per_xcd, int sx_ld,
    bool fields) {
  using C = RQ<WGC, WGT, MI, KSP>;
  constexpr int BK = C::BK;
  static_assert(KSP == 1 || MI == 32, "the K split is written for the 32x32 loop only");
  constexpr bool ASYM = QM == 1;
  extern __shared__ __align__(16) unsigned char smem_all[];

  // consecutive workgroup ids go to different XCDs; give each XCD a contiguous run of tiles
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= n_ct * n_tt) return;
  // within an XCD's run, sweep GC channel tiles per token tile so that co-resident
  // workgroups share both operands through the XCD's L2
  constexpr int GC = 4;
  const int grp = logical / (GC * n_tt), in_grp = logical % (GC * n_tt);
  const int gc = min(n_ct - grp * GC, GC);
  const int ct = grp * GC + in_grp % gc, tt = in_grp / gc;
  const int m0 = tt * C::TT;

  const int t = threadIdx.x, l = t & 63;
  const int w = (t >> 6) % C::NW, kp = (t >> 6) / C::NW;    // wave within its k-part, k-part
  const int wc = w % WGC, wt = w / WGC;
  unsigned char* const smem = smem_all + kp * (2 * C::STAGE_BYTES);   // the k-part's own two stages

  // ---- per-lane source pointers of this wave's loads ---------------------------------
  // load q of wave w fills LDS bytes [(w*IPW+q)*1024, +1024) of a stage: rows are the TC
  // channel rows followed by the TT token rows.  Rows past the edge re-read a valid row; their
  // results are discarded in the epilogue.
  const uint16_t* gsrc[C::IPW];
#pragma unroll
  for (int i = 0; i < C::IPW; i++) {
    const int ci = (w * C::IPW + i) * 64 + l;               // chunk index within the stage
    const int row = ci / C::CPR, phys = ci % C::CPR;
    const int logical_chunk = phys ^ C::swz(row);
    const uint16_t* base;
    if (row < C::TC) {
      const int v = ct * C::TC + row;                       // virtual channel
      int ch = v < r_pad ? min(v, r - 1) : min(r + (v - r_pad), K - 1);
      ch = max(ch, 0);
      base = Qt + (size_t)ch * K;
    } else {
      base = x + (size_t)min(m0 + row - C::TC, M - 1) * K;
    }
    gsrc[i] = base + logical_chunk * 8 + kp * (K / KSP);
  }
  i32x4 staged[C::IPW];
  const int nk = TAIL ? K / BK + 1 : K / (BK * KSP);        // (else K % (BK KSP) == 0); nk >= 1
  auto gload = [&](int q, int kt) {
    typedef const __attribute__((address_space(1))) uint16_t* gptr;   // (else the choice below makes it a flat load)
    gptr p = (gptr)(gsrc[q] + kt * BK);
    // (a lane's chunk of load q is in the upper half of the stage: bit 2 of its number, row / 8 = w IPW + q)
    if (TAIL && kt == nk - 1 && (((l >> 2) ^ (w * C::IPW + q)) & 1)) p = (gptr)&kZeros;
    staged[q] = *(const __attribute__((address_space(1))) i32x4*)p;
  };
  auto swrite = [&](int q, int buf) {
    *(i32x4*)(smem + buf * C::STAGE_BYTES + (w * C::IPW + q) * 1024 + l * 16) = staged[q];
  };

  // prologue: stage 0 into LDS, stage 1 into the registers.  Loads past the last stage re-read
  // it: unconditional loads keep the outstanding-load count the same in every iteration, so
  // the waits the compiler derives are exact.
#pragma unroll
  for (int q = 0; q < C::IPW; q++) gload(q, 0);
#pragma unroll
  for (int q = 0; q < C::IPW; q++) swrite(q, 0);
  __syncthreads();
  // the loads must be issued in the order the main loop consumes them: its waits count the loads
  // issued after the one needed
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < C::IPW; q++) {
    gload(q, min(1, nk - 1));
    __builtin_amdgcn_sched_barrier(0);
  }

  if constexpr (MI == 32) {
    // ======== 32x32x16 MFMA: wave tile = 4 tiles of 32 channels x 32 tokens ========
    f32x16 acc[4][1];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][0][v] = 0.0f;

    // operand read offsets (bytes within a stage) for k-step 0; k-step ks flips chunk bits
    int offA[4];
#pragma unroll
    for (int i = 0; i < 4; i++) offA[i] = (wc * 128 + i * 32 + (l & 31)) * C::ROWB;
    const int offB = (C::TC + wt * 32 + (l & 31)) * C::ROWB;
    const int sw = C::swz(l & 31);                            // tile bases are multiples of 32 rows

    bf16x8 a[2][4], b[2];
    int kt = 0;
    do {                                                      // nk >= 1
      const unsigned char* sb = smem + (kt & 1) * C::STAGE_BYTES;
      const int wbuf = (kt + 1) & 1, kt_load = min(kt + 2, nk - 1);
      // operands of k-step ks+1 are fetched from LDS while the MFMAs of k-step ks run
      auto lds_fetch = [&](int ks, int slot) {
        const int at = ((2 * ks + (l >> 5)) ^ sw) << 4;
#pragma unroll
        for (int i = 0; i < 4; i++) a[slot][i] = *(const bf16x8*)(sb + offA[i] + at);
        b[slot] = *(const bf16x8*)(sb + offB + at);
      };
      lds_fetch(0, 0);
#pragma unroll
      for (int ks = 0; ks < C::KS; ks++) {
        const int cur = ks & 1;
        int pair = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
          acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][i], b[cur], acc[i][0], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (i == 0 && ks + 1 < C::KS) lds_fetch(ks + 1, cur ^ 1);
          // the PP store/load pairs of this k-step, spread over its four MFMAs
          if (pair < C::PP && i >= (pair * 4) / C::PP) {
            const int q = ks * C::PP + pair;
            swrite(q, wbuf);
            gload(q, kt_load);
            pair++;
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();   // stage kt+1 is complete in LDS; stage kt may be overwritten
    } while (++kt < nk);

    if constexpr (KSP == 2) {
      // the second k-part hands its sums to the first through the stage buffers (every wave has passed the
      // loop's last barrier, so nothing reads them any more); the first adds them and goes on alone
      float4* red = (float4*)smem_all + (size_t)w * (16 * 64) + l;
      if (kp == 1) {
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
          for (int q = 0; q < 4; q++)
            red[(i * 4 + q) * 64] = make_float4(acc[i][0][4 * q], acc[i][0][4 * q + 1], acc[i][0][4 * q + 2], acc[i][0][4 * q + 3]);
      }
      __syncthreads();
      if (kp == 1) return;
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const float4 v = red[(i * 4 + q) * 64];
          acc[i][0][4 * q] += v.x;
          acc[i][0][4 * q + 1] += v.y;
          acc[i][0][4 * q + 2] += v.z;
          acc[i][0][4 * q + 3] += v.w;
        }
    }

    // ---- epilogue, in registers ------------------------------------------------------
    const int vb = ct * C::TC + wc * 128, tok_base = m0 + wt * 32;   // first virtual channel and token of this wave
    if (vb >= Kv) return;
    if (vb < r_pad) {
      rq::store_bf16(acc, vb, tok_base, M, r, xh);
      if (vb + 128 <= r_pad) return;                          // (else the split point lies inside this wave's channels)
    }
    if constexpr (QM == 2) {
      const int m = tok_base + (l & 31);
      float amax[1];
      rq::store_f32(acc, vb - r_pad, tok_base, M, K - r, xf, amax);
      if (l < 32 && m < M) pmax[(size_t)((vb - r_pad) >> 7) * sx_ld + m] = amax[0];
    } else {
      float tmax[1][4], tmin[1][4];
      rq::tile_extremes<QM>(acc, tmax, tmin);
      rq::group_extremes(g, tmax, tmin);
      rq::store_low<QM>(acc, tmax, tmin, vb - r_pad, tok_base, M, K - r, g, xl, sx, zx, sx_ld, fields);
    }
  } else {
    // ======== 16x16x32 MFMA: wave tile = 8 x 4 tiles of 16 channels x 16 tokens =========
    // Accumulator layout of a 16x16 tile: lane l holds channels 4*(l/16) .. +3 of token l%16, so
    // the 16 channels of one token sit in the four lanes {t, t+16, t+32, t+48}; a quantization
    // group (2, 4 or 8 tiles) is reduced in-lane and then across those four lanes.
    constexpr int NI = 8, NJ = 4;                           // 16-channel x 16-token tiles per wave
    constexpr int KS2 = BK / 32;                            // MFMA k-steps per stage
    constexpr int PPS = C::IPW / KS2;                       // store/load pairs per k-step
    static_assert(MI != 16 || (C::IPW % KS2 == 0 && PPS <= NI), "store/load pairs are spread over the 8 tile rows of a k-step");
    f32x4 acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; i++)
#pragma unroll
      for (int j = 0; j < NJ; j++)
#pragma unroll
        for (int v = 0; v < 4; v++) acc[i][j][v] = 0.0f;

    // operand reads: lane l takes row l%16 of a tile, 16-byte chunk 4*ks + l/16 of the stage's k range
    const int lr = l & 15, hq = l >> 4;
    const int offA = (wc * 128 + lr) * C::ROWB, offB = (C::TC + wt * 64 + lr) * C::ROWB;
    const int sw = C::swz(lr);                                // tile bases are multiples of 16 rows

    bf16x8 a[3], b[2][NJ];
    int kt = 0;
    do {                                                      // nk >= 1
      const unsigned char* sb = smem + (kt & 1) * C::STAGE_BYTES;
      const int wbuf = (kt + 1) & 1, kt_load = min(kt + 2, nk - 1);
      // flat index f = ks*NI + i over the stage's (k-step, channel tile) pairs; A tiles are fetched two
      // ahead of their MFMAs, the B tiles of the next k-step during the current one
      auto fetch_a = [&](int f) {
        const int ks = f / NI, i = f % NI;
        a[f % 3] = *(const bf16x8*)(sb + offA + i * 16 * C::ROWB + (((4 * ks + hq) ^ sw) << 4));
      };
      auto fetch_b = [&](int ks, int j) {
        b[ks & 1][j] = *(const bf16x8*)(sb + offB + j * 16 * C::ROWB + (((4 * ks + hq) ^ sw) << 4));
      };
#pragma unroll
      for (int j = 0; j < NJ; j++) fetch_b(0, j);
      fetch_a(0);
      fetch_a(1);
#pragma unroll
      for (int f = 0; f < KS2 * NI; f++) {
        const int ks = f / NI, i = f % NI;
        if (f + 2 < KS2 * NI) fetch_a(f + 2);
        if (ks + 1 < KS2 && i >= 2 && i < 2 + NJ) fetch_b(ks + 1, i - 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NJ; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[f % 3], b[ks & 1][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        // the PPS store/load pairs of this k-step, spread over its tile rows
#pragma unroll
        for (int p = 0; p < PPS; p++)
          if (i == (p * NI) / PPS) {
            const int q = ks * PPS + p;
            swrite(q, wbuf);
            gload(q, kt_load);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();   // stage kt+1 is complete in LDS; stage kt may be overwritten
    } while (++kt < nk);

    // ---- epilogue, in registers ------------------------------------------------------
    const int vb = ct * C::TC + wc * 128;                     // first virtual channel of this wave
    if (vb >= Kv) return;
    if (vb < r_pad) {
      // 16-bit part: the lane's 4 consecutive channels of a tile -> one 8-byte store
#pragma unroll
      for (int j = 0; j < NJ; j++) {
        const int m = m0 + wt * 64 + j * 16 + lr;
#pragma unroll
        for (int i = 0; i < NI; i++) {
          const int c = vb + i * 16 + 4 * hq;
          if (c < r && m < M) {
            uint2 o;
            o.x = f32_to_bf16_bits(acc[i][j][0]) | ((uint32_t)f32_to_bf16_bits(acc[i][j][1]) << 16);
            o.y = f32_to_bf16_bits(acc[i][j][2]) | ((uint32_t)f32_to_bf16_bits(acc[i][j][3]) << 16);
            *(uint2*)(xh + (size_t)m * r + c) = o;
          }
        }
      }
      if (vb + 128 <= r_pad) return;                          // (else the split point lies inside this wave's channels)
    }
    const int cl0 = vb - r_pad;                               // first 4-bit channel of this wave (negative: see above)
    const int KL = K - r;
    if constexpr (QM == 2) {
#pragma unroll
      for (int j = 0; j < NJ; j++) {
        const int m = m0 + wt * 64 + j * 16 + lr;
        float a = 0.0f;
#pragma unroll
        for (int i = 0; i < NI; i++) {
          const int cl = cl0 + i * 16;
          if (cl < KL) {
#pragma unroll
            for (int e = 0; e < 4; e++) a = fmaxf(a, fabsf(acc[i][j][e]));
            if (m < M)
              *(float4*)(xf + (size_t)m * KL + cl + 4 * hq) =
                  make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
          }
        }
        a = fmaxf(a, __shfl_xor(a, 16));
        a = fmaxf(a, __shfl_xor(a, 32));
        if (hq == 0 && m < M) pmax[(size_t)(cl0 >> 7) * sx_ld + m] = a;
      }
      return;
    }
    const size_t xl_ld = (size_t)KL / 2;
    const int gu = g >> 5, g_log2 = 31 - __builtin_clz(g);    // 32-channel units per group: 1, 2, 4
    // The four lanes of a token are the four 16-lane rows of the wave; data moves between them with
    // the row-swap instructions of gfx950 (4 swaps transpose a 4x4 block of dwords over rows x registers).
    auto swap16 = [](uint32_t& x, uint32_t& y) {              // rows (x1 <-> y0), (x3 <-> y2)
      auto v = __builtin_amdgcn_permlane16_swap(x, y, false, false);
      x = v[0];
      y = v[1];
    };
    auto swap32 = [](uint32_t& x, uint32_t& y) {              // rows (x2 <-> y0), (x3 <-> y1)
      auto v = __builtin_amdgcn_permlane32_swap(x, y, false, false);
      x = v[0];
      y = v[1];
    };
    auto transpose4 = [&](uint32_t (&v)[4]) {                 // afterwards v[h] on row q = old v[q] on row h
      swap16(v[0], v[1]);
      swap16(v[2], v[3]);
      swap32(v[0], v[2]);
      swap32(v[1], v[3]);
    };
#pragma unroll
    for (int j = 0; j < NJ; j++) {
      const int m = m0 + wt * 64 + j * 16 + lr;
      // absmax (symmetric) or min and max (asymmetric) per 32-channel unit (two tiles) in-lane;
      // after the transpose row q holds unit q's four partial results, so row q finishes unit q
      uint32_t um[4], un[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        if constexpr (ASYM) {
          float lo = acc[2 * u][j][0], hi = acc[2 * u][j][0];
#pragma unroll
          for (int e = 0; e < 4; e++) {
            lo = fminf(fminf(lo, acc[2 * u][j][e]), acc[2 * u + 1][j][e]);
            hi = fmaxf(fmaxf(hi, acc[2 * u][j][e]), acc[2 * u + 1][j][e]);
          }
          um[u] = __builtin_bit_cast(uint32_t, hi);
          un[u] = __builtin_bit_cast(uint32_t, lo);
        } else {
          float v = 0.0f;
#pragma unroll
          for (int e = 0; e < 4; e++) v = fmaxf(fmaxf(v, fabsf(acc[2 * u][j][e])), fabsf(acc[2 * u + 1][j][e]));
          um[u] = __builtin_bit_cast(uint32_t, v);
        }
      }
      auto f = [](uint32_t b) { return __builtin_bit_cast(float, b); };
      auto bits = [](float v) { return __builtin_bit_cast(uint32_t, v); };
      transpose4(um);
      float gm = fmaxf(fmaxf(f(um[0]), f(um[1])), fmaxf(f(um[2]), f(um[3]))), gn = 0.0f;
      if constexpr (ASYM) {
        transpose4(un);
        gn = fminf(fminf(f(un[0]), f(un[1])), fminf(f(un[2]), f(un[3])));
      }
      if (gu > 1) {                                           // groups of 2 or 4 units: combine rows
        uint32_t e0 = bits(gm), e1 = e0;
        swap16(e0, e1);                                       // e0 = rows (0,0,2,2), e1 = rows (1,1,3,3)
        gm = fmaxf(f(e0), f(e1));
        if constexpr (ASYM) {
          uint32_t d0 = bits(gn), d1 = d0;
          swap16(d0, d1);
          gn = fminf(f(d0), f(d1));
        }
        if (gu > 2) {
          uint32_t f0 = bits(gm), f1 = f0;
          swap32(f0, f1);                                     // f0 = rows (0,1,0,1), f1 = rows (2,3,2,3)
          gm = fmaxf(f(f0), f(f1));
          if constexpr (ASYM) {
            uint32_t c0 = bits(gn), c1 = c0;
            swap32(c0, c1);
            gn = fminf(f(c0), f(c1));
          }
        }
      }
      // row q: scale (and zero-point) of the group that unit q belongs to
      uint16_t sbits, zbits = 0;
      float sf, zf_q = 0.0f;
      if constexpr (ASYM) {
        zf_q = group_zero(gn, zbits);
        sf = group_scale_asym(gn, gm, sbits);
      } else {
        sf = group_scale(gm, sbits);
      }
      const float inv_q = group_inv(sf);
      const int clu = cl0 + 32 * hq;                          // first channel of unit hq
      const bool valid = clu >= 0 && clu < KL && m < M;
      if (valid && (hq & (gu - 1)) == 0) {
        sx[(size_t)(clu >> g_log2) * sx_ld + m] = sbits;
        if constexpr (ASYM) zx[(size_t)(clu >> g_log2) * sx_ld + m] = zbits;
      }
      // broadcast the four rows' values to all rows: b[u] = row u's value everywhere
      auto broadcast4 = [&](float v, float (&b)[4]) {
        uint32_t i0 = bits(v), i1 = i0;
        swap16(i0, i1);                                       // i0 = rows (0,0,2,2), i1 = rows (1,1,3,3)
        uint32_t i2 = i0, i3 = i1;
        swap32(i0, i2);                                       // i0 = row 0 everywhere, i2 = row 2 everywhere
        swap32(i1, i3);                                       // i1 = row 1 everywhere, i3 = row 3 everywhere
        b[0] = f(i0);
        b[1] = f(i1);
        b[2] = f(i2);
        b[3] = f(i3);
      };
      float inv[4], zf[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      broadcast4(inv_q, inv);
      if constexpr (ASYM) broadcast4(zf_q, zf);
      // codes: P[u] = the lane's 4 + 4 codes of unit u (tile 2u in the low half, tile 2u+1 in the high half)
      uint32_t P[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = acc[2 * u + (e >> 2)][j][e & 3];
        P[u] = quant_pack8<ASYM>(v, zf[u], inv[u]);
      }
      transpose4(P);                                          // P[h] = row h's codes of unit hq
      // unit hq = 16 bytes: tile 2hq (low halves, rows 0..3 in channel order), then tile 2hq+1
      uint4 o;
      o.x = (P[0] & 0xFFFFu) | (P[1] << 16);
      o.y = (P[2] & 0xFFFFu) | (P[3] << 16);
      o.z = (P[0] >> 16) | (P[1] & 0xFFFF0000u);
      o.w = (P[2] >> 16) | (P[3] & 0xFFFF0000u);
      if (!ASYM && fields) o = pipe::to_fields(o);
      if (valid) *(uint4*)(xl + (size_t)m * xl_ld + clu / 2) = o;
    }
  }
}

// Virtual channel order of the tiling: the 16-bit part [0, r) first, then the 4-bit part from r_pad on.  r_pad is r
// itself when the groups then still fall inside the 128-channel wave tiles (r a multiple of the group size: the
// wave that holds the split point stores both kinds), else r rounded up to 128.  The fp32 output for the 8-bit
// quantizer keeps the rounded form (its per-wave maxima are indexed by whole 128-channel tiles of the 4-bit part).
static void virtual_channels(int K, int r, int g, bool fp32_out, int& r_pad, int& Kv) {
  r_pad = (!fp32_out && r % g == 0) ? r : (r + 127) / 128 * 128;
  Kv = (r_pad + (K - r) + 127) / 128 * 128;
}

template <int WGC, int WGT, int MI, int QM, int KSP, bool TAIL>
static int launch_one(const uint16_t* x, const uint16_t* Qt, int M, int K, int r, int g, uint16_t* xh,
                      uint8_t* xl, uint16_t* sx, uint16_t* zx, float* xf, float* pmax, hipStream_t s, int sx_ld, bool fields) {
  using C = RQ<WGC, WGT, MI, KSP>;
  int r_pad, Kv;
  virtual_channels(K, r, g, QM == 2, r_pad, Kv);
  const int n_ct = (Kv + C::TC - 1) / C::TC;
  const int n_tt = (M + C::TT - 1) / C::TT;
  const long n_blocks = (long)n_ct * n_tt;
  const int per_xcd = (int)((n_blocks + 7) / 8);
  // (idempotent: two threads racing here would both set the same attribute)
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)rotate_quantize_kernel<WGC, WGT, MI, QM, KSP, TAIL>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM);
    if (e != hipSuccess) return hip_failed(e);
    attr_done.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((rotate_quantize_kernel<WGC, WGT, MI, QM, KSP, TAIL>), dim3(per_xcd * 8), dim3(C::NT), C::SMEM, s, x,
                     Qt, M, K, r, g, xh, xl, sx, zx, xf, pmax, r_pad, Kv, n_ct, n_tt, per_xcd, sx_ld, fields);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

template <int WGC, int WGT, int MI, int KSP = 1, bool TAIL = false>
static int launch_cfg(const RqOut& o, const uint16_t* x, const uint16_t* Qt, int M, int K, int r, int g,
                      hipStream_t s, int sx_ld) {
  if (o.xf) return launch_one<WGC, WGT, MI, 2, KSP, TAIL>(x, Qt, M, K, r, g, o.xh, o.xl, o.sx, o.zx, o.xf, o.pmax, s, sx_ld, o.fields);
  if (o.zx) return launch_one<WGC, WGT, MI, 1, KSP, TAIL>(x, Qt, M, K, r, g, o.xh, o.xl, o.sx, o.zx, o.xf, o.pmax, s, sx_ld, o.fields);
  return launch_one<WGC, WGT, MI, 0, KSP, TAIL>(x, Qt, M, K, r, g, o.xh, o.xl, o.sx, o.zx, o.xf, o.pmax, s, sx_ld, o.fields);
}

int launch_rotate_quantize(const uint16_t* x, const uint16_t* Qt, int M, int K, int r, int g, RqOut& o,
                           hipStream_t s) {
  // Few tokens: rotate_quantize_few.hip.  While one workgroup per CU holds everything: 128 x 64 tiles with K split over two
  // sets of waves, 128 x 128 tiles, then tiles of 128 x 160 to 128 x 256 fed by copies (rotate_quantize_dma.hip).  Beyond: 256
  // x 256 tiles (8 waves), and 256 x 128 or 128 x 256 ones fed by copies.
  // The large tiles run long enough to be limited by power (the shader clock drops under
  // sustained MFMA work on random data); there the 16x16x32 MFMA, which moves half the
  // accumulator bytes per multiply-add, is the faster one.  The smaller, latency-bound
  // launches are faster with the 32x32x16 MFMA and its shorter epilogue.
  int r_pad, Kv;
  virtual_channels(K, r, g, o.xf != nullptr, r_pad, Kv);
  auto tiles = [&](long channels, long tokens) { return ((Kv + channels - 1) / channels) * ((M + tokens - 1) / tokens); };
  int cus = 0;
  {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_failed(e);
    if (cus < 1) cus = 1;
  }
  // Few tokens: the split-K kernel, as long as all its workgroups are resident at once (its LDS admits one per CU); in
  // a second round it loses (K = 3072: 8.4 / 9.6 / 12.7 / 16.9 us at M = 1 / 77 / 256 / 384 against 20.0-20.9 here, 30
  // against 20 us at M = 512; K = 1152: 4.9-10 against 11 us up to M = 1280).  The smallest tile that fits: more workgroups,
  // each with fewer rows to pull (M = 77, K = 3072: 16 instead of 32 tokens 10.2 -> 9.6 us).
  struct FewTile { int channels, tokens; };
  auto fits = [&](FewTile t) { return (long)((Kv + t.channels - 1) / t.channels) * ((M + t.tokens - 1) / t.tokens) <= cus; };
  // (it writes nibbles whatever is asked for: the field form's code would cost every small call 0.05 us)
  const bool fields = o.fields;
  o.fields = false;
  if (o.xf) {
    // no groups: any channel tile (and the 4-bit part begins right behind the 16-bit one)
    for (FewTile t : {FewTile{32, 8}, {32, 16}, {32, 24}, {32, 32}, {64, 24}, {64, 32}, {64, 64}, {64, 96}})
      if ((long)((K + t.channels - 1) / t.channels) * ((M + t.tokens - 1) / t.tokens) <= cus) {
        o.pmax = nullptr;
        return launch_rotate_quantize_few(x, Qt, M, K, r, g, o, r, K, t.channels, t.tokens, s);
      }
  } else if (g == 128) {
    for (FewTile t : {FewTile{128, 8}, {128, 16}, {128, 32}})
      if (fits(t)) return launch_rotate_quantize_few(x, Qt, M, K, r, g, o, r_pad, Kv, t.channels, t.tokens, s);
  } else {
    for (FewTile t : {FewTile{64, 8}, {64, 16}, {64, 24}, {64, 32}, {64, 64}, {64, 96}})
      if (fits(t)) return launch_rotate_quantize_few(x, Qt, M, K, r, g, o, r_pad, Kv, t.channels, t.tokens, s);
  }
  o.fields = fields;
  // A launch this small is held back by the chain of stage latencies: with 128 x 64 tiles and the two halves of K on two sets
  // of waves per workgroup it has twice the workgroups and half the stages (11 instead of 13 us at M = 256, K = 1152; 21
  // instead of 26 at K = 3072).
  if (K % 128 == 0 && tiles(128, 64) <= cus) return launch_cfg<1, 2, 32, 2>(o, x, Qt, M, K, r, g, s, M);
  auto copied = [&](int channels, int tokens) {
    return launch_rotate_quantize_dma(x, Qt, M, K, r, g, o, r_pad, Kv, channels, tokens, s, M);
  };
  // 128 x 128: staged through registers, but fed by copies where K ends in half a stage (M = 1792, K = 2080: 23.5 us, 35.4 in
  // stages of 32), or where it is short and the split point lies inside a wave's 128 channels, which then store both kinds (the
  // copied tiles' waves have 64 channels).  K = 640 / 896 / 1024, M = 6397 / 4515 / 4014, registers | copies, us: r = 64 11.4 | 10.6,
  // 12.9 | 12.2, 13.8 | 13.3; r = 128 11.1 | 11.1, 12.5 | 12.8, 13.9 | 13.9 (with 30% fewer tokens 9.5 | 9.7, 11.0 | 11.6, 11.9 |
  // 12.6); equal at K = 1152; K = 3072, M = 1024 27.7 | 30.3.
  if (tiles(128, 128) <= cus)
    return K % 64 != 0 || (K <= 1024 && r_pad % 128 != 0) ? copied(128, 128) : launch_cfg<1, 4, 32>(o, x, Qt, M, K, r, g, s, M);
  // Then the smallest tile that still is one round, us against two of the above or a round of larger ones: M = 3931, K =
  // 1152 16.6 (128 x 160) against 22.2; M = 5211 18.8 (192) against 23.1; M = 7003 22.3 (256) against 30.7; K = 3072, M =
  // 1371 / 1883 / 2523: 35.5 / 40.8 / 50.1 against 42.4 / 45.3 / 52.8; K = 6144, M = 731 / 1115: 69.9 / 94 against 78.5 / 97.9.
  for (int tokens : {160, 192, 256})
    if (tiles(128, tokens) <= cus) return copied(128, tokens);
  // Beyond that: rounds of workgroups, in units of a round of 256 x 256 tiles (K = 3072: 81 us, K = 12288: 300-320).  One of
  // half-size tiles takes about 0.62 of it (K = 3072: 50; fed through registers 53), one of 128 x 256 tiles 0.66 (they fit
  // better where K / 128 is odd: M = 13403, K = 1152 43 us against 56 in two rounds of the largest).  The plans compared are:
  // one kind for all, or k full rounds of big tiles and the remaining tokens in a second launch of half-size ones.
  const long n_tc256 = (Kv + 255) / 256, big_tiles = tiles(256, 256);
  auto rounds = [&](long t) { return (double)((t + cus - 1) / cus); };
  constexpr double MID = 0.62, LOW = 0.66, SECOND_LAUNCH = 0.03;
  double best = rounds(big_tiles);                          // plan: one launch of big tiles
  enum { kBig = -1, kMid = 0, kLow = -2 };
  int plan_tt = kBig;                                       // or > 0: token tiles in the big launch
  if (rounds(tiles(256, 128)) * MID < best) {
    best = rounds(tiles(256, 128)) * MID;
    plan_tt = kMid;
  }
  if (rounds(tiles(128, 256)) * LOW < best) {
    best = rounds(tiles(128, 256)) * LOW;
    plan_tt = kLow;
  }
  for (long k = 1; k * cus < big_tiles; k++) {
    const long tt = k * cus / n_tc256;                      // token tiles of 256 that k rounds hold
    if (tt <= 0 || tt * 256 >= M) continue;
    const long rest = n_tc256 * ((M - tt * 256 + 127) / 128);
    const double c = rounds(tt * n_tc256) + rounds(rest) * MID + SECOND_LAUNCH;
    if (c < best) {
      best = c;
      plan_tt = (int)tt;
    }
  }
  if (plan_tt == kMid) return copied(256, 128);
  if (plan_tt == kLow) return copied(128, 256);
  auto big = [&](int tokens) {
    return K % 64 != 0 ? launch_cfg<2, 4, 16, 1, true>(o, x, Qt, tokens, K, r, g, s, M)
                       : launch_cfg<2, 4, 16>(o, x, Qt, tokens, K, r, g, s, M);
  };
  if (plan_tt == kBig) return big(M);
  const int first = plan_tt * 256, st = big(first);
  if (st) return st;
  RqOut rest = o;                                           // (the tokens behind the first ones)
  if (o.xh) rest.xh += (size_t)first * r;
  if (o.xl) rest.xl += (size_t)first * ((K - r) / 2);
  if (o.sx) rest.sx += first;
  if (o.zx) rest.zx += first;
  if (o.xf) rest.xf += (size_t)first * (K - r);
  if (o.pmax) rest.pmax += first;
  return launch_rotate_quantize_dma(x + (size_t)first * K, Qt, M - first, K, r, g, rest, r_pad, Kv, 256, 128, s, M);
}

}  // namespace dirotq
