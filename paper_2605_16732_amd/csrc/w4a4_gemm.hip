// Kernel B: y = x_h W'_h^T + sum_j s_x[:,j] s_w[:,j]^T * (q_x,j q_w,j^T)
// (forward-computation equation of Section 4.2 of the paper): layers of a few hundred to a few thousand tokens.
//
// Arithmetic.  A 4-bit code is an exact FP6 (E2M3) number: the nibble [s mmm] becomes [s 00 mmm] = +-m * 2^-3 (an unsigned one
// of asymmetric activations [0 0 u uuu]), and the block-scaled 32x32x64 MFMA with the E8M0 scale 2^3 on both operands
// returns the exact integer dot of a group in fp32.  The scale product of a group is an outer product of fp16 vectors: one
// fp16 MFMA (scales in k-slot 0) forms it exactly, one fma per accumulator and group applies it.  The 16-bit branch runs on
// bf16 MFMAs into the same accumulators.  Groups of 32: a stage holds two, each multiplied with the other's half of the
// weight operand cleared.
//
// Asymmetric activations.  The zero-point term sum_j z[m,j] (s_w[n,j] sum_k q_w[n,k]) is added by bf16 MFMAs on exact splits of
// its factors (z = z1 + z2, c = b1 + b2 + b3, all six products): the k-slots of one lane half hold a group, {z1 z2}
// three times against {b1 b1} {b2 b2} {b3 b3}, so that the token operand is one dword repeated and one MFMA takes two groups.
//
// Schedule.  128 channels x 128 tokens per workgroup, eight waves: four of 32 channels, twice, for the even and the odd
// stages of 64 channels of K.  A wave loads its channels' codes straight into the lanes that multiply them and unpacks them
// there: weights never pass through LDS and are unpacked once.  Tokens are unpacked once per workgroup, by the four
// waves of a part of K, and lie in LDS in the order in which the lanes read them (no bank conflicts, no swizzle; a lane's
// second 16 bytes hold the rest of its codes and its scale).  A wave multiplies 32 x 128 outputs per stage; the fma sweep of
// a token tile follows the MFMAs of the next one, and each part of the next stages' work (unpacking, LDS stores two
// stages ahead, loads three and four ahead) has its place between two tiles.  One barrier per stage.  One tile per
// workgroup: what walking several tiles costs in every stage (a compare, a branch, pointers) is more than it saves.
// Bound: instruction issue.  A tile of 32 x 32 and a group takes 64 cycles of MFMA, 40 of fma and about 26 integer
// operations of 4.3 cycles, which add up (measured 200 cycles; three waves per SIMD with K in three parts: 190, lost
// again in the exchange of their sums).  The 128 x 128 tiles before it had four waves that staged both operands through LDS
// as fp8: M = 1000, K = N = 3072, r = 128 34.0 us, with the 16-bit branch in the order of the MFMA lanes 24.8, staged by rows 23.5
// (asymmetric 39.1, 27.0, 25.7).
#include <algorithm>
#include <atomic>

#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "gemm_tail.h"
#include "pipe_unpack.h"
#include "tile_walk.h"
#include "w4a4_plan.h"

#include "dirotq_internal.h"

namespace dirotq {

namespace tile {

constexpr int NT = 512, NJ = 4, KS = 2, NBUF = 3;
constexpr int TNW = 128, TMW = 128;          // output channels, tokens of a workgroup
typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
#define GLOBAL __attribute__((address_space(1)))
typedef const GLOBAL uint8_t* gptr;

// A fragment: what 32 tokens x 64 channels are in LDS, in the order in which the lanes read it.
//   64 x 16 B: first 16 of a lane's 24 bytes of codes | 64 x {8 bytes of codes, s, 0} (lanes 32..63: s = 0) |
//   groups of 32: 64 x {s of the second group, 0} (same) | asymmetric: zero-points 64 x {Z, Z, Z, 0}
constexpr int gps(int gs) { return gs == 32 ? 2 : 1; }
constexpr int HI = 1024, SC1 = 2048;
constexpr int zp_at(int gs) { return SC1 + (gs == 32 ? 512 : 0); }
constexpr int frag_bytes(int gs, bool asym) { return zp_at(gs) + (asym ? 1024 : 0); }

template <int GS, bool OUT_F32, bool ASYM>
struct Geo {
  static constexpr int FRAG = frag_bytes(GS, ASYM), SLOT = NJ * FRAG, RING = NBUF * KS * SLOT;
  static constexpr int PASS = (TNW + TMW) * 128;                      // 16-bit branch: a buffer of 64 channels
  // the exchange: per wave two tiles of partial sums; then the rows of y
  static constexpr int X_WAVE = 2 * 4096, OUT_ROW = TNW * (OUT_F32 ? 4 : 2) + 16;
  static constexpr int X_BYTES = 8 * X_WAVE + TMW * OUT_ROW;
  static constexpr int LOOP = RING > 2 * PASS ? RING : 2 * PASS, SMEM = LOOP > X_BYTES ? LOOP : X_BYTES;
};

__device__ __forceinline__ void barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int GS, bool OUT_F32, bool ASYM, bool FIELDS>
__global__ __launch_bounds__(NT, 2) void w4a4_gemm_kernel(
    const uint16_t* __restrict__ xh, const uint8_t* __restrict__ xl, const uint16_t* __restrict__ sx,
    const uint16_t* __restrict__ zx, const uint16_t* __restrict__ wh, const uint8_t* __restrict__ wq,
    const uint16_t* __restrict__ sw, const int16_t* __restrict__ wsum, const uint16_t* __restrict__ bias, int M, int N,
    int K, int r, void* __restrict__ y, int n_mt, int n_nt, int per_xcd) {
  extern __shared__ __align__(16) unsigned char smem[];
  typedef Geo<GS, OUT_F32, ASYM> g_;
  constexpr int GPS = gps(GS), FRAG = g_::FRAG, SLOT = g_::SLOT, ZP = zp_at(GS);

  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || logical >= n_mt * n_nt) return;
  int m0, n0;
  tile_origin<4, TNW, TMW>(logical, n_mt, n_nt, m0, n0);

  const int t = threadIdx.x, l = t & 63, row = l & 31, half = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int ws = w & 3, kh = w >> 2;                                  // 32 channels (and the token tile that is staged), part of K
  const int KL = K - r, G = KL / GS, ldq = KL / 2;
  const int nq = (KL + 63) / 64, nqi = (nq + 1) / 2;                  // stages, intervals
  const bool short_last = GS == 32 && (KL % 64) != 0;
  const uint32_t rn = (uint32_t)(min(n0 + 32 * ws + row, N - 1) - n0), rm = (uint32_t)(min(m0 + 32 * ws + row, M - 1) - m0);
  const uint32_t lane16 = l * 16, lower = half ? 0u : 0xFFFFu;

  f32x16 acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; j++)
#pragma unroll
    for (int v = 0; v < 16; v++) acc[j][v] = 0.0f;

  // ---- 16-bit branch, ahead of everything else: 64 channels at a time of all rows, 128 bytes of a row by eight lanes, through two
  // LDS buffers; part kh multiplies 32 of them.  Bound: the LDS writes (32 KB a pass).  Loaded in the order of the MFMA lanes, 32
  // bytes of a row each, it got 15 bytes per clock and CU, also beside the first loads of the 4-bit part: M = 1000, K = N = 3072,
  // r = 64 / 256 / 1536 / 2944 26.1 / 26.4 / 39.3 / 52.2 us, now 24.7 / 24.1 / 30.3 / 30.9 (the four-wave kernel before: 34.6 /
  // 34.1 / 37.7 / 41.4).
  auto branch16 = [&]() {
    const int lrow = t >> 3, lchunk = t & 7, np = (r + 63) / 64;
    gptr src[4];
#pragma unroll
    for (int i = 0; i < 4; i++)
      src[i] = i < 2 ? (gptr)wh + (size_t)min(n0 + lrow + 64 * i, N - 1) * (2 * r)
                     : (gptr)xh + (size_t)min(m0 + lrow + 64 * (i - 2), M - 1) * (2 * r);
    u32x4 v[2][4];
    auto fetch = [&](auto set, int p) {                               // (past the end: the row's last 16 bytes, never used)
      const int off = min(p * 128 + lchunk * 16, 2 * r - 16);
#pragma unroll
      for (int i = 0; i < 4; i++) v[set][i] = *(const GLOBAL u32x4*)(src[i] + off);
    };
    auto pass = [&](auto set, int p) {
      unsigned char* buf = smem + set * g_::PASS;                     // [128 weight rows, 128 token rows][128 bytes]
#pragma unroll
      for (int i = 0; i < 4; i++) *(u32x4*)(buf + tile_off_bytes(lrow + 64 * i, lchunk)) = v[set][i];
      fetch(set, p + 2);
      barrier();
      if (kh == 0 || 64 * p + 32 < r) {
#pragma unroll
        for (int e = 0; e < 2; e++) {
          const int chunk = 2 * (2 * kh + e) + half;
          const i32x4 av = *(const i32x4*)(buf + tile_off_bytes(32 * ws + row, chunk));
#pragma unroll
          for (int j = 0; j < NJ; j++) {
            const i32x4 bv = *(const i32x4*)(buf + tile_off_bytes(TNW + 32 * j + row, chunk));
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv), acc[j], 0, 0, 0);
          }
        }
      }
    };
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    fetch(even, 0);
    fetch(odd, 1);
    for (int p = 0;;) {
      pass(even, p);
      if (++p == np) break;
      pass(odd, p);
      if (++p == np) break;
    }
    barrier();                                                        // (the buffers become the 4-bit part's ring)
  };

  if (r > 0) branch16();
  if (nq > 0) {
    // ---- loads of the 4-bit part: the part's stage i holds the 64 channels from 64 (2 i + kh) on
    const uint32_t vw = __umul24(rn, ldq) + half * 16, vx = __umul24(rm, ldq) + half * 16;
    const int first = min(kh, nq - 1);
    gptr wq_p = (gptr)wq + (size_t)n0 * ldq + first * 32, xl_p = (gptr)xl + (size_t)m0 * ldq + first * 32;
    u32x4 rw[2], rx[2];
    uint16_t rsw[2], rsx[2], rzs[2], rzx[2];
    int16_t rzw[2];
    int lw = 0, lx = 0;                                               // stage of the next load
    // a row's last 32 channels alone: both halves read them
    auto cut = [&](int sq) { return short_last && sq >= nq - 1 ? half * 16u : 0u; };
    // scales: group of lane half h of stage sq; a lane keeps its column and multiplies its row out
    const gptr sw_c = (gptr)(sw + n0 + rn), sx_c = (gptr)(sx + m0 + rm);
    const gptr sc_c = half ? sx_c : sw_c;                             // groups of 64, 128: one load for both, x one stage ahead
    const uint32_t sc_ld = half ? 2u * M : 2u * N;
    auto group = [&](int sq) { return GS == 128 ? sq >> 1 : GS == 64 ? sq : 2 * sq + half; };
    auto load_w = [&](auto set) {
      const int sq = 2 * lw + kh;
      rw[set] = *(const GLOBAL u32x4*)(wq_p + (GS == 32 ? vw - cut(sq) : vw));
      if constexpr (GS == 32) {
        rsw[set] = *(const GLOBAL uint16_t*)(sw_c + (uint64_t)(uint32_t)min(group(sq), G - 1) * (2u * N));
      } else {
        rsw[set] = *(const GLOBAL uint16_t*)(sc_c + (uint64_t)(uint32_t)min(group(sq + 2 * half), G - 1) * sc_ld);
      }
      if constexpr (ASYM) {
        if (GS == 32 || set == 0) {
          const int jz = min((GS == 32 ? sq : (lw >> 1) * KS + kh) * 2 + half, G - 1);
          const uint64_t o = (uint64_t)(uint32_t)jz * (2u * N);
          rzs[set] = *(const GLOBAL uint16_t*)(sw_c + o);
          rzw[set] = *(const GLOBAL int16_t*)((gptr)(wsum + n0 + rn) + o);
        }
      }
      lw++;
      wq_p += 2 * lw + kh < nq ? 64 : 0;
    };
    auto load_x = [&](auto set) {
      const int sq = 2 * lx + kh;
      rx[set] = *(const GLOBAL u32x4*)(xl_p + (GS == 32 ? vx - cut(sq) : vx));
      if constexpr (GS == 32) rsx[set] = *(const GLOBAL uint16_t*)(sx_c + (uint64_t)(uint32_t)min(group(sq), G - 1) * (2u * M));
      if constexpr (ASYM) {
        if (GS == 32 || set == 0) {
          const int jz = min((GS == 32 ? sq : (lx >> 1) * KS + kh) * 2 + half, G - 1);
          rzx[set] = *(const GLOBAL uint16_t*)((gptr)(zx + m0 + rm) + (uint64_t)(uint32_t)jz * (2u * M));
        }
      }
      lx++;
      xl_p += 2 * lx + kh < nq ? 64 : 0;
    };

    // ---- weights: raw -> operand registers (stage iw)
    i32x8 a[2];
    i32x2 sa[2][GPS];
    u32x4 za;
    int iw = 0;
    auto unpack_w = [&](auto set, int part) {
      uint32_t d[3];
      pipe::unpack16_fp6(rw[set][2 * part], rw[set][2 * part + 1], d);
#pragma unroll
      for (int e = 0; e < 3; e++) a[set][3 * part + e] = (int)d[e];
    };
    auto scale_w = [&](auto set) {
      const int sq = 2 * iw + kh;
      if constexpr (GS == 32) {
        // lanes 0..31 take both groups' scales: the second one's lie in the upper half
        const auto v = __builtin_amdgcn_permlane32_swap((uint32_t)rsw[set], (uint32_t)rsw[set], false, false);
        sa[set][0] = i32x2{(int)(v[0] & (2 * sq < G ? lower : 0u)), 0};
        sa[set][1] = i32x2{(int)(v[1] & (2 * sq + 1 < G ? lower : 0u)), 0};
      } else {
        sa[set][0] = i32x2{(int)(rsw[set] & (sq < nq ? lower : 0u)), 0};
      }
      if constexpr (ASYM) {
        if (GS == 32 || set == 0) {
          const int jz = (GS == 32 ? sq : (iw >> 1) * KS + kh) * 2 + half;
          const float c = jz < G ? f16_bits_to_f32(rzs[set]) * (float)rzw[set] : 0.0f;
          const uint32_t p1 = __builtin_bit_cast(uint32_t, c) & 0xFFFF0000u;
          const float c1 = c - __builtin_bit_cast(float, p1);
          const uint32_t p2 = __builtin_bit_cast(uint32_t, c1) & 0xFFFF0000u;
          const float c2 = c1 - __builtin_bit_cast(float, p2);
          const uint32_t p3 = __builtin_bit_cast(uint32_t, c2) & 0xFFFF0000u;
          za = u32x4{p1 | p1 >> 16, p2 | p2 >> 16, p3 | p3 >> 16, 0u};
        }
      }
      iw++;
    };
    // ---- tokens: raw -> LDS (stage ix)
    int ix = 0;
    const int frag = ws * FRAG;
    auto put_x = [&](auto set, uint16_t scale, int so) {
      uint32_t d0[3], d1[3];
      const u32x4 v = rx[set];
      if constexpr (FIELDS) {
        pipe::expand32_fp6(v, d0, d1);
      } else {
        pipe::half16_fp6<ASYM>(v[0], v[1], d0);
        pipe::half16_fp6<ASYM>(v[2], v[3], d1);
      }
      unsigned char* f = smem + (so + frag);
      const int sq = 2 * ix + kh;
      uint32_t s;
      if constexpr (GS == 32) {
        s = scale & (2 * sq + half < G ? 0xFFFFu : 0u);
      } else {
        s = __builtin_amdgcn_permlane32_swap((uint32_t)scale, (uint32_t)scale, false, false)[1] & (sq < nq ? lower : 0u);
      }
      *(u32x4*)(f + lane16) = u32x4{d0[0], d0[1], d0[2], d1[0]};
      *(u32x4*)(f + HI + lane16) = u32x4{d1[1], d1[2], GS == 32 && half ? 0u : s, 0u};
      if constexpr (GS == 32) *(u32x2*)(f + SC1 + ((half ^ 1) * 32 + row) * 8) = u32x2{half ? s : 0u, 0u};
      if constexpr (ASYM) {
        if (GS == 32 || set == 0) {
          const int jz = (GS == 32 ? sq : (ix >> 1) * KS + kh) * 2 + half;
          const float z = jz < G ? f16_bits_to_f32(rzx[set]) : 0.0f;
          const uint32_t z1 = __builtin_bit_cast(uint32_t, z) & 0xFFFF0000u;
          const uint32_t z2 = __builtin_bit_cast(uint32_t, z - __builtin_bit_cast(float, z1));
          const uint32_t Z = __builtin_amdgcn_perm(z2, z1, 0x07060302u);
          *(u32x4*)(f + ZP + lane16) = u32x4{Z, Z, Z, 0u};
        }
      }
      ix++;
    };
    // ---- operands of token tile j
    i32x8 b[2];
    i32x2 sb1[2];
    i32x4 zb[2];
    auto read_b = [&](auto zset, int j, int so) {
      const unsigned char* f = smem + (so + j * FRAG);
      b[j & 1] = __builtin_shufflevector(*(const i32x4*)(f + lane16), *(const i32x4*)(f + HI + lane16), 0, 1, 2, 3, 4, 5, 6, 7);
      if (GS == 32) sb1[j & 1] = *(const i32x2*)(f + SC1 + l * 8);
      if constexpr (ASYM) {
        if (GS == 32 || zset == 0) zb[j & 1] = *(const i32x4*)(f + ZP + lane16);
      }
    };

    typedef std::integral_constant<int, 0> S0;
    typedef std::integral_constant<int, 1> S1;
    int cur = kh * (NBUF * SLOT), nxt = cur + SLOT, fill = cur + 2 * SLOT;
    f32x16 I[2], P[2];
    const int low_keep = half ? 0 : -1;
    auto interval = [&](auto set) {
      constexpr int other = 1 - set;
      std::integral_constant<int, other> next;
#pragma unroll
      for (int j = 0; j < NJ; j++) {
#pragma unroll
        for (int jj = 0; jj < GPS; jj++) {
          f32x16 z;
#pragma unroll
          for (int v = 0; v < 16; v++) z[v] = 0.0f;
          i32x8 av = a[set];
          if constexpr (GS == 32) {
            const int keep = jj ? ~low_keep : low_keep;
#pragma unroll
            for (int e = 0; e < 6; e++) av[e] &= keep;
          }
          const i32x2 sbv = jj ? sb1[j & 1] : __builtin_shufflevector(b[j & 1], b[j & 1], 6, 7);
          const int sc = 127 + 3, s = (GPS * j + jj) & 1;
          P[s] = __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(f16x4, sa[set][jj]), __builtin_bit_cast(f16x4, sbv), z, 0, 0, 0);
          I[s] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, b[j & 1], z, 2, 2, 0, sc, 0, sc);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (ASYM) {
            if (jj == 0 && (GS == 32 || set == 0)) {
              acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, za), __builtin_bit_cast(bf16x8, zb[j & 1]), acc[j], 0, 0, 0);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
          if (jj == GPS - 1) {
            if (j + 1 < NJ) read_b(set, j + 1, cur);
            else read_b(next, 0, nxt);
            if (j == 0) {
              unpack_w(next, 0);
              unpack_w(next, 1);
            }
            if (j == 1) {
              // (the scale of this wave's tokens travels with the weights' of the stage before)
              put_x(set, GS == 32 ? rsx[set] : rsw[next], fill);
            }
            if (j == 2) {
              load_x(set);
            }
            if (j == 3) {
              scale_w(next);
              load_w(next);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          const int u = GPS * j + jj - 1;                             // the sweep of the tile before
          if (u >= 0) {
            const int jp = u / GPS;
#pragma unroll
            for (int v = 0; v < 16; v++) acc[jp][v] = fmaf(I[s ^ 1][v], P[s ^ 1][v], acc[jp][v]);
            asm volatile("" : "+v"(acc[jp]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int v = 0; v < 16; v++) acc[NJ - 1][v] = fmaf(I[1][v], P[1][v], acc[NJ - 1][v]);
      asm volatile("" : "+v"(acc[NJ - 1]));
      __builtin_amdgcn_sched_barrier(0);
      barrier();
      const int freed = cur;
      cur = nxt;
      nxt = fill;
      fill = freed;
    };

    // ---- prologue: stages 0 and 1 of the tokens in LDS, 2 and 3 on their way; stage 0 of the weights unpacked
    uint16_t s0;
    if constexpr (GS != 32) s0 = *(const GLOBAL uint16_t*)(sc_c + (uint64_t)(uint32_t)min(group(kh), G - 1) * sc_ld);
    load_x(S0{});
    load_w(S0{});
    load_x(S1{});
    load_w(S1{});
    put_x(S0{}, GS == 32 ? rsx[0] : s0, cur);
    load_x(S0{});
    put_x(S1{}, GS == 32 ? rsx[1] : rsw[0], nxt);
    load_x(S1{});
    unpack_w(S0{}, 0);
    unpack_w(S0{}, 1);
    scale_w(S0{});
    load_w(S0{});
    barrier();
    read_b(S0{}, 0, cur);
    int i = 0;
    for (; i + 1 < nqi; i += 2) {
      interval(S0{});
      interval(S1{});
    }
    if (i < nqi) interval(S0{});
  }

  // ---- the two parts of K exchange: part kh finishes the token tiles kh and 2 + kh
  barrier();
  float4* mine = (float4*)(smem + w * g_::X_WAVE);
#pragma unroll
  for (int p = 0; p < 2; p++)
#pragma unroll
    for (int q = 0; q < 4; q++) {
      float4 v;
      v.x = kh ? acc[2 * p][4 * q] : acc[2 * p + 1][4 * q];
      v.y = kh ? acc[2 * p][4 * q + 1] : acc[2 * p + 1][4 * q + 1];
      v.z = kh ? acc[2 * p][4 * q + 2] : acc[2 * p + 1][4 * q + 2];
      v.w = kh ? acc[2 * p][4 * q + 3] : acc[2 * p + 1][4 * q + 3];
      mine[(4 * p + q) * 64 + l] = v;
    }
  barrier();
  const float4* theirs = (const float4*)(smem + (w ^ 4) * g_::X_WAVE);
  unsigned char* rows = smem + 8 * g_::X_WAVE;
#pragma unroll
  for (int p = 0; p < 2; p++)
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const float4 o = theirs[(4 * p + q) * 64 + l];
      const int c = 32 * ws + 8 * q + 4 * half;                       // this lane's four channels of the quad
      float v[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
      for (int e = 0; e < 4; e++) v[e] += kh ? acc[2 * p + 1][4 * q + e] : acc[2 * p][4 * q + e];
      if (bias) {
        const int n = n0 + c;
        if (n + 4 <= N) {
          const uint2 bb = *(const uint2*)(bias + n);
          v[0] += bf16_bits_to_f32((uint16_t)(bb.x & 0xFFFF));
          v[1] += bf16_bits_to_f32((uint16_t)(bb.x >> 16));
          v[2] += bf16_bits_to_f32((uint16_t)(bb.y & 0xFFFF));
          v[3] += bf16_bits_to_f32((uint16_t)(bb.y >> 16));
        } else {
#pragma unroll
          for (int e = 0; e < 4; e++) v[e] += bf16_bits_to_f32(bias[min(n + e, N - 1)]);
        }
      }
      unsigned char* d = rows + (32 * (2 * p + kh) + row) * g_::OUT_ROW;
      if (OUT_F32) {
        *(float4*)(d + 4 * c) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
        *(uint2*)(d + 2 * c) = make_uint2(f32x2_to_bf16x2_bits(v[0], v[1]), f32x2_to_bf16x2_bits(v[2], v[3]));
      }
    }
  barrier();
  // ---- rows of y: 16 bytes a lane where they are aligned, else value by value
  constexpr int ES = OUT_F32 ? 4 : 2, LPR = TNW * ES / 16, EPL = 16 / ES;
  unsigned char* yb = (unsigned char*)y;
  if (N % EPL == 0) {
    const int c = (t % LPR) * EPL;
#pragma unroll
    for (int k = 0; k < TMW * LPR / NT; k++) {
      const int tok = k * (NT / LPR) + t / LPR;
      const uint4 d = *(const uint4*)(rows + tok * g_::OUT_ROW + c * ES);
      if (m0 + tok < M && n0 + c < N) *(uint4*)(yb + ((size_t)(m0 + tok) * N + n0 + c) * ES) = d;
    }
  } else {
    const int c = t % TNW;
#pragma unroll 4
    for (int k = 0; k < TMW * TNW / NT; k++) {
      const int tok = k * (NT / TNW) + t / TNW;
      if (m0 + tok < M && n0 + c < N) {
        if (OUT_F32) ((float*)y)[(size_t)(m0 + tok) * N + n0 + c] = *(const float*)(rows + tok * g_::OUT_ROW + c * 4);
        else ((uint16_t*)y)[(size_t)(m0 + tok) * N + n0 + c] = *(const uint16_t*)(rows + tok * g_::OUT_ROW + c * 2);
      }
    }
  }
}

template <int GS, bool OUT_F32, bool ASYM, bool FIELDS>
static int launch_one(const uint16_t* xh, const uint8_t* xl, const uint16_t* sx, const uint16_t* zx, const void* blob,
                      const uint16_t* bias, int M, int N, int K, int r, void* y, hipStream_t s) {
  typedef Geo<GS, OUT_F32, ASYM> g_;
  const BlobLayout L = blob_layout(N, K, r, GS);
  const char* bp = (const char*)blob;
  const int n_mt = (M + TMW - 1) / TMW, n_nt = (N + TNW - 1) / TNW;
  const int per_xcd = (int)(((long)n_mt * n_nt + 7) / 8);
  // (idempotent: two threads racing here would both set the same attribute)
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)w4a4_gemm_kernel<GS, OUT_F32, ASYM, FIELDS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, g_::SMEM);
    if (e != hipSuccess) return hip_failed(e);
    attr_done.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((w4a4_gemm_kernel<GS, OUT_F32, ASYM, FIELDS>), dim3(per_xcd * 8), dim3(NT), g_::SMEM, s, xh, xl, sx, zx,
                     (const uint16_t*)(bp + L.off_wh), (const uint8_t*)(bp + L.off_codes), (const uint16_t*)(bp + L.off_sw),
                     (const int16_t*)(bp + L.off_wsum), bias, M, N, K, r, y, n_mt, n_nt, per_xcd);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

}  // namespace tile

// Layers without 4-bit channels, more than one tile per CU: several workgroups of four waves per CU, of which one stores while
// others multiply, and no exchange of partial sums.  us, the tiles above | this: M = 32768, K = 1152, N = 4608 498 | 450; M =
// 4608, K = 3072, N = 12288 455 | 414; M = 4608, K = 12288, N = 3072 465 | 447; with a tile per CU or less the ones above are
// faster: M = 1000, K = N = 3072 33.6 | 41.
template <bool OUT_F32>
__global__ __launch_bounds__(NTHREADS, 2) void dense_gemm_kernel(const uint16_t* __restrict__ xh, const uint16_t* __restrict__ wh,
                                                                 const uint16_t* __restrict__ bias, int M, int N, int r,
                                                                 void* __restrict__ y, int n_mt, int n_nt, int per_xcd) {
  __shared__ __align__(16) unsigned char smem[(TN + TM) * 128];
  const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= n_mt * n_nt) return;
  int m0, n0;
  tile_origin<4, TN, TM>(logical, n_mt, n_nt, m0, n0);
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  f32x16 acc[2][2];
  int rowA[2], rowB[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    rowA[i] = (w & 1) * 64 + i * 32 + (l & 31);
    rowB[i] = TN + (w >> 1) * 64 + i * 32 + (l & 31);
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;
  }
  gemm_tail<OUT_F32>(acc, smem, xh, wh, bias, y, M, N, r, m0, n0, rowA, rowB);
}

template <bool OUT_F32>
static int launch_dense(const uint16_t* xh, const uint16_t* wh, const uint16_t* bias, int M, int N, int r, void* y, hipStream_t s) {
  const int n_mt = (M + TM - 1) / TM, n_nt = (N + TN - 1) / TN;
  const int per_xcd = (int)(((long)n_mt * n_nt + 7) / 8);
  hipLaunchKernelGGL((dense_gemm_kernel<OUT_F32>), dim3(per_xcd * 8), dim3(NTHREADS), 0, s, xh, wh, bias, M, N, r, y, n_mt, n_nt,
                     per_xcd);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

// The schedule of a layer (w4a4_plan.h).  DIROTQ_W4A4_KERNEL=pipe / large / small / ws / tile / skinny / skinny32 /
// skinny64 in the environment forces one of them wherever it applies (the tests use it to run all of them on the same
// inputs; large and small: the pipelined kernel with one kind of tile; skinny32 and skinny64: the split-K kernel with one
// of its two, skinny: with the cheaper one).
int w4a4_plan_layer(int M, int N, int K, int r, int g, bool asym, W4A4Plan& plan) {
  W4A4Schedule& sch = plan.schedule;
  long& big_tokens = plan.big_tokens;
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return hip_failed(e);
  if (cus < 1) cus = 1;
  const char* f = getenv("DIROTQ_W4A4_KERNEL");
  if (f && K > r) {
    const bool large = !strcmp(f, "large"), small = !strcmp(f, "small"), ws = !strcmp(f, "ws");
    big_tokens = 0;
    if (!strcmp(f, "tile") && w4a4_plan::tiles(M, N, tile::TMW, tile::TNW) <= w4a4_plan::MOST_TILES) return sch = W4A4Schedule::kTile, DIROTQ_OK;
    if (!strcmp(f, "skinny32")) return sch = W4A4Schedule::kSkinny32, DIROTQ_OK;
    if (!strcmp(f, "skinny64")) return sch = W4A4Schedule::kSkinny64, DIROTQ_OK;
    if (!strcmp(f, "skinny")) {
      const w4a4_plan::Cost cost(K, r, g, asym, cus);
      sch = cost.skinny32(M, N) <= cost.skinny64(M, N) ? W4A4Schedule::kSkinny32 : W4A4Schedule::kSkinny64;
      return DIROTQ_OK;
    }
    if (ws || large || small || !strcmp(f, "pipe")) {
      // (symmetric groups of 32 have no wave-specialised form, asymmetric layers no pipelined one)
      sch = asym || (ws && g != 32) ? W4A4Schedule::kWs : W4A4Schedule::kPipe;
      w4a4_pipe_plan(M, N, cus, big_tokens);
      if (large || small) big_tokens = large ? M : 0;
      return DIROTQ_OK;
    }
  }
  sch = w4a4_choose(M, N, K, r, g, asym, cus, big_tokens);
  return DIROTQ_OK;
}

int launch_w4a4_gemm(const W4A4Plan& plan, bool fields, const uint16_t* xh, const uint8_t* xl, const uint16_t* sx,
                     const uint16_t* zx, const void* blob, const uint16_t* bias, int M, int N, int K, int r, int g, void* y,
                     int y_dtype, hipStream_t s) {
  // (asymmetric layers: the wave-specialised schedule, the split-K ones or this file's kernel)
  if (plan.schedule == W4A4Schedule::kPipe)
    return launch_w4a4_gemm_pipe(xh, xl, sx, blob, bias, M, N, K, r, g, y, y_dtype, plan.big_tokens, fields, s);
  if (plan.schedule == W4A4Schedule::kWs)
    return launch_w4a4_gemm_ws(xh, xl, sx, zx, blob, bias, M, N, K, r, g, y, y_dtype, s);
  if (plan.schedule == W4A4Schedule::kSkinny32 || plan.schedule == W4A4Schedule::kSkinny64)
    return launch_w4a4_gemm_skinny(xh, xl, sx, zx, blob, bias, M, N, K, r, g, y, y_dtype, plan.schedule == W4A4Schedule::kSkinny32, s);
  // (without 4-bit channels the activations are rows of x_h alone, so that the slabs need nothing but their first token)
  const long slab = w4a4_plan::slab_tokens(N);
  if (K == r && M > slab) {
    int st = DIROTQ_OK;
    for (long m = 0; m < M && !st; m += slab)
      st = launch_w4a4_gemm(plan, fields, xh + (size_t)m * r, xl, sx, zx, blob, bias, (int)std::min(slab, M - m), N, K, r, g,
                            (char*)y + (size_t)m * N * (y_dtype ? 4 : 2), y_dtype, s);
    return st;
  }
  if (plan.schedule == W4A4Schedule::kDense) {
    const uint16_t* wh = (const uint16_t*)((const char*)blob + blob_layout(N, K, r, g).off_wh);
    return y_dtype ? launch_dense<true>(xh, wh, bias, M, N, r, y, s) : launch_dense<false>(xh, wh, bias, M, N, r, y, s);
  }
#define DIROTQ_TILE(GS, OUT, ASYM, FIELDS) tile::launch_one<GS, OUT, ASYM, FIELDS>(xh, xl, sx, zx, blob, bias, M, N, K, r, y, s)
#define DIROTQ_CASE(GS)                                                                                          \
  case GS:                                                                                                       \
    if (fields) return DIROTQ_TILE(GS, false, false, true);                                                      \
    if (zx) return y_dtype ? DIROTQ_TILE(GS, true, true, false) : DIROTQ_TILE(GS, false, true, false);           \
    return y_dtype ? DIROTQ_TILE(GS, true, false, false) : DIROTQ_TILE(GS, false, false, false);
  switch (g) {
    DIROTQ_CASE(32)
    DIROTQ_CASE(64)
    DIROTQ_CASE(128)
  }
#undef DIROTQ_CASE
#undef DIROTQ_TILE
  return DIROTQ_ERR_SHAPE;
}

}  // namespace dirotq

