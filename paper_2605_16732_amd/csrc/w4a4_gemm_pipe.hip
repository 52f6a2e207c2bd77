// Kernel B, large schedule for symmetric activation codes:
//   y = x_h W'_h^T + sum_j s_x[:,j] s_w[:,j]^T * (q_x,j q_w,j^T)
// (forward-computation equation of Section 4.2 of the paper).
//
// Arithmetic.  A 4-bit code is an exact FP6 (E2M3) number: the nibble [s mmm] becomes [s 00 mmm] = +-m * 2^-3, and
// the block-scaled 32x32x64 MFMA with the E8M0 scale 2^3 on both operands returns the exact integer dot of a group in
// fp32.  With FP6 operands that instruction takes half the cycles it takes with fp8 ones (35 against 64).  The scale
// product of a group is an outer product of fp16 vectors: one fp16 MFMA (scales in k-slot 0) forms it exactly, one fma
// per accumulator and group applies it.  The 16-bit branch runs on bf16 MFMAs into the same accumulators.
//
// Schedule.  Eight waves (two per SIMD), each 64 output channels x 32 NB tokens, and every wave both stages and
// multiplies.  What a lone wave can issue is the limit of a separate staging wave per SIMD (the wave-specialised
// schedule): one VALU instruction per 5-6 cycles, ~160 instructions a stage, so a stage takes as long as that however
// fast the matrix pipe is (FP6 operands alone gained nothing there).  Spread over the multiplying waves the same work
// runs in the slots between the issue of a tile's MFMAs and their results.  Bound: the VALU.  A tile of 32 x 32 and a
// group cost 16 fma + 8 unpacking (NB = 4; 12 with NB = 2) + ~3 other instructions = 114 cycles beside 64 of MFMA; it
// runs at 152 (of the busy CUs' SIMD-cycles VALU active 74%, MFMA 39%, both at once 16%; K = 12288, N = 3072).  256 x 256
// tiles because the unpacking per tile and group goes with (rows staged) / (tiles multiplied).  In whole layers the
// activations come in field form (FIELDS; pipe_unpack.h), which takes 5 instead of 8 of these operations (7 of 12).
// Measured against the wave-specialised schedule (M = 4608, us): K = 3072, N = 9216 / 3072 / 12288: 204 / 67 / 248
// against 261 / 79 / 272; K = 12288, N = 3072: 229 against 257; M = 32768, K = 1152, N = 4608: 294 against 356; groups
// of 32 (K = 12288, N = 3072): 443 against 543.
//
// K is walked in stages of 32 bytes per row: first the 16-bit branch (16 bf16 channels per stage, copied), then the
// 4-bit channels (64 per stage, expanded to 48 bytes of FP6).  In interval s the waves multiply stage s, read the
// first operands of stage s+1, write stage s+2 into the LDS ring (three slots) and load stage s+4 into the registers
// that this frees; one barrier per interval.  Workgroups are persistent, one per CU, and the stage stream is
// continuous across a workgroup's tiles.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "gemm_tail.h"
#include "pipe_plan.h"
#include "pipe_stage.h"
#include "pipe_unpack.h"
#include "tile_walk.h"

namespace dirotq {

namespace pipe {

constexpr int NT = 512;
constexpr int NBUF = 3;
constexpr int tmw(int nb) { return 64 * nb; }                     // tokens per workgroup tile (2 waves of 32 nb)
constexpr int rows(int nb) { return TNW + tmw(nb); }
constexpr int gps(int gs) { return gs == 32 ? 2 : 1; }            // scale groups per stage
constexpr int scale_bytes(int gs) { return gps(gs) * 512 * 16; }  // fp16 {scale, 0, 0, 0 | 0, 0, 0, 0} per row
constexpr int slot_bytes(int nb, int gs) { return rows(nb) * SB + scale_bytes(gs); }
// behind the ring: per wave a [32 tokens][64 channels] bf16 block (rows padded to 144 B) through which finished
// outputs are turned from the accumulator layout (a lane holds one token) into whole rows
constexpr int OUT_ROW = 144, OUT_WAVE_BYTES = 32 * OUT_ROW;
constexpr int out_off(int nb, int gs) { return NBUF * slot_bytes(nb, gs); }
constexpr int smem_bytes(int nb, int gs) { return out_off(nb, gs) + 8 * OUT_WAVE_BYTES; }

typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
#define GLOBAL __attribute__((address_space(1)))
typedef const GLOBAL uint8_t* gptr;

// bf16 store of a wave's block of 64 output channels (which all exist, N a multiple of 8) x 32 NB tokens: in the
// accumulator layout a store instruction would touch 32 rows with 16 bytes each; via the wave's LDS block it writes 8
// rows of 128 contiguous bytes.  tb: the wave's own LDS block (no other wave touches it: no barrier).
template <int NB>
__device__ __forceinline__ void store_block_rows(const f32x16 (&acc)[2][NB], const uint16_t* __restrict__ bias,
                                                 uint16_t* __restrict__ y, int M, int N, int m_base, int n_base,
                                                 unsigned char* tb) {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));   // (addresses below are formed here, per tile: not carried in registers through the loops)
  const int h = l >> 5;
  unsigned char* wr = tb + (l & 31) * OUT_ROW + 8 * h;          // this lane's token row, channel 4 h
  const unsigned char* rd = tb + (l >> 3) * OUT_ROW + (l & 7) * 16;   // row l >> 3 (+ 8 k), channels 8 (l & 7) ..
  uint16_t* dst = y + (size_t)(m_base + (l >> 3)) * N + n_base + 8 * (l & 7);
#pragma unroll
  for (int j = 0; j < NB; j++) {
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        if (bias) {
          const uint2 bb = *(const uint2*)(bias + n_base + i * 32 + 8 * q + 4 * h);
          v[0] += bf16_bits_to_f32((uint16_t)(bb.x & 0xFFFF));
          v[1] += bf16_bits_to_f32((uint16_t)(bb.x >> 16));
          v[2] += bf16_bits_to_f32((uint16_t)(bb.y & 0xFFFF));
          v[3] += bf16_bits_to_f32((uint16_t)(bb.y >> 16));
        }
        uint2 o;
        o.x = f32x2_to_bf16x2_bits(v[0], v[1]);
        o.y = f32x2_to_bf16x2_bits(v[2], v[3]);
        *(uint2*)(wr + (i * 32 + 8 * q) * 2) = o;
      }
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const uint4 d = *(const uint4*)(rd + k * 8 * OUT_ROW);
      if (m_base + j * 32 + k * 8 + (l >> 3) < M) *(uint4*)(dst + (size_t)(j * 32 + k * 8) * N) = d;
    }
  }
}

// The tiles of one workgroup among the tokens [m_begin, m_end) (m_begin a multiple of the tile).  gridDim.x = 8 * wpx;
// workgroup b runs on XCD b & 7 and takes, of that XCD's run of per_xcd consecutive logical tiles, the tiles
// slot + it * wpx, it = 0, 1, ...
template <int GS, bool OUT_F32, int NB, bool FIELDS>
__device__ __forceinline__ void run_tiles(
    const uint16_t* __restrict__ xh, const uint8_t* __restrict__ xl, const uint16_t* __restrict__ sx,
    const uint16_t* __restrict__ wh, const uint8_t* __restrict__ wq, const uint16_t* __restrict__ sw,
    const uint16_t* __restrict__ bias, int M, int N, int K, int r, void* __restrict__ y, int m_begin, int m_end,
    int slot, int wpx) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int GPS = gps(GS), TM_ = tmw(NB), SLOT = slot_bytes(NB, GS), SCALE_OFF = rows(NB) * SB;
  constexpr bool WIDE_X = NB == 4;                                    // a thread stages 16 bytes of a token row (else 8)

  const int n_mt = (m_end - m_begin + TM_ - 1) / TM_, n_nt = (N + TNW - 1) / TNW;
  const int per_xcd = (n_mt * n_nt + 7) / 8;
  const int run0 = (blockIdx.x & 7) * per_xcd, first = slot;
  const int run_len = min(per_xcd, n_mt * n_nt - run0);
  if (first >= run_len) return;
  const int T = (run_len - first + wpx - 1) / wpx;                    // tiles of this workgroup (>= 1)

  const int t = threadIdx.x, l = t & 63, h = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);               // wave index as a scalar
  const int wn = w & 3, wt = w >> 2;
  const int KL = K - r;                                               // number of 4-bit channels (> 0)
  const int G = KL / GS;
  // stages of a tile: 16-bit (an even number), 4-bit (padded to an even number: the extra one has zero scales)
  const int nbf = r / 16, nq_real = (KL + 63) / 64, nq = (nq_real + 1) / 2 * 2, nst = nbf + nq;
  const int ldq = KL / 2;

  // the zeros behind every scale (the stages write the scales only)
  for (int i = t; i < NBUF * GPS * 512; i += NT)
    *(uint4*)(smem + i / (GPS * 512) * SLOT + SCALE_OFF + i % (GPS * 512) * 16) = make_uint4(0u, 0u, 0u, 0u);

  // ---- staging role: 16-byte half (t & 1) of weight row t >> 1; of the token rows the same (NB = 4) or the 8-byte
  // quarter t & 3 of row t >> 2 (NB = 2); the scales of row t of (weights, tokens)
  const int half = t & 1;
  const int xrow = WIDE_X ? t >> 1 : t >> 2, xpart = WIDE_X ? half : t & 3, xhalf = WIDE_X ? half : xpart >> 1;
  // LDS offsets within a slot (pipe_stage.h)
  const RowPart part_w = row_part<GS>(t >> 1, half);
  constexpr int XOFF = TNW * SB;                                      // (the token rows follow the weight rows)
  const RowPart part_x = WIDE_X ? RowPart{part_w.at + XOFF, part_w.at_hi + XOFF, part_w.at_copy + XOFF}
                                : row_part<GS>(TNW + xrow, xhalf);
  const bool short_last = GS == 32 && (KL % 64) != 0;                 // the last stage holds one 32-channel group

  // load cursor: the tile and stage the next load is for.  Uniform bases of the tile; per-lane byte offsets from
  // them (below 2^31: a tile's rows span at most 256 rows of at most 2^19 bytes)
  gptr wq_b, xl_b, wh_b, xh_b, sc_b;                                  // (sc_b: this wave's scales, weights or tokens)
  const size_t sc_ld = w < 4 ? (size_t)N * 2 : (size_t)M * 2;
  uint32_t row_w, row_x, vos;
  int lt = 0, lst = 0;
  auto set_tile = [&](int it) {
    int m0, n0;
    tile_origin<NB == 4 ? 4 : 2, TNW, TM_>(run0 + first + it * wpx, n_mt, n_nt, m0, n0);
    m0 += m_begin;
    wq_b = (gptr)wq + (size_t)n0 * ldq;
    xl_b = (gptr)xl + (size_t)m0 * ldq;
    wh_b = (gptr)wh + (size_t)n0 * (2 * r);
    xh_b = (gptr)xh + (size_t)m0 * (2 * r);
    row_w = (uint32_t)(min(n0 + (t >> 1), N - 1) - n0);
    row_x = (uint32_t)(min(m0 + xrow, M - 1) - m0);
    sc_b = w < 4 ? (gptr)sw + (size_t)n0 * 2 : (gptr)sx + (size_t)m0 * 2;
    vos = 2u * (w < 4 ? (uint32_t)(min(n0 + t, N - 1) - n0) : (uint32_t)(min(m0 + t - 256, M - 1) - m0));
  };
  set_tile(0);

  // two register sets, one stage each.  Loads are straight-line code of one shape, whatever the stage's kind, so
  // that the count of loads in flight is exact and a store waits for its own set only.
  typedef std::conditional_t<WIDE_X, u32x4, u32x2> x_t;
  u32x4 rw[2];
  x_t rx[2];
  uint16_t rs[2][GPS];
  auto gload = [&](auto set) {                                        // loads the cursor's stage, then moves on
    const bool is_b = lst < nbf;
    const int sq = max(lst - nbf, 0);
    const size_t off = (size_t)(is_b ? lst : min(sq, nq_real - 1)) * 32;
    const uint32_t ld = is_b ? 2 * r : ldq;
    uint32_t ow = half * 16, ox = xpart * (WIDE_X ? 16 : 8);
    if (GS == 32) {                                                   // (both halves read the group that exists)
      const bool last = short_last && !is_b && sq >= nq_real - 1;
      ow -= last ? half * 16 : 0;
      ox -= last ? xhalf * 16 : 0;
    }
    const gptr wb = (is_b ? wh_b : wq_b) + off, xb = (is_b ? xh_b : xl_b) + off;
    rw[set] = *(const GLOBAL u32x4*)(wb + (__umul24(row_w, ld) + ow));
    rx[set] = *(const GLOBAL x_t*)(xb + (__umul24(row_x, ld) + ox));
#pragma unroll
    for (int jj = 0; jj < GPS; jj++) {
      const int j = GS == 128 ? sq >> 1 : sq * GPS + jj;              // group of these channels
      rs[set][jj] = *(const GLOBAL uint16_t*)(sc_b + (size_t)min(j, G - 1) * sc_ld + vos);
    }
    lst++;
  };
  // (called every second stage, where a tile can end; past the last tile its stages are read again, unused)
  auto wrap_loads = [&]() {
    if (lst == nst) {
      lst = 0;
      if (lt + 1 < T) set_tile(++lt);
    }
  };
  int sst = 0;                                                        // store cursor: stage within its tile
  // One stage from registers to LDS.  `copy`: a stage of the 16-bit branch, stored as it is.  The kind selects values
  // and addresses, not code (a second copy of the loop bodies for it makes the compiler move accumulators between
  // register sets).  d0, d1: the two expanded 16-channel parts of a row half.
  auto store_half = [&](unsigned char* sp, const RowPart& part, bool copy, u32x4 v, const uint32_t (&d0)[3],
                        const uint32_t (&d1)[3]) {
    const Stores at = wide_stores<GS>(part, copy);
    if constexpr (GS == 32) {                                         // lane halves of the operand: d0 | d1 of the group
      *(u32x4*)(sp + at.second) = u32x4{d1[0], d1[1], d1[2], 0u};
      *(u32x4*)(sp + at.first) = copy ? v : u32x4{d0[0], d0[1], d0[2], 0u};
    } else {                                                          // lane half = row half: 24 bytes
      *(u32x4*)(sp + at.first) = copy ? v : u32x4{d0[0], d0[1], d0[2], d1[0]};
      *(u32x2*)(sp + at.second) = u32x2{d1[1], d1[2]};
    }
  };
  auto put_x_narrow = [&](unsigned char* sp, bool copy, u32x2 v) {    // 8 bytes of a token row: one 16-channel part
    const int part = xpart & 1;
    const Stores at = FIELDS ? narrow_fields_stores<GS>(part_x, part, copy) : narrow_stores<GS>(part_x, part, copy);
    uint32_t d[3];
    if constexpr (FIELDS) {
      const uint32_t k0 = part ? kOwn2 : kOwn03, k1 = part ? kOwn03 : kOwn1;
      d[0] = v[0] & k0;
      d[1] = v[1] & k1;
      d[2] = (v[1] & ~k1) | (v[0] & ~k0);
      if constexpr (GS == 32) {
        *(u32x2*)(sp + at.first) = copy ? v : u32x2{part ? d[1] : d[0], part ? d[2] : d[1]};
        *(u32x2*)(sp + at.second) = u32x2{part ? d[0] : d[2], 0u};
      } else {
        *(uint32_t*)(sp + at.second) = d[2];
        *(u32x2*)(sp + at.first) = copy ? v : u32x2{d[0], d[1]};
      }
      return;
    }
    unpack16_fp6(v[0], v[1], d);
    if constexpr (GS == 32) {
      *(u32x2*)(sp + at.first) = copy ? v : u32x2{d[0], d[1]};
      *(u32x2*)(sp + at.second) = u32x2{d[2], 0u};
    } else {                                                          // dwords 0 1 2 of the row half's six, or 3 4 5
      *(uint32_t*)(sp + at.second) = part ? d[0] : d[2];
      *(u32x2*)(sp + at.first) = copy ? v : u32x2{part ? d[1] : d[0], part ? d[2] : d[1]};
    }
  };
  auto put_s = [&](auto set, int so) {
    unsigned char* sp = smem + so;                     // (a 16-bit stage's are not read)
    const int sq = sst - nbf;
#pragma unroll
    for (int jj = 0; jj < GPS; jj++) {
      // (a group past the end gets a zero scale: its codes are a re-read of real ones and contribute exactly nothing)
      const int j = GS == 128 ? sq >> 1 : sq * GPS + jj;
      const uint32_t keep = j < G ? 0xFFFFu : 0u;
      *(uint32_t*)(sp + SCALE_OFF + jj * (512 * 16) + t * 16) = rs[set][jj] & keep;
    }
  };

  // ---- multiplying role: operands of a 64-channel stage: 24 bytes of a row per lane (GS = 32: 12 per group)
  typedef std::conditional_t<GS == 32, i32x4, i32x2> hi_t;
  i32x4 a[2], b[2];
  hi_t a2[2], b2[2];
  f16x4 sa[2][GPS], sb[2][GPS];
  // lane half h reads chunk 2 h (of a 16-bit stage, and 16 of the 24 bytes) and the 8 bytes in chunk 2 h + 1; groups of
  // 32: chunk h (16-bit stage, group 0) and 2 + h (group 1).  Tile bases are multiples of 32 rows, so the lane's part of
  // an address is the same for weights and tokens.
  const int ln_lo = read_lo<GS>(l & 31, h), ln_hi = read_hi<GS>(l & 31, h);
  const int ln_s = SCALE_OFF + (l & 31) * 16 + h * 8;                 // (lanes 32..63, k-slots 4..7, read the zeros)
  const int rowA = wn * 64, rowB = TNW + wt * (32 * NB);
  // (of a 16-bit stage only the first 16 bytes mean something)
  auto read_a = [&](int i, int so) {
    const unsigned char *p = smem + (so + rowA * SB), *ps = smem + (so + rowA * 16);
    a[i] = *(const i32x4*)(p + ln_lo + i * (32 * SB));
    a2[i] = *(const hi_t*)(p + ln_hi + i * (32 * SB));
#pragma unroll
    for (int jj = 0; jj < GPS; jj++) sa[i][jj] = *(const f16x4*)(ps + ln_s + (i * 32 + jj * 512) * 16);
  };
  auto read_b = [&](int j, int so) {
    const unsigned char *p = smem + (so + rowB * SB), *ps = smem + (so + rowB * 16);
    b[j & 1] = *(const i32x4*)(p + ln_lo + j * (32 * SB));
    b2[j & 1] = *(const hi_t*)(p + ln_hi + j * (32 * SB));
#pragma unroll
    for (int jj = 0; jj < GPS; jj++) sb[j & 1][jj] = *(const f16x4*)(ps + ln_s + (j * 32 + jj * 512) * 16);
  };

  f32x16 acc[2][NB];
  // the same during the 4-bit stages, value by value: as one register group the compiler gives the sweep three-address fma
  // instructions, which take 2.7 cycles beside MFMAs instead of 2.4 (1% of the kernel)
  float fa[2][NB][16];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < NB; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;
  };

  int cur = 0, nxt = SLOT, fill = 2 * SLOT;   // ring slots of stages s, s + 1, s + 2

  // Step q of writing the store cursor's stage from register set `set` into the ring slot at `so` and reloading the set:
  // the work of an interval in even portions (in two lumps it costs 5-8% of the whole kernel).
  constexpr int STEPS = NB == 4 ? 6 : 4;
  uint32_t d0[3], d1[3];
  auto stage_step = [&](auto set, int q, int so) {
    const bool copy = sst < nbf;
    unsigned char* sp = smem + so;
    if (q == 0) unpack16_fp6(rw[set][0], rw[set][1], d0);
    if (q == 1) {
      unpack16_fp6(rw[set][2], rw[set][3], d1);
      store_half(sp, part_w, copy, rw[set], d0, d1);
    }
    if constexpr (WIDE_X) {
      if (!FIELDS && q == 2) unpack16_fp6(rx[set][0], rx[set][1], d0);
      if (q == 3) {
        if constexpr (FIELDS) expand32_fp6(rx[set], d0, d1);
        else unpack16_fp6(rx[set][2], rx[set][3], d1);
        store_half(sp, part_x, copy, rx[set], d0, d1);
      }
    } else {
      if (q == 2) put_x_narrow(sp, copy, rx[set]);
    }
    if (q == STEPS - 2 + (NB == 2)) put_s(set, so);
    if (q == STEPS - 1) gload(set);
  };

  // One interval: stage s (of the 16-bit branch: is_b) multiplied, stage s + 2 written, stage s + 4 loaded.
  // Straight-line code: a branch between a tile's MFMAs and their use would let the compiler move the MFMAs behind it.
  auto interval = [&](auto set, auto is_b) {
    constexpr int NWIN = 2 * NB;
#pragma unroll
    for (int q = 0; q < NWIN; q++) {
      const int j = q >> 1, i = q & 1;
      auto between = [&]() {
        // behind the issue of the tile's MFMAs: operands that have fallen free are refilled
        if (i == 0) {
          if (j + 1 < NB) read_b(j + 1, cur);
          else read_b(0, nxt);
        }
        if (j == NB - 1) read_a(i, nxt);
        stage_step(set, q, fill);                                     // and a share of the staging work
      };
      if constexpr (is_b) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i]),
                                                            __builtin_bit_cast(bf16x8, b[j & 1]), acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        between();
        __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int jj = 0; jj < GPS; jj++) {
          const i32x4 zero4 = {0, 0, 0, 0};
          f32x16 z;
#pragma unroll
          for (int v = 0; v < 16; v++) z[v] = 0.0f;
          i32x8 av, bv;
          if constexpr (GS == 32) {
            av = __builtin_shufflevector(jj ? a2[i] : a[i], zero4, 0, 1, 2, 3, 4, 5, 6, 7);
            bv = __builtin_shufflevector(jj ? b2[j & 1] : b[j & 1], zero4, 0, 1, 2, 3, 4, 5, 6, 7);
          } else {
            av = __builtin_shufflevector(a[i], __builtin_shufflevector(a2[i], a2[i], 0, 1, -1, -1), 0, 1, 2, 3, 4, 5, -1, -1);
            bv = __builtin_shufflevector(b[j & 1], __builtin_shufflevector(b2[j & 1], b2[j & 1], 0, 1, -1, -1), 0, 1, 2, 3, 4, 5, -1, -1);
          }
          const int sc = 127 + 3;                              // E8M0 block scale 2^3 on both operands: the integer dot
          const f32x16 P = __builtin_amdgcn_mfma_f32_32x32x8f16(sa[i][jj], sb[j & 1][jj], z, 0, 0, 0);
          const f32x16 I = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, z, 2, 2, 0, sc, 0, sc);
          __builtin_amdgcn_sched_barrier(0);
          if (jj == GPS - 1) between();
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int v = 0; v < 16; v++) {
            fa[i][j][v] = fmaf(I[v], P[v], fa[i][j][v]);
            asm volatile("" : "+v"(fa[i][j][v]));              // (accumulated in place)
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    // this wave's stores into the ring are done (they precede the last reads by several windows)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int freed = cur;
    cur = nxt;
    nxt = fill;
    fill = freed;
    if (++sst == nst) sst = 0;
  };

  typedef std::integral_constant<int, 0> S0;
  typedef std::integral_constant<int, 1> S1;
  typedef std::true_type Yes;
  typedef std::false_type No;
  gload(S0{});
  gload(S1{});
  wrap_loads();
  __syncthreads();                                                    // (the scale rows are cleared)
#pragma unroll
  for (int q = 0; q < STEPS; q++) stage_step(S0{}, q, cur);
  sst++;
#pragma unroll
  for (int q = 0; q < STEPS; q++) stage_step(S1{}, q, nxt);
  if (++sst == nst) sst = 0;
  __syncthreads();
  read_a(0, cur);
  read_b(0, cur);
  read_a(1, cur);

  for (int it = 0; it < T; it++) {
    clear();
    for (int st = 0; st < nbf; st += 2) {
      wrap_loads();
      interval(S0{}, Yes{});
      interval(S1{}, Yes{});
    }
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < NB; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) fa[i][j][v] = acc[i][j][v];
    for (int st = 0; st < nq; st += 2) {
      wrap_loads();
      interval(S0{}, No{});
      interval(S1{}, No{});
    }
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < NB; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[i][j][v] = fa[i][j][v];
    int m0, n0;
    tile_origin<NB == 4 ? 4 : 2, TNW, TM_>(run0 + first + it * wpx, n_mt, n_nt, m0, n0);
    m0 += m_begin + wt * (32 * NB);
    n0 += wn * 64;
    if (!OUT_F32 && (N & 7) == 0 && n0 + 64 <= N) {
      store_block_rows<NB>(acc, bias, (uint16_t*)y, M, N, m0, n0, smem + out_off(NB, GS) + w * OUT_WAVE_BYTES);
    } else {
#pragma unroll
      for (int jp = 0; jp < NB; jp += 2) {
        const f32x16 part[2][2] = {{acc[0][jp], acc[0][jp + 1]}, {acc[1][jp], acc[1][jp + 1]}};
        store_tile<OUT_F32>(part, bias, y, M, N, m0 + jp * 32, n0);
      }
    }
  }
}

// Tokens [0, m_split) in tiles of 256 x 256, the others in tiles of 256 x 128 (GS = 32: m_split = 0).
template <int GS, bool OUT_F32, bool BIG, bool FIELDS>
__global__ __launch_bounds__(NT, 2) void w4a4_gemm_pipe_kernel(
    const uint16_t* __restrict__ xh, const uint8_t* __restrict__ xl, const uint16_t* __restrict__ sx,
    const uint16_t* __restrict__ wh, const uint8_t* __restrict__ wq, const uint16_t* __restrict__ sw,
    const uint16_t* __restrict__ bias, int M, int N, int K, int r, void* __restrict__ y, int m_split, int wpx) {
  const int slot = blockIdx.x >> 3;
  if constexpr (BIG) {
    run_tiles<GS, OUT_F32, 4, FIELDS>(xh, xl, sx, wh, wq, sw, bias, M, N, K, r, y, 0, m_split, slot, wpx);
    if (m_split >= M) return;
    __syncthreads();                                                  // (the ring is laid out anew)
  }
  // (from the other end: the workgroups that had one large tile less come first)
  run_tiles<GS, OUT_F32, 2, FIELDS>(xh, xl, sx, wh, wq, sw, bias, M, N, K, r, y, m_split, M, wpx - 1 - slot, wpx);
}

template <int GS, bool OUT_F32, bool BIG, bool FIELDS>
static int launch_one(const uint16_t* xh, const uint8_t* xl, const uint16_t* sx, const void* blob,
                      const uint16_t* bias, int M, int N, int K, int r, void* y, int m_split, int cus, hipStream_t s) {
  const BlobLayout L = blob_layout(N, K, r, GS);
  const char* bp = (const char*)blob;
  const long n_nt = (N + TNW - 1) / TNW;
  const long big = BIG ? (long)((m_split + 255) / 256) * n_nt : 0;
  const long small = m_split < M ? (long)((M - m_split + 127) / 128) * n_nt : 0;
  if (std::max(big, small) > 0x7FFFFFF0L) return DIROTQ_ERR_SHAPE;
  const int wpx = (int)std::max(1L, std::min((long)cus / 8, (big + small + 7) / 8));
  constexpr int SMEM = BIG ? std::max(smem_bytes(4, GS), smem_bytes(2, GS)) : smem_bytes(2, GS);
  // (idempotent: two threads racing here would both set the same attribute)
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)w4a4_gemm_pipe_kernel<GS, OUT_F32, BIG, FIELDS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return hip_failed(e);
    attr_done.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((w4a4_gemm_pipe_kernel<GS, OUT_F32, BIG, FIELDS>), dim3(wpx * 8), dim3(NT), SMEM, s, xh, xl, sx,
                     (const uint16_t*)(bp + L.off_wh), (const uint8_t*)(bp + L.off_codes),
                     (const uint16_t*)(bp + L.off_sw), bias, M, N, K, r, y, m_split, wpx);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

}  // namespace pipe

int launch_w4a4_gemm_pipe(const uint16_t* xh, const uint8_t* xl, const uint16_t* sx, const void* blob,
                          const uint16_t* bias, int M, int N, int K, int r, int g, void* y, int y_dtype,
                          long big_tokens, bool fields, hipStream_t s) {
  int cus = 0;
  {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_failed(e);
  }
  // (32-channel groups: 256 x 128 tiles only, two groups' operands and 128 accumulators do not fit the register file)
  const int m_split = g == 32 ? 0 : (int)big_tokens;
  // (field form: between the two kernels of a whole layer, whose output is bf16)
#define DIROTQ_PIPE(GS, BIG)                                                                                           \
  return fields ? pipe::launch_one<GS, false, BIG, true>(xh, xl, sx, blob, bias, M, N, K, r, y, m_split, cus, s)       \
       : y_dtype ? pipe::launch_one<GS, true, BIG, false>(xh, xl, sx, blob, bias, M, N, K, r, y, m_split, cus, s)      \
                 : pipe::launch_one<GS, false, BIG, false>(xh, xl, sx, blob, bias, M, N, K, r, y, m_split, cus, s)
  switch (g) {
    case 32: DIROTQ_PIPE(32, false);
    case 64:
      if (m_split) DIROTQ_PIPE(64, true);
      DIROTQ_PIPE(64, false);
    case 128:
      if (m_split) DIROTQ_PIPE(128, true);
      DIROTQ_PIPE(128, false);
  }
#undef DIROTQ_PIPE
  return DIROTQ_ERR_SHAPE;
}

}  // namespace dirotq
