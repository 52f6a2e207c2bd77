// Kernel B for few tokens: the same sum as w4a4_gemm.hip,
//   y = x_h W'_h^T + sum_j s_x[:,j] s_w[:,j]^T * (q_x,j q_w,j^T)   [+ sum_j z[:,j] (s_w[:,j] sum q_w,j)^T]
// (forward-computation equation of Section 4.2 of the paper; the last term with asymmetric codes), scheduled for latency.
//
// With a few hundred tokens the tiled kernels put a handful of workgroups on a 256-CU chip, and each walks the
// whole K axis stage by stage (global load -> LDS -> barrier -> MFMA) alone on its CU: the time is a sum of
// memory latencies.  Here the K axis is split over the 8 waves of a workgroup instead.  A workgroup owns 64 output
// channels x 64 tokens, or 32 x 32 while those spread the work over more CUs; wave w takes the work items w, w + 8, ...
// of the K axis (an item = 16 channels of the 16-bit branch or one 64-channel piece of the 4-bit part; a 32-channel
// group when g = 32).  Nothing is shared between waves, so operands go from global memory straight into registers in
// the MFMA operand layout (a lane loads the 16 bytes of its row and k-half), one or two items ahead; there is no LDS
// staging and no barrier in the loop.  The eight partial accumulators then meet in LDS and are summed in a fixed order.
// Arithmetic per item as in the other schedules: fp8 MFMA on the codes (block scale 2^9 on both operands: the
// group dot comes back as the integer), fp16 MFMA for the scale product, one fma per accumulator.
// Measured (us, graph replay, symmetric / asymmetric, r = 128, g = 64): N = K = 3072: M = 1 5.9 / 6.2, M = 77 8.4 / 9.0,
// M = 512 20.0 / 21.6 (64 x 64 outputs: 10.3 / 12.0, 12.1 / 14.2, 22.9 / 26.9; 128 x 128 tiles: 28.5 / 33.0, 29.1 / 33.7,
// 30.7 / 35.6); N = 3072, K = 12288, M = 77: 21.5 / 24.0 (28.8 / 36.1; 101 / 121).
#include <atomic>
#include <type_traits>

#include "gemm_tail.h"

namespace dirotq {

namespace skinny {

constexpr int NW = 8, NT = NW * 64;
constexpr int smem_bytes(int ni, int nj) { return NW * ni * nj * 4 * 64 * 16; }   // partial sums: [wave][register quad][lane] float4

typedef __attribute__((ext_vector_type(8))) int i32x8;

// registers of one work item: the lane's operand bytes for NI weight tiles and NJ token tiles, their scales, and (with
// asymmetric codes) the group's code sums and zero-points
template <int NI, int NJ>
struct Item {
  uint4 a[NI], b[NJ];
  uint16_t sa[NI], sb[NJ], wa[NI], zb[NJ];
};

template <int GS, bool OUT_F32, bool ASYM, int NI, int NJ>
__global__ __launch_bounds__(NT, 2) void w4a4_gemm_skinny_kernel(
    const uint16_t* __restrict__ xh, const uint8_t* __restrict__ xl, const uint16_t* __restrict__ sx,
    const uint16_t* __restrict__ zx, const uint16_t* __restrict__ wh, const uint8_t* __restrict__ wq,
    const uint16_t* __restrict__ sw, const int16_t* __restrict__ wsum, const uint16_t* __restrict__ bias, int M, int N,
    int K, int r, void* __restrict__ y, int n_nt) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int nt = blockIdx.x % n_nt, mt = blockIdx.x / n_nt;
  const int n0 = nt * (32 * NI), m0 = mt * (32 * NJ);
  const int t = threadIdx.x, l = t & 63, h = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int KL = K - r;
  constexpr int ICH = GS == 32 ? 32 : 64;    // 4-bit channels per item
  const int nb = r / 16, nq = KL / ICH, items = nb + nq;
  const size_t ldq = (size_t)KL / 2;

  // the lane's rows (clamped at the edges: those results are not stored)
  size_t rowA[NI], rowB[NJ];
#pragma unroll
  for (int i = 0; i < NI; i++) rowA[i] = (size_t)min(n0 + i * 32 + (l & 31), N - 1);
#pragma unroll
  for (int j = 0; j < NJ; j++) rowB[j] = (size_t)min(m0 + j * 32 + (l & 31), M - 1);

  // loads of one shape whatever the item's kind (16 bytes per operand row, the scale halfwords): straight-line code
  const uint8_t* whb = (const uint8_t*)wh;
  const uint8_t* xhb = (const uint8_t*)xh;
  auto load = [&](Item<NI, NJ>& it, int idx) {
    const bool is_b = idx < nb;
    const int qi = max(idx - nb, 0);
    // 16 bf16 channels: this lane's 8 (k = 8 h ..); 64 4-bit channels: this lane's 32 = 16 packed bytes;
    // a 32-channel group: its 16 packed bytes, of which the lane uses the half h
    const size_t offq = GS == 32 ? (size_t)qi * 16 : (size_t)qi * 32 + h * 16;
    const size_t offb = (size_t)idx * 32 + h * 16;
#pragma unroll
    for (int i = 0; i < NI; i++)
      it.a[i] = *(const uint4*)(is_b ? whb + rowA[i] * (size_t)(2 * r) + offb : wq + rowA[i] * ldq + offq);
#pragma unroll
    for (int j = 0; j < NJ; j++)
      it.b[j] = *(const uint4*)(is_b ? xhb + rowB[j] * (size_t)(2 * r) + offb : xl + rowB[j] * ldq + offq);
    const size_t grp = (size_t)(qi * ICH) / GS;         // (group 0 for an item of the 16-bit branch: unused)
#pragma unroll
    for (int i = 0; i < NI; i++) it.sa[i] = sw[grp * N + rowA[i]];
#pragma unroll
    for (int j = 0; j < NJ; j++) it.sb[j] = sx[grp * M + rowB[j]];
    if constexpr (ASYM) {
#pragma unroll
      for (int i = 0; i < NI; i++) it.wa[i] = (uint16_t)wsum[grp * N + rowA[i]];
#pragma unroll
      for (int j = 0; j < NJ; j++) it.zb[j] = zx[grp * M + rowB[j]];
    }
  };

  f32x16 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; i++)
#pragma unroll
    for (int j = 0; j < NJ; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;

  auto compute = [&](const Item<NI, NJ>& it, int idx) {
    if (idx < nb) {
#pragma unroll
      for (int i = 0; i < NI; i++)
#pragma unroll
        for (int j = 0; j < NJ; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, it.a[i]),
                                                              __builtin_bit_cast(bf16x8, it.b[j]), acc[i][j], 0, 0, 0);
      return;
    }
    // nibbles -> fp8 bytes [s 0000 mmm] (unsigned: [0000 uuuu]); even channels of a dword to one register, odd ones to
    // another (the same permutation on both operands)
    i32x8 av[NI], bv[NJ];
    auto expand = [&](const uint4& p, auto unsigned_codes) -> i32x8 {
      auto un = [&](uint32_t d, uint32_t& e, uint32_t& o) {
        if constexpr (unsigned_codes) unpack8u(d, e, o);
        else unpack8(d, e, o);
      };
      uint32_t e[4], o[4];
      if (GS == 32) {                                  // the lane's 8 bytes of the group's 16; upper k half empty
        un(h ? p.z : p.x, e[0], o[0]);
        un(h ? p.w : p.y, e[1], o[1]);
        return i32x8{(int)e[0], (int)o[0], (int)e[1], (int)o[1], 0, 0, 0, 0};
      }
      un(p.x, e[0], o[0]);
      un(p.y, e[1], o[1]);
      un(p.z, e[2], o[2]);
      un(p.w, e[3], o[3]);
      return i32x8{(int)e[0], (int)o[0], (int)e[1], (int)o[1], (int)e[2], (int)o[2], (int)e[3], (int)o[3]};
    };
#pragma unroll
    for (int i = 0; i < NI; i++) av[i] = expand(it.a[i], std::false_type{});
#pragma unroll
    for (int j = 0; j < NJ; j++) bv[j] = expand(it.b[j], std::integral_constant<bool, ASYM>{});
    // scale vectors {s, 0, 0, 0} in lanes 0..31 (k-slot 0 of the fp16 MFMA), zeros in lanes 32..63
    f16x4 sa[NI], sb[NJ];
#pragma unroll
    for (int i = 0; i < NI; i++) sa[i] = __builtin_bit_cast(f16x4, make_uint2(h ? 0u : (uint32_t)it.sa[i], 0u));
#pragma unroll
    for (int j = 0; j < NJ; j++) sb[j] = __builtin_bit_cast(f16x4, make_uint2(h ? 0u : (uint32_t)it.sb[j], 0u));
    const int sc9 = 127 + 9;                           // E8M0 block scale 2^9: (q 2^-9 2^9)(q' 2^-9 2^9) = q q'
#pragma unroll
    for (int i = 0; i < NI; i++)
#pragma unroll
      for (int j = 0; j < NJ; j++) {
        f32x16 z, p;
#pragma unroll
        for (int v = 0; v < 16; v++) z[v] = p[v] = 0.0f;
        const f32x16 I = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av[i], bv[j], z, 0, 0, 0, sc9, 0, sc9);
        const f32x16 P = __builtin_amdgcn_mfma_f32_32x32x8f16(sa[i], sb[j], p, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 16; v++) acc[i][j][v] = fmaf(I[v], P[v], acc[i][j][v]);
      }
    if constexpr (ASYM) {
      // zero-point term z (s_w sum q_w), once per group: exact bf16 splits z = z1 + z2, s_w sum q_w = c1 + c2 + c3 in
      // six k-slots of one bf16 MFMA (c1 c2 c3 c1 c2 c3 against z1 z1 z1 z2 z2 z2), lanes 32..63 zero
      if (GS != 128 || ((idx - nb) & 1) == 0) {
        auto hi16 = [](float v) { return __builtin_bit_cast(uint32_t, v) & 0xFFFF0000u; };
        auto f = [](uint32_t b) { return __builtin_bit_cast(float, b); };
        auto pair = [](uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); };   // the upper halves
        uint4 ca[NI], cb[NJ];
#pragma unroll
        for (int i = 0; i < NI; i++) {
          const float v = h ? 0.0f : f16_bits_to_f32(it.sa[i]) * (float)(int16_t)it.wa[i];
          const uint32_t p1 = hi16(v), p2 = hi16(v - f(p1)), p3 = hi16(v - f(p1) - f(p2));
          ca[i] = make_uint4(pair(p1, p2), pair(p3, p1), pair(p2, p3), 0u);
        }
#pragma unroll
        for (int j = 0; j < NJ; j++) {
          const float v = h ? 0.0f : f16_bits_to_f32(it.zb[j]);
          const uint32_t p1 = hi16(v), p2 = hi16(v - f(p1));
          cb[j] = make_uint4(pair(p1, p1), pair(p1, p2), pair(p2, p2), 0u);
        }
#pragma unroll
        for (int i = 0; i < NI; i++)
#pragma unroll
          for (int j = 0; j < NJ; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ca[i]),
                                                                __builtin_bit_cast(bf16x8, cb[j]), acc[i][j], 0, 0, 0);
      }
    }
  };

  // Register sets in turn: while an item is multiplied the next one's loads are in flight.  Where the registers allow a
  // second set with the one after as well: faster for 32 x 32 outputs, but not for 64 x 64 ones, whose 12 loads an item keep
  // a wave's queue full by themselves (one item ahead and unconditional, an index past the end re-reads the last item:
  // 2.8% faster over 160 layers of 1 to 600 workgroups, up to 14%).  32 x 32: nothing is loaded past the end (a wave has 7
  // items at K = 3072, and one superfluous item each cost 10-20% of the whole kernel).
  if constexpr (NI * NJ > 1 && !ASYM) {
    Item<NI, NJ> A, B;
    auto load_or_last = [&](Item<NI, NJ>& it, int idx) { load(it, min(idx, items - 1)); };
    load_or_last(A, w);
    for (int idx = w; idx < items; idx += 2 * NW) {
      load_or_last(B, idx + NW);
      compute(A, idx);
      load_or_last(A, idx + 2 * NW);
      if (idx + NW < items) compute(B, idx + NW);
    }
  } else {
    constexpr int DEPTH = NI * NJ > 1 ? 1 : 2;
    Item<NI, NJ> set[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; d++)
      if (w + d * NW < items) load(set[d], w + d * NW);
    for (int idx = w; idx < items; idx += DEPTH * NW) {
#pragma unroll
      for (int d = 0; d < DEPTH; d++) {
        if (idx + d * NW < items) compute(set[d], idx + d * NW);
        if (idx + (d + DEPTH) * NW < items) load(set[d], idx + (d + DEPTH) * NW);
      }
    }
  }

  // ---- the eight partial sums meet in LDS; a thread sums register quads over the waves, in wave order ----
  constexpr int NQ = NI * NJ * 4;                      // register quads per wave
  float4* part = (float4*)smem;
#pragma unroll
  for (int i = 0; i < NI; i++)
#pragma unroll
    for (int j = 0; j < NJ; j++)
#pragma unroll
      for (int q = 0; q < 4; q++)
        part[((w * NQ) + (i * NJ + j) * 4 + q) * 64 + l] =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < (NQ * 64 + NT - 1) / NT; pass++) {
    const int slot = t + pass * NT;                    // (register quad, lane)
    if (NQ * 64 < NT && slot >= NQ * 64) continue;
    const int tq = slot >> 6, lane = slot & 63;
    float4 v = part[tq * 64 + lane];
#pragma unroll
    for (int ww = 1; ww < NW; ww++) {
      const float4 u = part[(ww * NQ + tq) * 64 + lane];
      v.x += u.x;
      v.y += u.y;
      v.z += u.z;
      v.w += u.w;
    }
    const int i = tq / (NJ * 4), j = tq / 4 % NJ, q = tq & 3;
    const int m = m0 + j * 32 + (lane & 31), n = n0 + i * 32 + 8 * q + 4 * (lane >> 5);
    if (m >= M || n >= N) continue;
    float o[4] = {v.x, v.y, v.z, v.w};
    const bool full = (N % 4) == 0 && n + 4 <= N;
    if (bias) {
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (n + e < N) o[e] += bf16_bits_to_f32(bias[n + e]);
    }
    if (OUT_F32) {
      float* dst = (float*)y + (size_t)m * N + n;
      if (full) {
        *(float4*)dst = make_float4(o[0], o[1], o[2], o[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
          if (n + e < N) dst[e] = o[e];
      }
    } else {
      uint16_t* dst = (uint16_t*)y + (size_t)m * N + n;
      if (full) {
        *(uint2*)dst = make_uint2(f32x2_to_bf16x2_bits(o[0], o[1]), f32x2_to_bf16x2_bits(o[2], o[3]));
      } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
          if (n + e < N) dst[e] = f32_to_bf16_bits(o[e]);
      }
    }
  }
}

template <int GS, bool OUT_F32, bool ASYM, int NI, int NJ>
static int launch_one(const uint16_t* xh, const uint8_t* xl, const uint16_t* sx, const uint16_t* zx, const void* blob,
                      const uint16_t* bias, int M, int N, int K, int r, void* y, hipStream_t s) {
  const BlobLayout L = blob_layout(N, K, r, GS);
  const char* bp = (const char*)blob;
  const int n_mt = (M + 32 * NJ - 1) / (32 * NJ), n_nt = (N + 32 * NI - 1) / (32 * NI);
  const long n_blocks = (long)n_mt * n_nt;
  if (n_blocks > 0x7FFFFFFFL) return DIROTQ_ERR_SHAPE;
  constexpr int SMEM = smem_bytes(NI, NJ);
  // (idempotent: two threads racing here would both set the same attribute)
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)w4a4_gemm_skinny_kernel<GS, OUT_F32, ASYM, NI, NJ>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return hip_failed(e);
    attr_done.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((w4a4_gemm_skinny_kernel<GS, OUT_F32, ASYM, NI, NJ>), dim3((unsigned)n_blocks), dim3(NT), SMEM, s, xh,
                     xl, sx, zx, (const uint16_t*)(bp + L.off_wh), (const uint8_t*)(bp + L.off_codes),
                     (const uint16_t*)(bp + L.off_sw), (const int16_t*)(bp + L.off_wsum), bias, M, N, K, r, y, n_nt);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

template <int GS>
static int launch_group(const uint16_t* xh, const uint8_t* xl, const uint16_t* sx, const uint16_t* zx, const void* blob,
                        const uint16_t* bias, int M, int N, int K, int r, void* y, int y_dtype, bool small, hipStream_t s) {
#define DIROTQ_SKINNY(F32, ASYM)                                                                        \
  return small ? launch_one<GS, F32, ASYM, 1, 1>(xh, xl, sx, zx, blob, bias, M, N, K, r, y, s)          \
               : launch_one<GS, F32, ASYM, 2, 2>(xh, xl, sx, zx, blob, bias, M, N, K, r, y, s)
  if (zx) {
    if (y_dtype) DIROTQ_SKINNY(true, true);
    DIROTQ_SKINNY(false, true);
  }
  if (y_dtype) DIROTQ_SKINNY(true, false);
  DIROTQ_SKINNY(false, false);
#undef DIROTQ_SKINNY
}

}  // namespace skinny

int launch_w4a4_gemm_skinny(const uint16_t* xh, const uint8_t* xl, const uint16_t* sx, const uint16_t* zx,
                            const void* blob, const uint16_t* bias, int M, int N, int K, int r, int g, void* y,
                            int y_dtype, bool small, hipStream_t s) {
  switch (g) {
    case 32: return skinny::launch_group<32>(xh, xl, sx, zx, blob, bias, M, N, K, r, y, y_dtype, small, s);
    case 64: return skinny::launch_group<64>(xh, xl, sx, zx, blob, bias, M, N, K, r, y, y_dtype, small, s);
    case 128: return skinny::launch_group<128>(xh, xl, sx, zx, blob, bias, M, N, K, r, y, y_dtype, small, s);
  }
  return DIROTQ_ERR_SHAPE;
}

}  // namespace dirotq
