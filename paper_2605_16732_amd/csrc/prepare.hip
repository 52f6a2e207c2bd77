// Offline side of the layer (weight-fusion step of Section 4.2 of the paper, just before
// its forward-computation equation): W' = W Q in fp64, split at r, round-to-nearest
// INT4 with fp16 group scales; plus import/export of the prepared-weight blob and the
// bf16 transposed rotation operand.  None of this is on the per-step hot path.
#include "dirotq_internal.h"

namespace dirotq {

// ---- Qt[c][k] = bf16(Q[k][c]) ---------------------------------------------------
__global__ __launch_bounds__(256) void transpose_to_bf16_kernel(const float* __restrict__ Q, int K,
                                                                uint16_t* __restrict__ Qt) {
  __shared__ float tile[32][33];
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;   // bx: c block, by: k block
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5; // 32 x 8
  for (int i = ty; i < 32; i += 8) tile[i][tx] = Q[(size_t)(by + i) * K + bx + tx];   // tile[k][c]
  __syncthreads();
  for (int i = ty; i < 32; i += 8) Qt[(size_t)(bx + i) * K + by + tx] = f32_to_bf16_bits(tile[tx][i]);
}

int launch_prepare_rotation(const float* Q, int K, uint16_t* Qt, hipStream_t s) {
  hipLaunchKernelGGL(transpose_to_bf16_kernel, dim3(K / 32, K / 32), dim3(256), 0, s, Q, K, Qt);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

// ---- Wp[n][c] = fp32( sum_k W[n][k] Q[k][c] ) with fp64 accumulation ------------
// Bound: the fp64 matrix pipe (78.6 TFLOP/s; a 16x16x4 MFMA takes 64 cycles).  A workgroup owns 32 (n) x 32 (c) outputs and
// its four waves split K: wave w takes the runs of 16 k w, w + 4, ..., operands straight from global memory in the MFMA
// layout (fp32, made fp64 in registers: exact; 16 conversions and 10 loads beside 16 MFMAs), the next run's loads in
// flight; no LDS and no barrier in the loop.  The four partial sums meet in LDS, in wave order.  The unit of work is what a
// SIMD can be left with too many of: at N = K = 1536 a SIMD has 9 of these, and 4 or 5 of 32 x 16 outputs over all of K
// (the form before: 64 x 32 per workgroup through LDS).  Four waves per SIMD (128 registers; three: 5% slower).
// Fusion and quantizer, us: N = K = 1536 152 -> 135, 640 24.8 -> 19.1, N = 320, K = 1408 46.5 -> 34.0; N = 3072, K = 12288 15.4
// -> 14.4 ms (64 TFLOP/s).
// Within a run of 16 k lane group q = l / 16 takes k = 4 q .. 4 q + 3, one per MFMA, on both operands.
typedef __attribute__((ext_vector_type(4))) double f64x4;
constexpr int FN = 32, FC = 32, FK = 16, FW = 4;
__global__ __launch_bounds__(FW * 64, 4) void fuse_rotation_fp64_kernel(const float* __restrict__ W,
                                                                     const float* __restrict__ Q, int N, int K,
                                                                     float* __restrict__ Wp, long n_tiles, long per_xcd) {
  __shared__ __align__(16) f64x4 part[FW][4][64];
  const int t = threadIdx.x, l = t & 63, r16 = l & 15, q4 = (l >> 4) * 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n_ct = K / FC, runs = K / FK;
  // consecutive workgroup ids go to different XCDs: each XCD gets a run of tiles, c fastest (its rows of W stay in its L2)
  for (long b = blockIdx.x; b < 8 * per_xcd; b += gridDim.x) {
    const long tile = (b & 7) * per_xcd + (b >> 3);
    if (tile >= n_tiles) continue;
    const int n0 = (int)(tile / n_ct) * FN, c0 = (int)(tile % n_ct) * FC;
    const float* w0 = W + (size_t)min(n0 + r16, N - 1) * K + q4;
    const float* w1 = W + (size_t)min(n0 + 16 + r16, N - 1) * K + q4;
    const float* q0 = Q + (size_t)q4 * K + c0 + r16;
    float4 a[2][2];
    float bq[2][2][4];
    auto load = [&](int set, int k0) {
      a[set][0] = *(const float4*)(w0 + k0);
      a[set][1] = *(const float4*)(w1 + k0);
#pragma unroll
      for (int s = 0; s < 4; s++)
#pragma unroll
        for (int j = 0; j < 2; j++) bq[set][j][s] = q0[(size_t)(k0 + s) * K + 16 * j];
    };
    f64x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
    auto multiply = [&](int set) {
      const float av[2][4] = {{a[set][0].x, a[set][0].y, a[set][0].z, a[set][0].w}, {a[set][1].x, a[set][1].y, a[set][1].z, a[set][1].w}};
#pragma unroll
      for (int s = 0; s < 4; s++)
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int j = 0; j < 2; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[i][s], (double)bq[set][j][s], acc[i][j], 0, 0, 0);
    };
    if (w < runs) load(0, w * FK);
    for (int run = w; run < runs; run += 2 * FW) {
      if (run + FW < runs) load(1, (run + FW) * FK);
      multiply(0);
      if (run + 2 * FW < runs) load(0, (run + 2 * FW) * FK);
      if (run + FW < runs) multiply(1);
    }
    // wave w finishes tile (w / 2, w % 2)
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++) part[w][2 * i + j][l] = acc[i][j];
    __syncthreads();
    f64x4 sum = part[0][w][l];
#pragma unroll
    for (int ww = 1; ww < FW; ww++) sum += part[ww][w][l];
    // accumulator e of lane l: row 4 e + l / 16, column l % 16 of its 16 x 16 tile
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int n = n0 + (w >> 1) * 16 + 4 * e + (l >> 4);
      if (n < N) Wp[(size_t)n * K + c0 + (w & 1) * 16 + r16] = (float)sum[e];
    }
    __syncthreads();                                      // (before the next tile's sums)
  }
}

// ---- split + quantize rows of an fp32 matrix -------------------------------------
// Bound: one read of the matrix.  A thread takes 8 consecutive channels of a row at a time, the channels of the 16-bit part
// first (unit u: row u / (r/8)), then those of the 4-bit part from unit n_hi_pad on; a group is 4, 8 or 16 neighbouring
// lanes.  (One thread per group, consecutive threads on consecutive rows, read 4 of every 64 bytes: 24 -> 5 us at
// N = K = 1536, 910 -> 35 us at N = 3072, K = 12288.)
constexpr long QUANT_BLOCKS = 1 << 16;               // (more units than these have threads: several runs of 256 per block)
__global__ __launch_bounds__(256) void split_quantize_rows_kernel(const float* __restrict__ src, int rows,
                                                                  int K, int r, int g, long n_hi_pad, long n_blocks,
                                                                  uint16_t* __restrict__ hi,
                                                                  uint8_t* __restrict__ codes,
                                                                  uint16_t* __restrict__ scales,
                                                                  int16_t* __restrict__ wsum) {
  const int KL = K - r;
  for (long b = blockIdx.x; b < n_blocks; b += gridDim.x) {
    const long u = b * 256 + threadIdx.x;
    if (u < n_hi_pad) {                              // (a multiple of 256: the same for a whole block)
      if (u >= (long)rows * (r / 8)) continue;
      const long row = u / (r / 8);
      const int c = (int)(u % (r / 8)) * 8;
      const float4 lo = *(const float4*)(src + row * K + c), up = *(const float4*)(src + row * K + c + 4);
      uint4 o;
      o.x = f32_to_bf16_bits(lo.x) | (uint32_t)f32_to_bf16_bits(lo.y) << 16;
      o.y = f32_to_bf16_bits(lo.z) | (uint32_t)f32_to_bf16_bits(lo.w) << 16;
      o.z = f32_to_bf16_bits(up.x) | (uint32_t)f32_to_bf16_bits(up.y) << 16;
      o.w = f32_to_bf16_bits(up.z) | (uint32_t)f32_to_bf16_bits(up.w) << 16;
      *(uint4*)(hi + row * r + c) = o;
      continue;
    }
    const long v = u - n_hi_pad;                     // (groups do not straddle waves)
    const bool live = KL > 0 && v < (long)rows * (KL / 8);   // (whole groups are live or not)
    const long row = live ? v / (KL / 8) : 0;
    const int c = live ? (int)(v % (KL / 8)) * 8 : 0;
    float f[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (live) {
      const float4 lo = *(const float4*)(src + row * K + r + c), up = *(const float4*)(src + row * K + r + c + 4);
      f[0] = lo.x, f[1] = lo.y, f[2] = lo.z, f[3] = lo.w, f[4] = up.x, f[5] = up.y, f[6] = up.z, f[7] = up.w;
    }
    float amax = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; e++) amax = fmaxf(amax, fabsf(f[e]));
    for (int o = 1; o < g / 8; o <<= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
    uint16_t sbits;
    const float sf = group_scale(amax, sbits);
    const float inv = group_inv(sf);
    uint32_t p = 0;
    int sum = 0;
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const int q = quant_code(f[e], inv);
      p |= code_nibble(q) << (4 * e);
      sum += q;
    }
    for (int o = 1; o < g / 8; o <<= 1) sum += __shfl_xor(sum, o);   // |sum| <= 7 * 128
    if (!live) continue;
    *(uint32_t*)(codes + row * (KL / 2) + c / 2) = p;
    if (c % g == 0) {
      scales[(size_t)(c / g) * rows + row] = sbits;
      wsum[(size_t)(c / g) * rows + row] = (int16_t)sum;
    }
  }
}

int launch_prepare_weights(const float* W, const float* Q, int N, int K, int r, int g, void* blob,
                           float* scratch, hipStream_t s) {
  const BlobLayout L = blob_layout(N, K, r, g);
  char* bp = (char*)blob;
  // (only shapes whose fp32 scratch alone would exceed 2^45 bytes are refused; both kernels loop over their work)
  const long n_tiles64 = (long)((K + 63) / 64) * (long)((N + 63) / 64);
  if (n_tiles64 > 0x7FFFFFFFL) return DIROTQ_ERR_SHAPE;
  const long n_hi_pad = ((long)N * (r / 8) + 255) / 256 * 256;
  const long n_blocks = (n_hi_pad + (long)N * ((K - r) / 8) + 255) / 256;
  const long n_tiles = (long)(K / FC) * (long)((N + FN - 1) / FN), per_xcd = (n_tiles + 7) / 8;
  const unsigned grid = (unsigned)(8 * (per_xcd < (1 << 18) ? per_xcd : (1 << 18)));   // (beyond: several tiles each)
  hipLaunchKernelGGL(fuse_rotation_fp64_kernel, dim3(grid), dim3(FW * 64), 0, s, W, Q, N, K, scratch, n_tiles, per_xcd);
  hipError_t e0 = hipGetLastError();
  if (e0 != hipSuccess) return hip_failed(e0);      // nothing else is enqueued on an unwritten scratch
  hipLaunchKernelGGL(split_quantize_rows_kernel, dim3((unsigned)(n_blocks < QUANT_BLOCKS ? n_blocks : QUANT_BLOCKS)),
                     dim3(256), 0, s, scratch, N, K, r, g, n_hi_pad, n_blocks, (uint16_t*)(bp + L.off_wh),
                     (uint8_t*)(bp + L.off_codes), (uint16_t*)(bp + L.off_sw), (int16_t*)(bp + L.off_wsum));
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

// ---- import / export of the blob -------------------------------------------------
__global__ __launch_bounds__(256) void import_kernel(const uint16_t* __restrict__ Wh,
                                                     const int8_t* __restrict__ codes,
                                                     const uint16_t* __restrict__ sw, int N, int K, int r,
                                                     int g, uint16_t* __restrict__ bwh,
                                                     uint8_t* __restrict__ bq, uint16_t* __restrict__ bsw,
                                                     int16_t* __restrict__ bwsum) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n_wh = (long)N * r, n_q = (long)N * (K - r) / 2;
  const int G = (K - r) / g;
  if (i < n_wh) bwh[i] = Wh[i];
  // (codes outside [-7, 7] are clamped: the symmetric 4-bit quantizer never produces -8)
  auto clamp7 = [](int q) { return min(max(q, -7), 7); };
  if (i < n_q) bq[i] = (uint8_t)(code_nibble(clamp7(codes[2 * i])) | (code_nibble(clamp7(codes[2 * i + 1])) << 4));
  if (i < (long)N * G) {
    const int n = (int)(i / G), j = (int)(i % G);
    bsw[(size_t)j * N + n] = sw[i];
    const int8_t* c = codes + (size_t)n * (K - r) + (size_t)j * g;
    int sum = 0;
    for (int p = 0; p < g; p++) sum += clamp7(c[p]);
    bwsum[(size_t)j * N + n] = (int16_t)sum;
  }
}

__global__ __launch_bounds__(256) void export_kernel(const uint16_t* __restrict__ bwh,
                                                     const uint8_t* __restrict__ bq,
                                                     const uint16_t* __restrict__ bsw, int N, int K, int r,
                                                     int g, uint16_t* __restrict__ Wh,
                                                     int8_t* __restrict__ codes, uint16_t* __restrict__ sw) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n_wh = (long)N * r, n_q = (long)N * (K - r) / 2;
  const int G = (K - r) / g;
  if (Wh && i < n_wh) Wh[i] = bwh[i];
  if (codes && i < n_q) {
    const int b = bq[i];
    codes[2 * i] = (int8_t)nibble_code(b & 15);
    codes[2 * i + 1] = (int8_t)nibble_code(b >> 4);
  }
  if (sw && i < (long)N * G) {
    const int n = (int)(i / G), j = (int)(i % G);
    sw[i] = bsw[(size_t)j * N + n];
  }
}

static long max3(long a, long b, long c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }

int launch_import_weights(const uint16_t* Wh, const int8_t* codes, const uint16_t* sw, int N, int K, int r,
                          int g, void* blob, hipStream_t s) {
  const BlobLayout L = blob_layout(N, K, r, g);
  char* bp = (char*)blob;
  const long n = max3((long)N * r, (long)N * (K - r) / 2, (long)N * ((K - r) / g));
  if (n == 0) return DIROTQ_OK;
  hipLaunchKernelGGL(import_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Wh, codes, sw, N, K,
                     r, g, (uint16_t*)(bp + L.off_wh), (uint8_t*)(bp + L.off_codes),
                     (uint16_t*)(bp + L.off_sw), (int16_t*)(bp + L.off_wsum));
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

int launch_export_weights(const void* blob, int N, int K, int r, int g, uint16_t* Wh, int8_t* codes,
                          uint16_t* sw, hipStream_t s) {
  const BlobLayout L = blob_layout(N, K, r, g);
  const char* bp = (const char*)blob;
  const long n = max3((long)N * r, (long)N * (K - r) / 2, (long)N * ((K - r) / g));
  if (n == 0) return DIROTQ_OK;
  hipLaunchKernelGGL(export_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     (const uint16_t*)(bp + L.off_wh), (const uint8_t*)(bp + L.off_codes),
                     (const uint16_t*)(bp + L.off_sw), N, K, r, g, Wh, codes, sw);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DIROTQ_OK : hip_failed(e);
}

}  // namespace dirotq
