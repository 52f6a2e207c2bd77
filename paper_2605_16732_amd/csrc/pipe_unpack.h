// Expansion of packed codes to FP6 (E2M3) operands, shared by the pipelined kernels.
#pragma once

#include "dirotq_internal.h"

namespace dirotq {
namespace pipe {

__device__ __forceinline__ uint32_t and_or(uint32_t v, uint32_t mask, uint32_t o) {   // (the compiler would build it from
  uint32_t r;                                                                         // four instructions per three terms)
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(mask), "v"(o));
  return r;
}

// 16 sign-magnitude nibbles (two dwords) -> 16 FP6 numbers [s 00 mmm] in three dwords.  Six-bit field f takes a nibble
// that one of the shifts 0, +2, +4 over the 64-bit pair brings there (16 instructions); the order that results is the
// same for weights and tokens, so a dot product does not see it.
__device__ __forceinline__ void unpack16_fp6(uint32_t p0, uint32_t p1, uint32_t (&d)[3]) {
  const uint32_t s2 = p0 << 2, s4 = p0 << 4;
  const uint32_t t2 = __builtin_amdgcn_alignbit(p1, p0, 30), t4 = __builtin_amdgcn_alignbit(p1, p0, 28);
  d[0] = and_or(s4, 0x00800800u, and_or(s2, 0xE01E01E0u, p0 & 0x07007007u));
  d[1] = and_or(t4, 0x08008008u, and_or(t2, 0x01E01E01u, p1 & 0x70070070u));
  d[2] = and_or(t4, 0x80080080u, and_or(t2, 0x1C01C01Cu, and_or(s2, 0x02002000u, and_or(p0, 0x00700700u, (p1 >> 30) & 2u))));
}

// 16 unsigned nibbles -> 16 FP6 numbers [s 0 bbbb] with sign 0 (values 0 ... 15 in units of 2^-3), in the fields of unpack16_fp6
__device__ __forceinline__ void spread16u_fp6(uint32_t p0, uint32_t p1, uint32_t (&d)[3]) {
  const uint32_t s2 = p0 << 2, t2 = __builtin_amdgcn_alignbit(p1, p0, 30);
  d[0] = and_or(s2, 0xC03C03C0u, p0 & 0x0F00F00Fu);
  d[1] = and_or(t2, 0x03C03C03u, p1 & 0xF00F00F0u);
  d[2] = and_or(t2, 0x3C03C03Cu, p0 & 0x00F00F00u);
}

// 16 nibbles of either kind
template <bool ASYM>
__device__ __forceinline__ void half16_fp6(uint32_t p0, uint32_t p1, uint32_t (&d)[3]) {
  if constexpr (ASYM) spread16u_fp6(p0, p1, d);
  else unpack16_fp6(p0, p1, d);
}

// Field form of 32 symmetric codes, 16 bytes like the nibbles: dwords 0 1 2 and 3 of their six FP6 dwords (unpack16_fp6 of each
// half) with dwords 4 and 5 in the bits that are always zero there (two of every six, which fall exactly where the
// other two dwords have theirs set), so that expanding them takes 8 operations instead of 32 and no shift.  Kernel A
// writes it for the kernels B that expand every activation once per output tile.  M = 32768, K = 1152, N = 4608 353.5 -> 344.5 us,
// M = 4608, K = 3072, N = 12288 304.9 -> 295.8 (whole layer).  Asymmetric codes, whose nibbles expand in 16 operations: no
// gain (M = 1000, K = N = 3072: 53.2 -> 54.4).
constexpr uint32_t kOwn03 = 0xE79E79E7u, kOwn1 = 0x79E79E79u, kOwn2 = 0x9E79E79Eu;   // bits of dwords 0 and 3, 1, 2 that are their own
template <class V>
__device__ __forceinline__ void expand32_fp6(V p, uint32_t (&d0)[3], uint32_t (&d1)[3]) {
  d0[0] = p[0] & kOwn03;
  d0[1] = p[1] & kOwn1;
  d0[2] = p[2] & kOwn2;
  d1[0] = p[3] & kOwn03;
  d1[1] = and_or(p[3], ~kOwn03, p[2] & ~kOwn2);
  d1[2] = and_or(p[1], ~kOwn1, p[0] & ~kOwn03);
}
// 32 nibbles -> field form
__device__ __forceinline__ uint4 to_fields(uint4 n) {
  uint32_t d0[3], d1[3];
  unpack16_fp6(n.x, n.y, d0);
  unpack16_fp6(n.z, n.w, d1);
  return make_uint4(d0[0] | (d1[2] & ~kOwn03), d0[1] | (d1[2] & ~kOwn1), d0[2] | (d1[1] & ~kOwn2), d1[0] | (d1[1] & ~kOwn03));
}
// ... by two lanes l and l ^ 32, each with the 16 nibbles (and the two dwords of the result) of its half h
__device__ __forceinline__ uint2 to_fields_pair(uint2 n, int h) {
  uint32_t d[3];
  unpack16_fp6(n.x, n.y, d);
  const uint32_t o = __shfl_xor(d[2], 32);                  // dword 5 for half 0, dword 2 for half 1
  return h ? make_uint2(o | (d[1] & ~kOwn2), d[0] | (d[1] & ~kOwn03)) : make_uint2(d[0] | (o & ~kOwn03), d[1] | (o & ~kOwn1));
}

// The low (high) nibbles of the bytes of two dwords in one: nibble 2 i from byte i of a, 2 i + 1 from byte i of b
__device__ __forceinline__ uint32_t low_nibbles(uint32_t a, uint32_t b) { return (a & 0x0F0F0F0Fu) | ((b << 4) & 0xF0F0F0F0u); }
__device__ __forceinline__ uint32_t high_nibbles(uint32_t a, uint32_t b) { return ((a >> 4) & 0x0F0F0F0Fu) | (b & 0xF0F0F0F0u); }

// 16 unsigned nibbles -> 16 FP6 numbers [s 0 bbbb], in the fields that unpack16_fp6 gives them; the signs are those of `sign`
__device__ __forceinline__ void spread16_fp6(uint32_t p0, uint32_t p1, const uint32_t (&sign)[3], uint32_t (&d)[3]) {
  const uint32_t s2 = p0 << 2, t2 = __builtin_amdgcn_alignbit(p1, p0, 30);
  d[0] = and_or(sign[0], 0x20820820u, and_or(s2, 0xC03C03C0u, p0 & 0x0F00F00Fu));
  d[1] = and_or(sign[1], 0x08208208u, and_or(t2, 0x03C03C03u, p1 & 0xF00F00F0u));
  d[2] = and_or(sign[2], 0x82082082u, and_or(t2, 0x3C03C03Cu, p0 & 0x00F00F00u));
}

}  // namespace pipe
}  // namespace dirotq
