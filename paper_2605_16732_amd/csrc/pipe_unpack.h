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
