// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): the counter-based
// generator behind every uniform of the path (Sec. IV.b random-number
// component; Sec. III reproducibility).  Key = (seed lo, seed hi).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mg {

constexpr uint32_t PHILOX_M0 = 0xD2511F53u, PHILOX_M1 = 0xCD9E8D57u;
constexpr uint32_t PHILOX_W0 = 0x9E3779B9u, PHILOX_W1 = 0xBB67AE85u;

// a ^ b ^ c in one instruction
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// One round of two words is two 64-bit multiply-adds and two three-way xors,
// which bound the draw: 5e6 uniforms (hit or miss) in 12.6 us, 17.0 us with
// the halves of the products and the xors one by one.
__device__ __forceinline__ void philox10(uint32_t& c0, uint32_t& c1, uint32_t& c2, uint32_t& c3,
                                         uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += PHILOX_W0;
      k1 += PHILOX_W1;
    }
    // both halves from one 64-bit multiply-add instruction
    const uint64_t p0 = (uint64_t)PHILOX_M0 * c0, p1 = (uint64_t)PHILOX_M1 * c2;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t n0 = xor3(hi1, c1, k0), n2 = xor3(hi0, c3, k1);
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
}

__device__ __forceinline__ double bits_to_u(uint32_t lo, uint32_t hi) {
  const uint64_t w = ((uint64_t)hi << 32) | lo;
  return ((double)(w >> 11) + 0.5) * 0x1p-53;
}

}  // namespace mg
