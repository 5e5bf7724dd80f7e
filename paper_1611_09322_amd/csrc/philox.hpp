// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as
// easy as 1, 2, 3", SC 2011).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pse {

// hi:lo = a K, a product of 64-bit integers in four 32 x 32 + 64 bit
// multiply-adds (one instruction each).  The separate products for the low and
// the high word that the plain form compiles to take 203 integer
// multiplications a block against 140, and the fused x pass, which is bound by
// its vector instructions, 230 us against 214 (256^3, noise and forces).
__device__ __forceinline__ void mul64_wide(uint64_t a, uint64_t K, uint64_t &hi, uint64_t &lo) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), k0 = (uint32_t)K, k1 = (uint32_t)(K >> 32);
  const uint64_t p = (uint64_t)a0 * k0;
  const uint64_t t = (uint64_t)a1 * k0 + (uint32_t)(p >> 32);
  const uint64_t u = (uint64_t)a0 * k1 + (uint32_t)t;
  hi = (uint64_t)a1 * k1 + (uint32_t)(t >> 32) + (uint32_t)(u >> 32);
  lo = (u << 32) | (uint32_t)p;
}

__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B97F4A7C15ull;
      k1 += 0xBB67AE8584CAA73Bull;
    }
    uint64_t hi0, lo0, hi1, lo1;
    mul64_wide(c[0], 0xD2E7470EE14C6C93ull, hi0, lo0);
    mul64_wide(c[2], 0xCA5A826395121157ull, hi1, lo1);
    const uint64_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
  }
}

}  // namespace pse
