// Proposals and acceptance of the Metropolis chains (App. C, "Efficient Sampling Strategy"),
// shared by the kernel per step and the kernel that keeps its chains through a sweep.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tdo {

struct Philox4x32 {
  uint32_t c[4];
};

// Philox4x32 with 10 rounds: each round forms the 64-bit products of counter
// words 0 and 2 with the two round multipliers, then mixes their high halves
// with counter words 1 and 3 and the round key; the key is bumped by the two
// Weyl increments between rounds.
__device__ __forceinline__ Philox4x32 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                               uint32_t k1) {
  constexpr uint32_t kMul0 = 0xD2511F53u, kMul1 = 0xCD9E8D57u;
  constexpr uint32_t kWeyl0 = 0x9E3779B9u, kWeyl1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)kMul0 * c0, p1 = (uint64_t)kMul1 * c2;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += kWeyl0;
    k1 += kWeyl1;
  }
  return Philox4x32{{c0, c1, c2, c3}};
}

// Proposal t of a chain on (alpha, beta): flips bits of (a, b) and returns the acceptance uniform.
__device__ __forceinline__ double propose_move(uint64_t& a, uint64_t& b, int n, uint64_t t, uint32_t chain, uint64_t seed,
                                               uint64_t pair_thr) {
  const Philox4x32 r = philox10((uint32_t)t, (uint32_t)(t >> 32), chain, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
  // as two masks: a branch that writes a or b puts both on the stack (a proposal of 2000 chains 2.2 -> 2.8 us)
  uint64_t fa, fb;
  if ((uint64_t)r.c[0] < pair_thr) {
    fa = fb = 1ull << (int)(((uint64_t)r.c[1] * (uint64_t)n) >> 32);
  } else {
    const int j = (int)(((uint64_t)r.c[1] * (uint64_t)(2 * n)) >> 32);
    fa = j < n ? 1ull << j : 0ull;
    fb = j < n ? 0ull : 1ull << (j - n);
  }
  a ^= fa;
  b ^= fb;
  return ((double)r.c[2] + 0.5) * 0x1p-32;
}

// Proposal t of a diagonal chain: flips one site of a.
__device__ __forceinline__ double propose_diag(uint64_t& a, int n, uint64_t t, uint32_t chain, uint64_t seed) {
  const Philox4x32 r = philox10((uint32_t)t, (uint32_t)(t >> 32), chain, 1u, (uint32_t)seed, (uint32_t)(seed >> 32));
  a ^= 1ull << (int)(((uint64_t)r.c[1] * (uint64_t)n) >> 32);
  return ((double)r.c[2] + 0.5) * 0x1p-32;
}

// |rho'|^2 / |rho|^2, or |rho'| / |rho| on the diagonal, in FP64 from the real parts of log rho.
__device__ __forceinline__ double accept_ratio(float lr_new, float lr_old, bool diag) {
  const double d = (double)lr_new - (double)lr_old;
  return exp(diag ? d : 2.0 * d);
}

}  // namespace tdo
