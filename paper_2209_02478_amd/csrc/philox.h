// Counter-based random numbers for dropout: Philox4x32 with ten rounds (Salmon, Moraes, Dror,
// Shaw, SC'11).  A mask is a pure function of (seed, iteration, site, element number), so the
// forward of a checkpointed layer that is run again before its backward meets the masks of its
// first run without anything being stored.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace mk {

// a * m, all 64 bits, in one instruction (v_mad_u64_u32 issues as fast as either half's product alone)
__device__ __forceinline__ uint64_t mul_wide(uint32_t a, uint32_t m) {
  uint64_t d, carry;
  asm("v_mad_u64_u32 %0, %1, %2, %3, 0" : "=v"(d), "=s"(carry) : "v"(a), "s"(m));
  return d;
}
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }

__device__ __forceinline__ uint4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                               uint32_t k1) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // (the site, in c2 at first, is the same in every lane: a scalar product)
    const uint64_t p0 = mul_wide(c0, M0), p1 = r ? mul_wide(c2, M1) : (uint64_t)c2 * M1;
    c0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    c1 = (uint32_t)p1;
    c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c3 = (uint32_t)p0;
    k0 += W0;
    k1 += W1;
  }
  return make_uint4(c0, c1, c2, c3);
}

// the four words of block `block` (elements 4*block .. 4*block+3) at this site and iteration
__device__ __forceinline__ uint4 drop_words(const DropDesc& d, uint64_t block) {
  return philox4x32_10((uint32_t)block, (uint32_t)(block >> 32), d.site, d.step, d.k0, d.k1);
}

// Attention probabilities [B, nh, L, L]: every row of L keys is padded to a multiple of four, so
// four neighbouring keys of one query share a block whatever L is:
//   block = row * ceil(L / 4) + key / 4,  row = (b * nh + h) * L + query,  word = key % 4.
__device__ __forceinline__ uint4 attn_drop_words(const DropDesc& d, int64_t row, int L4q, int key) {
  return drop_words(d, (uint64_t)row * (uint64_t)L4q + (uint64_t)(key >> 2));
}
// The words w of lane t of each four lanes are of query t and four keys; this lane's key is number lane % 4
// of them: keep[t] is whether query t keeps it.  Every lane's four decisions are packed as bits and go round
// the four lanes by DPP.  (12 padded samples of 153-397 tokens, 12 heads: dK/dV 60 us with cross-lane reads of
// the words and the products' halves apart, 42 so; the forward, wide products alone, 30 -> 24.)
__device__ __forceinline__ void quad_keep(const uint4& w, uint32_t thr, int lane, bool (&keep)[4]) {
  const int bits = (w.x >= thr ? 1 : 0) | (w.y >= thr ? 2 : 0) | (w.z >= thr ? 4 : 0) | (w.w >= thr ? 8 : 0);
  const int mine = 1 << (lane & 3);
  keep[0] = __builtin_amdgcn_update_dpp(0, bits, 0x00, 0xF, 0xF, true) & mine;
  keep[1] = __builtin_amdgcn_update_dpp(0, bits, 0x55, 0xF, 0xF, true) & mine;
  keep[2] = __builtin_amdgcn_update_dpp(0, bits, 0xAA, 0xF, 0xF, true) & mine;
  keep[3] = __builtin_amdgcn_update_dpp(0, bits, 0xFF, 0xF, 0xF, true) & mine;
}

}  // namespace mk
