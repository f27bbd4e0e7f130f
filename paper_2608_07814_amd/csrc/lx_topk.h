// Top-k of one token's router logits by one wavefront.
//
// The k largest logits in descending order, equal logits ordered by the
// lower expert index, NaN below every number; the weights are the softmax of
// the chosen logits (= the full softmax restricted to them and renormalised).
// Logits come from the skinny GEMM over implicit 32-row tiles: either final
// ([T][E] fp32, S <= 1) or S partial tiles per (32-row tile, 64-column tile)
// item, added here in split order (run-to-run deterministic).
// Lane l holds experts l, l + 64, ...; k rounds of a wavefront-wide (value,
// lower index) maximum; lane j < k returns the j-th choice.
#pragma once

#include "lx_internal.h"

namespace lx {

__device__ __forceinline__ bool topk_better(float v, int i, float bv, int bi) {
  return v > bv || (v == bv && i < bi);
}

// (value, index) of lane l's partner under a DPP pattern (all lanes valid).
template <int CTRL>
__device__ __forceinline__ void dpp_pair(float v, int i, float& ov, int& oi) {
  ov = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
  oi = __builtin_amdgcn_update_dpp(0, i, CTRL, 0xF, 0xF, false);
}

// Wavefront-wide best (value, lower index) of every lane's candidate, on
// every lane. The order is total, so the winner does not depend on the
// combining pattern: inside each row of 16 lanes by DPP (rotate by 8, by 4,
// then the quad permutations xor 2 and xor 1), across the four rows by swaps of
// neighbouring rows and of the wavefront's halves (SWAP: the shorter chain) or by
// two lane exchanges through LDS (fewer VALU instructions, the better where
// wavefronts fill the chip).
template <bool SWAP>
__device__ __forceinline__ void wave_best(float& bv, int& bi) {
  float ov;
  int oi;
  dpp_pair<0x128>(bv, bi, ov, oi);  // row_ror:8
  if (topk_better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
  dpp_pair<0x124>(bv, bi, ov, oi);  // row_ror:4
  if (topk_better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
  dpp_pair<0x4E>(bv, bi, ov, oi);   // quad_perm [2, 3, 0, 1]
  if (topk_better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
  dpp_pair<0xB1>(bv, bi, ov, oi);   // quad_perm [1, 0, 3, 2]
  if (topk_better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
  if constexpr (SWAP) {
    // a swap of a register with itself leaves one row (half) of each pair in both
    // places of the first result and the other in both of the second
    auto better_of = [&](uint32_t v0, uint32_t v1, uint32_t i0, uint32_t i1) {
      const float f0 = __builtin_bit_cast(float, v0), f1 = __builtin_bit_cast(float, v1);
      const bool b = topk_better(f1, (int)i1, f0, (int)i0);
      bv = b ? f1 : f0;
      bi = b ? (int)i1 : (int)i0;
    };
    {
      const uint32_t v = __builtin_bit_cast(uint32_t, bv);
      const auto pv = __builtin_amdgcn_permlane16_swap(v, v, false, false);
      const auto pi = __builtin_amdgcn_permlane16_swap((uint32_t)bi, (uint32_t)bi, false, false);
      better_of(pv[0], pv[1], pi[0], pi[1]);
    }
    {
      const uint32_t v = __builtin_bit_cast(uint32_t, bv);
      const auto pv = __builtin_amdgcn_permlane32_swap(v, v, false, false);
      const auto pi = __builtin_amdgcn_permlane32_swap((uint32_t)bi, (uint32_t)bi, false, false);
      better_of(pv[0], pv[1], pi[0], pi[1]);
    }
  } else {
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      ov = __shfl_xor(bv, off, 64);
      oi = __shfl_xor(bi, off, 64);
      if (topk_better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
  }
}

// One token per wavefront, E <= 64 PER. Every lane of the wavefront must call it
// (wavefront-wide shuffles).
template <int PER, bool SWAP>
__device__ __forceinline__ void topk_token(const float* __restrict__ logits, const float* __restrict__ part, int S,
                                           int E, int k, int t, int& id, float& weight) {
  const int lane = threadIdx.x & 63;
  const int ntn = (E + kSkinnyBN - 1) / kSkinnyBN;
  float v[PER];
  const int ti = t / kSkinnyBM, row = t % kSkinnyBM;
  if (S <= 1) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = lane + 64 * j;
      v[j] = logits[(int64_t)t * E + (e < E ? e : E - 1)];
    }
  } else {
    // slot (item * S + split), item = ti * ntn + e / 64; inside a slot
    // [wavefront = (e % 64) / 32][row][e % 32]; all PER loads of a split together,
    // of 4 splits (2 for PER = 8, which keeps 8 wavefronts per SIMD: 82 VGPRs
    // took 166 instead of 154 us at T = 16384, E = 384, k = 32). Offsets: at most
    // kSplitCap slots are in use where S > 1.
    static_assert((int64_t)kSplitCap * kSkinnyBM * kSkinnyBN < ((int64_t)1 << 31), "32-bit slot offsets");
    int q[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e0 = lane + 64 * j, e = e0 < E ? e0 : E - 1;
      q[j] = (ti * ntn + e / 64) * S * (kSkinnyBM * kSkinnyBN) + ((e & 63) >> 5) * (32 * 32) + row * 32 + (e & 31);
      v[j] = part[q[j]];
    }
#pragma unroll (PER <= 4 ? 4 : 2)
    for (int sp = 1; sp < S; ++sp) {
#pragma unroll
      for (int j = 0; j < PER; ++j) v[j] += part[q[j] + sp * (kSkinnyBM * kSkinnyBN)];
    }
  }
  uint32_t taken = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (lane + 64 * j >= E) taken |= 1u << j;
    v[j] = v[j] == v[j] ? v[j] : -INFINITY;
  }
  float my_v = -INFINITY;
  int my_i = 0;
  for (int round = 0; round < k; ++round) {
    float bv = -INFINITY;
    int bi = 0x7FFFFFFF;
#pragma unroll
    for (int j = 0; j < PER; ++j)
      if (!((taken >> j) & 1u) && topk_better(v[j], lane + 64 * j, bv, bi)) {
        bv = v[j];
        bi = lane + 64 * j;
      }
    wave_best<SWAP>(bv, bi);
    // every lane holds the winner (k <= E: an untaken expert always exists)
    if ((bi & 63) == lane) taken |= 1u << (bi >> 6);
    if (lane == round) {
      my_v = bv;
      my_i = bi;
    }
  }
  const float m = __shfl(my_v, 0, 64);  // the largest chosen logit
  const float ex = lane < k ? expf(my_v - m) : 0.f;
  float s = ex;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);  // same tree on every lane
  id = my_i;
  weight = ex / s;
}

}  // namespace lx
