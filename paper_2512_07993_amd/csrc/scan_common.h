// Pieces shared by the two scan variants (scan.hip: two passes over K; scan_fused.hip: one).
#pragma once

#include "common.h"

namespace skipkv {

constexpr float kScale2 = 0.08838834764831845f * 1.4426950408889634f;  // log2(e) / sqrt(128)
// A row's sum relative to a reference that its first logits fixed is taken as it is between these: further down terms
// may be missing, further up the sums of a head's 1e5 records, which may all have that reference, need not fit any more.
constexpr float kMinRowSum = 1e-30f, kMaxRowSum = 1e30f;
constexpr float kRescaleSlack = 16.f;  // a lane's reference is refreshed when a logit exceeds it by this much (log2 units)

// Item `item` of a two-pass scan: the head, and which of the units (runs, chunks) of all sequences.  Each head's units are
// taken from another place on, a golden ratio of them further than the head's before: the number of workgroups is often a multiple
// of the units, and a workgroup would meet the same ones in every head it comes to, all of them or none left by the single-pass
// scan.  (Bf16, 32 layers x 8 heads, us, both passes, all heads from the first unit on / like this: 16 sequences of 4 K tokens, one of
// them left: 1237 / 217; 8 of 4 K, four left: 807 / 347; everything left or forced: the same.)
__device__ __forceinline__ void two_pass_item(uint32_t item, uint32_t units, int &lh, int &unit) {
  const uint32_t head = item / units, x = item - head * units + (uint32_t)(((uint64_t)(head * 0x9E3779B9u) * units) >> 32);
  lh = (int)head;
  unit = (int)(x >= units ? x - units : x);
}

template <int DT>
struct Tr;
template <>
struct Tr<SKIPKV_BF16> {
  static constexpr int ESZ = 2, ROWB = 256, LSTR = 272;  // LDS row stride: +16 B so that 16-byte reads of 8 consecutive rows hit distinct banks
};
template <>
struct Tr<SKIPKV_F32> {
  static constexpr int ESZ = 4, ROWB = 512, LSTR = 528;
};

// acc[T] += Q[16T.., :] * K[token, :]^T for the lane's token.  Both operands use the same
// (arbitrary but identical) assignment of head-dim slices to MFMA k-steps: lane group g covers
// bytes [64g, 64g+64) of a bf16 row over the 4 k-steps, so every lane reads contiguous 16-byte
// pieces.
template <int DT, int NT>
__device__ __forceinline__ void tile_logits(const char *qt, const char *krow, int c16, int g, f32x4 (&acc)[NT]) {
  static_assert(DT == SKIPKV_F32, "the bf16 scans keep their query fragments in registers");
  constexpr int LSTR = Tr<DT>::LSTR;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const float4 bfrag = *reinterpret_cast<const float4 *>(krow + c * 64 + g * 16);
#pragma unroll
    for (int T = 0; T < NT; ++T) {
      const float4 afrag = *reinterpret_cast<const float4 *>(qt + (16 * T + c16) * LSTR + c * 64 + g * 16);
      acc[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(afrag.x, bfrag.x, acc[T], 0, 0, 0);
      acc[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(afrag.y, bfrag.y, acc[T], 0, 0, 0);
      acc[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(afrag.z, bfrag.z, acc[T], 0, 0, 0);
      acc[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(afrag.w, bfrag.w, acc[T], 0, 0, 0);
    }
  }
}

}  // namespace skipkv
