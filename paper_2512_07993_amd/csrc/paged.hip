// Paged KV cache (Appendix, "System-Level Evaluation on vLLM"): the translation from logical
// tokens to block slots, done once per step for the whole batch.  The kernels that touch K and V
// then address rows through this map instead of through the block table.
#include <algorithm>

#include "common.h"

namespace skipkv {

__global__ void k_row_map_reset(int32_t *seq_bad, int n, PlanHeader *hdr) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0 && hdr) reset_header(hdr);
  if (i < n) seq_bad[i] = 0;
}

// grid = (x, batch, groups of heads): the blocks of column (b, group) walk the tokens of sequence b, whose blocks are
// looked up once for the heads of the group.
__global__ void __launch_bounds__(256) k_row_map(RowMapArgs a, int heads) {
  const int b = blockIdx.y, lh0 = blockIdx.z * heads, lh1 = min(lh0 + heads, a.n_lh);
  const int tok0 = a.seq_off[b], n_tok = a.seq_off[b + 1] - tok0;
  const int32_t *table = a.block_table + (int64_t)b * a.table_stride;
  const int first_h = lh0 % a.n_kv_heads;
  const uint32_t first_row = (uint32_t)(lh0 / a.n_kv_heads) * (uint32_t)a.unit_layer + (uint32_t)first_h * (uint32_t)a.unit_head;
  const uint32_t next_layer = (uint32_t)a.unit_layer - (uint32_t)(a.n_kv_heads - 1) * (uint32_t)a.unit_head;
  bool bad = false;
  for (int t = blockIdx.x * 256 + threadIdx.x; t < n_tok; t += gridDim.x * 256) {
    const int bi = t / a.block_size;
    int p = bi < a.table_stride ? table[bi] : -1;
    if (p < 0 || p >= a.n_blocks) {
      bad = true;
      p = 0;
    }
    // (a slot row fits 31 bits, so its parts may wrap)
    const uint32_t row = (uint32_t)p * (uint32_t)a.unit_block + (uint32_t)(t - bi * a.block_size) * (uint32_t)a.unit_tok;
    uint32_t head_row = first_row;
    int h = first_h;
    int32_t *out = a.row_map + (int64_t)lh0 * a.total_tokens + tok0 + t;
    for (int lh = lh0; lh < lh1; ++lh, out += a.total_tokens) {
      *out = (int32_t)(head_row + row);
      const bool wrap = ++h == a.n_kv_heads;
      head_row += wrap ? next_layer : (uint32_t)a.unit_head;
      h = wrap ? 0 : h;
    }
  }
  if (__any(bad) && (threadIdx.x & 63) == 0) {
    for (int lh = lh0; lh < lh1; ++lh) a.seq_bad[lh * a.batch + b] = 1;  // every writer stores the same value
    if (a.dev_status) atomicOr(a.dev_status, SKIPKV_DEV_BAD_BLOCK_TABLE);
  }
}

hipError_t launch_row_map(const RowMapArgs &a, hipStream_t st) {
  if (a.batch == 0 || a.n_lh == 0) return hipSuccess;
  const int n_flags = a.n_lh * a.batch;
  if (!a.flags_reset) hipLaunchKernelGGL(k_row_map_reset, dim3((n_flags + 255) / 256), dim3(256), 0, st, a.seq_bad, n_flags, a.hdr);
  // Maps per head: eight workgroups per sequence, each for as many heads, up to eight, as leave some 8192 in all: with one
  // for every head they are bound by their number.  They are not dealt out by the mean length: one sequence may be much
  // longer than the others.  With their reset, us, one head / the heads of this rule each:
  //   28 layers x 4 heads, 64 x 1152 tokens: 42 / 18;  65536 + 63 x 600 tokens: 65 / 43 (one workgroup per 1024 tokens
  //   of the mean: 19 and 237);  32 x 8, 16 x 4096: 32 / 20;  1 x 16384: 15 / 16.
  const int heads = (int)std::min<int64_t>(8, std::max<int64_t>(1, 8 * (int64_t)a.batch * a.n_lh / 8192));
  hipLaunchKernelGGL(k_row_map, dim3(a.n_lh > 1 ? 8 : 64, a.batch, (a.n_lh + heads - 1) / heads), dim3(256), 0, st, a, heads);
  return hipGetLastError();
}

}  // namespace skipkv
