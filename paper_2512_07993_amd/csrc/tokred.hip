// Token redundancy (Sec. 4.1 "Token Redundancy Score", Eq. 5): per head, with Kbar the rows of K
// scaled to unit length, R[t] = mean over rows i of softmax_j(Kbar Kbar^T)[i, t].
//
// The cosine matrix is symmetric and its entries lie in [-1, 1], so no running maximum is
// needed: with E = exp(Kbar Kbar^T), l = E 1 (row sums) and R = (1/N) E (1 / l).  Both are sums
// over the same symmetric N x N matrix, which is never stored:
//   sweep 1:  l_i = sum_j e_ij
//   sweep 2:  R_i = (1/N) sum_j e_ij / l_j
// with e_ij = exp2(<k_i, k_j> * c_i * c_j), where c = sqrt(log2 e) / (||k|| + eps) carries both the
// normalisation and the change of base.  The dot products run on the bf16 matrix cores with the
// RAW keys (exact products, fp32 accumulation; fp32 caches are rounded to bf16 first) and the
// scale factors are applied to the accumulators.
//
// Only the blocks at and right of the diagonal are computed.  One workgroup owns 256 rows (32 per
// wave: the A operands stay in registers) and walks the 64-column blocks from its own rows to the
// end of the sequence, staged through LDS and shared by the 8 waves; the next block is fetched
// while the current one is multiplied.  The 64 x 64 squares on the diagonal are
// computed in full and give row sums only; every block right of them gives e_ij both to row i
// (weighted with column j's factor) and, by symmetry, to row j (weighted with row i's factor):
// the column sums of a block are reduced over the workgroup's rows and added to the row's total.
//
// What bounds a sweep: vector instructions, and then power.  Per lane an entry costs two scale multiplies, an exponential (two
// issue slots) and two fmas, and a matrix instruction's 16 cycles for four; counters show the vector pipe issuing for 75 % of a SIMD's
// cycles (62 % when the products of a tile came before its exponentials instead of among those of the tile before: the two
// hardly overlapped) and the matrix pipe busy for 36 %, at a clock that has come down from 2.25 to 2.13 GHz meanwhile.  So: the
// products of a tile are issued among the vector instructions of the one before; 32 rows per wave in some 115 registers, which lets
// four waves share a SIMD (64 rows took 237: two waves); column blocks go straight to LDS, their addresses a scalar base and one
// offset per lane; one barrier per column block and two LDS buffers; column sums of four column tiles reduced over the lane
// groups together (three permutes); squares of 64 instead of 256 on the diagonal.  32 layers x 8 heads, 4 x 2-4 K tokens:
// the sweeps take 1640 + 1690 us (1780 + 1805 with the products first and addresses formed in 64 bits; 2376 each with 64 rows
// per wave).
// Totals are accumulated across workgroups as 64-bit FIXED-POINT integers (integer addition is
// associative: the result does not depend on the order in which workgroups arrive, and the
// conversion of an fp32 partial sum is exact at the chosen scale for all but negligible terms),
// then turned back into fp32 by a small kernel after each sweep.
#include <algorithm>
#include <type_traits>

#include "scan_dev.h"

namespace skipkv {

namespace {

constexpr int kRows = kTokredRows;  // rows per workgroup
constexpr int kWaves = 8;            // waves per workgroup
constexpr int kTW = kRows / 16 / kWaves;  // 16-row tiles per wave
constexpr int kCols = 64;            // columns per staged block
constexpr int kColB = kCols * 256;   // bytes per staged block
constexpr float kSqrtLog2e = 1.2011224087864498f;
// fixed-point scales of the two accumulations: row sums l <= e * N (2^40: room for N up to 2^21 tokens,
// resolution 1e-12 against terms >= 0.37), and R <= e^2 / N... <= 8 (2^50: resolution 1e-15 against R ~ 1/N)
constexpr float kFix1 = 1099511627776.f, kFix2 = 1125899906842624.f;

__device__ __forceinline__ void add_fixed(unsigned long long *dst, float x, float scale) {
  atomicAdd(dst, (unsigned long long)__float2ll_rn(x * scale));  // x >= 0
}

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {  // two fp32 -> packed bf16, nearest even
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
  bf16x2_t v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

// 16 bytes of a key row as bf16: piece p (8 elements) of the row at `row_ptr`.
template <int DT>
__device__ __forceinline__ uint4 load_piece_bf16(const char *row_ptr, int piece) {
  if constexpr (DT == SKIPKV_BF16) {
    return *reinterpret_cast<const uint4 *>(row_ptr + piece * 16);
  } else {
    const float4 x = *reinterpret_cast<const float4 *>(row_ptr + piece * 32);
    const float4 y = *reinterpret_cast<const float4 *>(row_ptr + piece * 32 + 16);
    return make_uint4(pack2(x.x, x.y), pack2(x.z, x.w), pack2(y.x, y.y), pack2(y.z, y.w));
  }
}

// c[t] = sqrt(log2 e) / (||k_t|| + eps) for every key row; 16 lanes per row.
template <int DT>
__global__ void __launch_bounds__(256) k_key_scale(TokRedArgs a) {
  constexpr int ESZ = DT == SKIPKV_BF16 ? 2 : 4;
  const int lane16 = threadIdx.x & 15;
  const int64_t n_rows = (int64_t)a.n_layers * a.n_kv_heads * a.total_tokens;
  for (int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4; row < n_rows; row += ((int64_t)gridDim.x * 256) >> 4) {
    const int64_t lh = row / a.total_tokens, t = row % a.total_tokens;
    const int l = (int)(lh / a.n_kv_heads), h = (int)(lh % a.n_kv_heads);
    const int64_t slot = a.row_map ? (int64_t)a.row_map[t] : t;  // paged cache: the token's slot row
    const char *p = static_cast<const char *>(a.k) + ((int64_t)l * a.stride_layer + (int64_t)h * a.stride_head + slot * a.stride_tok) * ESZ;
    float ss = 0.f;
    if constexpr (DT == SKIPKV_BF16) {
      const uint4 v = *reinterpret_cast<const uint4 *>(p + lane16 * 16);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = __uint_as_float(w[i] << 16), y = __uint_as_float(w[i] & 0xFFFF0000u);
        ss += x * x + y * y;
      }
    } else {
      // the dot products use the keys rounded to bf16: the norm is taken of the same values
      const uint4 v = load_piece_bf16<DT>(p, lane16);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = __uint_as_float(w[i] << 16), y = __uint_as_float(w[i] & 0xFFFF0000u);
        ss += x * x + y * y;
      }
    }
    ss = row16_sum(ss);
    if (lane16 == 0) {
      a.scale[row] = kSqrtLog2e / (sqrtf(ss) + 1e-12f);
      a.acc[row] = 0ull;  // the first sweep's accumulator
    }
  }
}

// Sums of four columns' partial sums over the four lane groups: lane (g, c16) gets the total of v_g's column.
// The first swap leaves (v0 | v2) and (v1 | v3) in the wave's halves, the second one sorts the rows.
__device__ __forceinline__ float sum_lane_groups(float v0, float v1, float v2, float v3) {
  typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
  auto swap32 = [](float x, float y) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(swap32(v0, v2)), __float_as_uint(swap32(v1, v3)), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// SWEEP 1: adds every row's sum of e_ij into acc (scale kFix1).  SWEEP 2: adds R (scale kFix2).
// SIMPLE: contiguous cache with a row pitch below 16 MB (32-bit offsets within a column block).
template <int DT, int SWEEP, bool SIMPLE>
__global__ void __launch_bounds__(64 * kWaves, 4) k_tokred_sweep(TokRedArgs a) {
  constexpr int ESZ = DT == SKIPKV_BF16 ? 2 : 4;
  constexpr float kFix = SWEEP == 1 ? kFix1 : kFix2;
  __shared__ __align__(256) char cols[2][kColB];  // rows of 256 bytes, swizzled (swz16)
  __shared__ float col_cw[2][2][kCols];  // of each staged column: scale factor; weight in a row's sum: 1 (sweep 1), 1 / l (sweep 2)
  __shared__ float cpart[2][kWaves][kCols];  // [block parity]: column sums of a block over each wave's rows

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c16 = lane & 15, g = lane >> 4;
  // ---- which (head, sequence, row block) is this?
  const uint32_t item = xcd_contiguous_item(blockIdx.x, gridDim.x);
  if (item >= (uint32_t)a.n_layers * a.n_kv_heads * (uint32_t)a.nrb_max) return;
  const int lh = item / a.nrb_max;
  int j = item % a.nrb_max, b = 0, n_tok = 0, tok0 = 0;
  for (; b < a.batch; ++b) {
    tok0 = a.seq_off[b];
    n_tok = a.seq_off[b + 1] - tok0;
    const int cnt = (n_tok + kRows - 1) / kRows;
    if (j < cnt) break;
    j -= cnt;
  }
  if (b >= a.batch) return;
  const int r0 = j * kRows;
  if (a.len) n_tok = min(n_tok, a.len[lh * a.batch + b]);  // per-head ranges: the head's own length within the sequence's room
  if (r0 >= n_tok) return;
  const int l = lh / a.n_kv_heads, h = lh % a.n_kv_heads;
  // paged cache: rows are looked up in the row map (slot rows from the head's base), else they follow tok0
  const int32_t *rmap = !SIMPLE && a.row_map ? a.row_map + tok0 : nullptr;
  const char *kbase = static_cast<const char *>(a.k) + ((int64_t)l * a.stride_layer + (int64_t)h * a.stride_head + (rmap ? 0 : (int64_t)tok0 * a.stride_tok)) * ESZ;
  const int64_t pitch = a.stride_tok * ESZ;
  auto slot_of = [&](int row) -> int64_t { return rmap ? (int64_t)rmap[row] : (int64_t)row; };
  const int64_t col0 = (int64_t)lh * a.total_tokens + tok0;  // index of the sequence's first token in the per-token arrays

  // ---- A operands: this wave's rows, lane (row c16 of a tile, head-dim slice g)
  const int rw0 = __builtin_amdgcn_readfirstlane(r0 + 16 * kTW * wave);
  bf16x8 af[kTW][4];
  float row_c[kTW][4];  // scale factors of the lane's output rows (rows 4g+j of every tile)
  float row_w[kTW][4];  // their weights in a column's sum (0 for rows past the end)
#pragma unroll
  for (int t = 0; t < kTW; ++t) {
    const int row = min(rw0 + 16 * t + c16, n_tok - 1);
    const int64_t srow = slot_of(row);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) af[t][kk] = __builtin_bit_cast(bf16x8, load_piece_bf16<DT>(kbase + srow * pitch, 4 * g + kk));
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int r = rw0 + 16 * t + 4 * g + jj;
      row_c[t][jj] = a.scale[col0 + min(r, n_tok - 1)];
      row_w[t][jj] = r < n_tok ? (SWEEP == 1 ? 1.f : a.inv_l[col0 + r]) : 0.f;
    }
  }
  float rsum[kTW][4];
#pragma unroll
  for (int t = 0; t < kTW; ++t)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) rsum[t][jj] = 0.f;
  const float inv_n = SWEEP == 1 ? 1.f : 1.f / (float)n_tok;

  // A column block is 64 rows x 16 pieces of 16 bytes: kPieces loads of four rows per wave.  bf16 rows go straight to LDS
  // (no register holds them over a block's products), fp32 rows are converted on the way.
  constexpr int kPieces = kCols * 16 / (64 * kWaves);
  constexpr bool DIRECT = DT == SKIPKV_BF16;
  [[maybe_unused]] uint4 pre[kPieces];
  float pre_c = 0.f, pre_w = 0.f;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  // A whole block of a simple cache: a scalar base and one offset per lane (rows 32 further on lie 32 pitches behind it and
  // are swizzled alike).
  const int ld_row = 4 * wave_u + (lane >> 4), ld_piece = (lane & 15) ^ swz16(ld_row & 15);
  [[maybe_unused]] const uint32_t ld_off = (uint32_t)ld_row * (uint32_t)pitch + (uint32_t)ld_piece * 16;
  static_assert(kCols == 64 && 4 * kWaves % 16 == 0, "the loads of a lane have rows that are swizzled alike");
  // Other caches: a lane's rows of the block that is fetched next.  They are looked up a block ahead: looked up with the fetch, each
  // of them waits for the direct loads before it, too (pages, bf16, us, both sweeps looked up with the fetch / ahead: 4096 heads of 300
  // tokens 523 / 494, 64 of 4096 457 / 425, 7168 of 1000 5221 / 4679; fp32, 64 of 4096 577 / 520).
  [[maybe_unused]] int ahead[kPieces];
  auto look_up = [&](int jb) {
    if constexpr (!SIMPLE) {
#pragma unroll
      for (int it = 0; it < kPieces; ++it) {
        const int row = min(jb + 4 * kWaves * it + ld_row, n_tok - 1);
        ahead[it] = rmap ? rmap[row] : row;
      }
    }
  };
  auto fetch = [&](int jb, int buf) {
    const int left = n_tok - jb;
    if (SIMPLE && DIRECT && left >= kCols) {
#pragma unroll
      for (int it = 0; it < kPieces; ++it)
        load_to_lds_16_sbase(scalar64(kbase + (int64_t)(jb + 4 * kWaves * it) * pitch), ld_off, cols[buf] + (it * kWaves + wave_u) * 1024);
    } else {
#pragma unroll
      for (int it = 0; it < kPieces; ++it) {
        const char *src = kbase + (int64_t)(SIMPLE ? jb + min(4 * kWaves * it + ld_row, left - 1) : ahead[it]) * pitch;
        if constexpr (DIRECT) load_to_lds_16(src + ld_piece * 16, cols[buf] + (it * kWaves + wave_u) * 1024);
        else pre[it] = load_piece_bf16<DT>(src, ld_piece);
      }
    }
    if (wave_u == 0) {
      const int64_t at = col0 + jb;
      const int col = min(lane, left - 1);
      pre_c = a.scale[at + col];
      pre_w = lane < left ? (SWEEP == 1 ? 1.f : a.inv_l[at + col]) : 0.f;  // weight 0 drops columns past the end
    }
  };
  auto commit = [&](int buf) {
    if constexpr (!DIRECT) {
#pragma unroll
      for (int it = 0; it < kPieces; ++it) *reinterpret_cast<uint4 *>(cols[buf] + (it * kWaves + wave) * 1024 + lane * 16) = pre[it];
    }
    if (wave_u == 0) {
      col_cw[0][buf][lane] = pre_c;
      col_cw[1][buf][lane] = pre_w;
    }
  };

  // The column sums of block jb are added to the totals one block later, right after the next fetch has
  // been issued: the atomics then travel during that block's products.  The waves take turns.
  auto emit = [&](int jb, int buf) {
    if (wave == ((jb / kCols) & (kWaves - 1)) && jb + lane < n_tok) {
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) tot += cpart[buf][w][lane];
      add_fixed(a.acc + col0 + jb + lane, tot * inv_n, kFix);
    }
  };
  int buf = 0;
  look_up(r0);
  fetch(r0, buf);
  look_up(r0 + kCols);
#pragma unroll 1
  for (int jb = r0; jb < n_tok; jb += kCols, buf ^= 1) {
    commit(buf);
    // One barrier per block: a buffer is written again two blocks later, when every wave has passed the barrier
    // of the block in between and with it the end of its own reads.
    wait_vm<0>();  // (the compiler does not know of the direct loads)
    __syncthreads();
    if (jb + kCols < n_tok) {
      fetch(jb + kCols, buf ^ 1);  // lands while this block is multiplied
      look_up(jb + 2 * kCols);
    }
    if (jb > r0 + kCols) emit(jb - kCols, buf ^ 1);  // the first block has no mirror image
    // 64 x 64 squares on the diagonal are computed in full, blocks right of them stand for their transposes
    // too, blocks left of them are the transposes
    const bool square = (jb & -kCols) == (rw0 & -kCols);
    if (rw0 < n_tok && (jb > rw0 || square)) {
      float csum[kCols / 16];  // the lane's columns over the wave's rows
      // row 16 ct + c16, piece 4g + kk: the slice index kk is an XOR on bits 4..5
      const uint32_t tile = lds_addr(cols[buf]) + (uint32_t)(c16 * 256 + (((4 * g) ^ swz16(c16)) << 4));
      const float *wts = &col_cw[0][buf][c16];
      // Tiles of 16 rows x 16 columns in the order (column tile, row tile).  The products of a tile are issued among the
      // vector instructions of the tile before it, so that the matrix cores work while those are issued; the order is pinned.
      constexpr int CT = kCols / 16, NTILE = CT * kTW;
      bf16x8 bfr[4];
      f32x4 acc[2];
      float cc[2], cw[2];
      auto fragments = [&](int ct) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) bfr[kk] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>((uintptr_t)((tile ^ (kk << 4)) + ct * 4096));
        cc[ct & 1] = wts[16 * ct];
        cw[ct & 1] = wts[2 * kCols + 16 * ct];
      };
      auto half_product = [&](int i, int half) {  // of tile i: two of the four slices of the head dimension
        f32x4 &x = acc[i & 1];
        if (half == 0) x = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 2 * half; kk < 2 * half + 2; ++kk) x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i % kTW][kk], bfr[kk], x, 0, 0, 0);
      };
      fragments(0);
      half_product(0, 0);
      half_product(0, 1);
      float cs[2] = {0.f, 0.f};
#pragma unroll
      for (int i = 0; i < NTILE; ++i) {
        const int ct = i / kTW, t = i % kTW;
        float e[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) e[jj] = row_c[t][jj] * cc[ct & 1];
        __builtin_amdgcn_sched_barrier(0);
        if (i + 1 < NTILE) half_product(i + 1, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) e[jj] = __builtin_amdgcn_exp2f(acc[i & 1][jj] * e[jj]);
        __builtin_amdgcn_sched_barrier(0);
        if (i + 1 < NTILE) half_product(i + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          rsum[t][jj] = fmaf(e[jj], cw[ct & 1], rsum[t][jj]);
          cs[jj & 1] = fmaf(e[jj], row_w[t][jj], cs[jj & 1]);
        }
        if ((i + 2) % kTW == 0 && i + 2 < NTILE) fragments((i + 2) / kTW);  // the products just issued were the last ones with the old ones
        if (t == kTW - 1) {
          csum[ct] = cs[0] + cs[1];
          cs[0] = cs[1] = 0.f;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      const float sum = sum_lane_groups(csum[0], csum[1], csum[2], csum[3]);
      cpart[buf][wave][lane] = square ? 0.f : sum;
    } else {
      cpart[buf][wave][lane] = 0.f;
    }
  }
  __syncthreads();
  {
    const int last = r0 + (n_tok - 1 - r0) / kCols * kCols;
    if (last > r0) emit(last, ((last - r0) / kCols) & 1);
  }

  // ---- sums across the 16 column lanes, then the rows' share of their totals
#pragma unroll
  for (int t = 0; t < kTW; ++t) {
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const float s = row16_sum(rsum[t][jj]);
      const int row = rw0 + 16 * t + 4 * g + jj;
      if (c16 == 0 && row < n_tok) add_fixed(a.acc + col0 + row, s * inv_n, kFix);
    }
  }
}

// After sweep 1: inv_l = 1 / l, accumulator cleared for sweep 2.  After sweep 2: R.  Entries that no row
// contributed to (beyond a head's own length) stay as they are.
template <int SWEEP>
__global__ void __launch_bounds__(256) k_tokred_finish(TokRedArgs a) {
  const int64_t n = (int64_t)a.n_layers * a.n_kv_heads * a.total_tokens;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const unsigned long long v = a.acc[i];
    if (v == 0ull) continue;
    if (SWEEP == 1) {
      a.inv_l[i] = 1.f / ((float)v * (1.f / kFix1));
      a.acc[i] = 0ull;
    } else {
      a.out[i] = (float)v * (1.f / kFix2);
    }
  }
}

}  // namespace

hipError_t launch_token_redundancy(const TokRedArgs &a, hipStream_t st) {
  const int64_t n_lh = (int64_t)a.n_layers * a.n_kv_heads;
  if (n_lh == 0 || a.total_tokens == 0 || a.batch == 0) return hipSuccess;
  const int64_t rows = n_lh * a.total_tokens;
  const unsigned g0 = (unsigned)std::min<int64_t>((rows + 15) / 16, 1 << 16);
  const int64_t items = n_lh * a.nrb_max;
  const unsigned g1 = (unsigned)((items + 7) / 8 * 8);
  const unsigned g2 = (unsigned)std::min<int64_t>((rows + 255) / 256, 1 << 16);
  auto sweeps = [&](auto dt, auto simple) {
    constexpr int DT = decltype(dt)::value;
    constexpr bool SIMPLE = decltype(simple)::value;
    hipLaunchKernelGGL(k_key_scale<DT>, dim3(g0), dim3(256), 0, st, a);
    hipLaunchKernelGGL((k_tokred_sweep<DT, 1, SIMPLE>), dim3(g1), dim3(64 * kWaves), 0, st, a);
    hipLaunchKernelGGL(k_tokred_finish<1>, dim3(g2), dim3(256), 0, st, a);
    hipLaunchKernelGGL((k_tokred_sweep<DT, 2, SIMPLE>), dim3(g1), dim3(64 * kWaves), 0, st, a);
    hipLaunchKernelGGL(k_tokred_finish<2>, dim3(g2), dim3(256), 0, st, a);
  };
  auto of_type = [&](auto dt) {
    if (!a.row_map && a.stride_tok * (decltype(dt)::value == SKIPKV_BF16 ? 2 : 4) < (1 << 24)) sweeps(dt, std::true_type{});
    else sweeps(dt, std::false_type{});
  };
  if (a.dtype == SKIPKV_BF16) of_type(std::integral_constant<int, SKIPKV_BF16>{});
  else of_type(std::integral_constant<int, SKIPKV_F32>{});
  return hipGetLastError();
}

}  // namespace skipkv
