// Two-pass key scan of fp32 caches (Sec. 4.1 "Token Importance Score", Eq. 4, and the sentence embedding of
// Eq. 2 taken over the head's keys); scan_rows.hip has the bf16 form, scan_fused.hip the single-pass one.
//
// One workgroup (4 waves) handles one chunk of one head: a run of whole sentences of up to
// kChunkCap tokens (longer only when a single sentence is).  Keys stream HBM -> LDS in tiles of TT tokens with 16-byte-per-lane
// coalesced loads; each wave multiplies its 16 tokens against all query rows of the GQA
// group on the matrix cores (16x16 MFMA tiles, fp32 accumulate), so a lane ends up holding, for
// ONE token, the logits of every (window query a, group head i) pair assigned to its lane group.
//
// The softmax of Eq. 4 runs over all N keys of the head, which span many chunks, so it takes
// two passes over K:
//   pass A (PASSB = false): per chunk, the running (max, sum of exp) of every query row, and the
//       mean-pooled, L2-normalised key of every sentence of the chunk (split into bf16 hi + lo);
//   k_row_norm (scan_rows.hip): merges the per-chunk statistics into log2 of each row's normaliser;
//   pass B (PASSB = true): recomputes the logits, forms I[t] = (1/alpha) sum_a max_i softmax and
//       its mean over the unprotected part of every sentence.
// exp() is evaluated in base 2: logits are scaled by log2(e)/sqrt(d).
#include "scan_common.h"

#include <algorithm>

namespace skipkv {

namespace {

template <int NP, int AL, bool PASSB>
__global__ void __launch_bounds__(256) k_scan(ScanArgs a) {
  constexpr int DT = SKIPKV_F32, NSUB = 1;
  constexpr int SL = NP * AL;        // used (a, i) slots per lane group
  constexpr int NT = (SL + 3) / 4;   // row tiles
  constexpr int SLP = 4 * NT;        // slots incl. padding
  constexpr int R = 16 * NT;         // padded query rows
  constexpr int WT = 16 * NSUB;      // tokens per wave per tile
  constexpr int TT = 4 * WT;         // tokens per tile
  constexpr int LSTR = Tr<DT>::LSTR, ROWB = Tr<DT>::ROWB, ESZ = Tr<DT>::ESZ;
  constexpr int PPR = ROWB / 16;     // 16-byte pieces per row
  constexpr int LOADS = TT * PPR / 256;

  __shared__ __align__(16) char kt[TT * LSTR];
  __shared__ __align__(16) char qt[R * LSTR];
  __shared__ int soff[kChunkMaxSent + 1];
  // pass A: sentence key sums [kChunkMaxSent][128] then per-wave row statistics [4][R][2]
  // pass B: token importance of the tile [TT], sentence sums of I and of R [2][kChunkMaxSent]
  constexpr int SBUF = PASSB ? (TT + 2 * kChunkMaxSent) : (kChunkMaxSent * kD);
  __shared__ float sbuf[SBUF];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c16 = lane & 15, g = lane >> 4;
  // Fallback path: only sequences that the single-pass scan cannot take (a sentence longer than
  // a chunk, or too many chunks), unless the caller forces this path for everything.
  if (!a.force_two_pass && a.ws.hdr->n_unfused == 0) return;
  const int n_lh = a.n_layers * a.n_kv_heads;
  const int n_chunks = hdr_chunks(a.ws.hdr->ranges);
  const uint32_t n_items = (uint32_t)n_lh * (uint32_t)n_chunks;
  const int n = a.n_q_heads / a.n_kv_heads;
  for (uint32_t item = blockIdx.x; item < n_items; item += gridDim.x) {
  int lh, c;
  two_pass_item(item, n_chunks, lh, c);
  const Chunk ch = a.ws.chunks[c];
  const int b = ch.b, ns = ch.ns;
  if (!a.force_two_pass && a.ws.seq_fused[b] && !a.ws.head_redo[(int64_t)lh * a.batch + b]) continue;  // done by the single-pass scan
  const int l = lh / a.n_kv_heads, h = lh % a.n_kv_heads;
  const int tok0 = ch.tok0;
  const int n_tok = ch.n_tok;
  const int sent_col0 = ch.soff_idx - b;  // column of the chunk's first sentence in [.., S_total] arrays
  __syncthreads();  // the previous item's readers of LDS are done

  if (tid <= ns) soff[tid] = a.sent_off[ch.soff_idx + tid];
  for (int i = tid; i < SBUF; i += 256) sbuf[i] = 0.f;

  // ---- queries of the group -> LDS, one padded row per (lane group, slot)
  {
    const char *qbase = static_cast<const char *>(a.q);
    // layer, KV head and sequence that address the query rows (the real ones under per-head ranges)
    int ql = l, qh = h, qb = b, q_batch = a.batch, q_heads = a.n_q_heads;
    if (a.virt_hk > 0) {
      const int lh_r = b / a.virt_b;
      qb = b % a.virt_b;
      ql = lh_r / a.virt_hk;
      qh = lh_r % a.virt_hk;
      q_batch = a.virt_b;
      q_heads = a.virt_hk * n;
    }
    for (int r0 = 0; r0 < R; r0 += 256 / PPR) {
      const int r = r0 + tid / PPR, piece = tid % PPR;
      const int slot = 4 * (r >> 4) + (r & 3), gq = (r >> 2) & 3;
      const int al = slot / NP, i = slot % NP, aq = gq + 4 * al;
      uint4 val = make_uint4(0, 0, 0, 0);
      if (slot < SL && i < n && aq < a.alpha) {
        const int64_t row = (((int64_t)ql * q_batch + qb) * q_heads + (qh * n + i)) * a.alpha + aq;
        val = *reinterpret_cast<const uint4 *>(qbase + row * ROWB + piece * 16);
      }
      *reinterpret_cast<uint4 *>(qt + r * LSTR + piece * 16) = val;
    }
  }
  __syncthreads();

  const int t_begin = soff[0], t_end = soff[ns];
  // contiguous cache: row t of the sequence is row tok0 + t of the head; paged cache: the row map says where it is
  const int32_t *rmap = a.row_map ? a.row_map + tok0 : nullptr;
  const char *kbase = static_cast<const char *>(a.k) +
                      ((int64_t)l * a.stride_layer + (int64_t)h * a.stride_head + (rmap ? 0 : (int64_t)tok0 * a.stride_tok)) * ESZ;
  const int64_t tok_pitch = (a.row_map ? a.map_stride : a.stride_tok) * ESZ;  // paged: bytes per unit of the row map
  const int last_free = n_tok - a.alpha;  // keys t <= last_free are visible to every window query

  // per-lane state
  float ref[SLP], lsum[SLP];  // pass A: reference (uniform over the 16 lanes of a row) and sum of exp2(x - ref)
  float cn[SLP];              // pass B: log2 normaliser of the slot's query row (+inf: unused slot)
  if constexpr (!PASSB) {
#pragma unroll
    for (int q = 0; q < SLP; ++q) {
      ref[q] = kRefInit;
      lsum[q] = 0.f;
    }
  } else {
    const float *rn = a.ws.row_norm + ((int64_t)lh * a.batch + b) * R;
#pragma unroll
    for (int q = 0; q < SLP; ++q) {
      const int al = q / NP, i = q % NP;
      const bool used = q < SL && i < n && (g + 4 * al) < a.alpha;
      cn[q] = used ? rn[16 * (q >> 2) + 4 * g + (q & 3)] : INFINITY;
    }
  }
  const int p_start = n_tok - min(a.protect, n_tok);  // first protected token

  for (int tile_t = t_begin; tile_t < t_end; tile_t += TT) {
    // ---- stream the tile into LDS
    {
      uint4 regs[LOADS];
      int rows[LOADS];
#pragma unroll
      for (int it = 0; it < LOADS; ++it) {
        const int t = tile_t + (it * 256 + tid) / PPR;
        rows[it] = t;
        if (rmap && t < t_end) rows[it] = rmap[t];
      }
#pragma unroll
      for (int it = 0; it < LOADS; ++it) {
        const int idx = it * 256 + tid, row = idx / PPR, piece = idx % PPR, t = tile_t + row;
        regs[it] = make_uint4(0, 0, 0, 0);
        if (t < t_end) regs[it] = *reinterpret_cast<const uint4 *>(kbase + (int64_t)rows[it] * tok_pitch + piece * 16);
      }
#pragma unroll
      for (int it = 0; it < LOADS; ++it) {
        const int idx = it * 256 + tid, row = idx / PPR, piece = idx % PPR;
        *reinterpret_cast<uint4 *>(kt + row * LSTR + piece * 16) = regs[it];
      }
    }
    __syncthreads();

    const int wt0 = tile_t + wave * WT;  // first token of this wave's share
    f32x4 acc[NSUB][NT];
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
#pragma unroll
      for (int T = 0; T < NT; ++T) acc[s][T] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (wt0 + 16 * s < t_end)
        tile_logits<DT, NT>(qt, kt + (wave * WT + 16 * s + c16) * LSTR, c16, g, acc[s]);
    }

    if constexpr (!PASSB) {
      // ---- running softmax statistics of every query row over this wave's tokens
      float tmax[SLP];
#pragma unroll
      for (int q = 0; q < SLP; ++q) tmax[q] = -INFINITY;
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        const int t = wt0 + 16 * s + c16;
        const bool edge = (wt0 + 16 * s + 15 >= t_end) || (wt0 + 16 * s + 15 > last_free);
#pragma unroll
        for (int q = 0; q < SLP; ++q) {
          float x = acc[s][q >> 2][q & 3] * kScale2;
          if (edge) {
            const int aq = g + 4 * (q / NP);
            if (!(t < t_end && t <= last_free + aq)) x = -INFINITY;
          }
          acc[s][q >> 2][q & 3] = x;
          tmax[q] = fmaxf(tmax[q], x);
        }
      }
      bool need = false;
#pragma unroll
      for (int q = 0; q < SLP; ++q) need |= tmax[q] > ref[q] + kRescaleSlack;
      if (__any(need)) {
#pragma unroll
        for (int q = 0; q < SLP; ++q) {
          const float nr = fmaxf(ref[q], row16_max(tmax[q]));
          lsum[q] *= __builtin_amdgcn_exp2f(ref[q] - nr);
          ref[q] = nr;
        }
      }
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int q = 0; q < SLP; ++q) lsum[q] += __builtin_amdgcn_exp2f(acc[s][q >> 2][q & 3] - ref[q]);

      // ---- sentence key sums: wave w takes sentences w, w + 4, ... of the chunk, lane = 2 head-dim
      // columns.  A sentence's rows are added in token order by one wave only (also across the tiles
      // of the chunk), so the sums are the same bits on every run.
      {
        const int t_hi = min(tile_t + TT, t_end);
        for (int si = __popcll(__ballot(lane < ns && soff[lane + 1] <= tile_t)); si < ns && soff[si] < t_hi; ++si) {
          if ((si & 3) != wave) continue;
          const int lo = max(soff[si], tile_t), hi = min(soff[si + 1], t_hi);
          float s0 = 0.f, s1 = 0.f;
          for (int t = lo; t < hi; ++t) {
            const char *rowp = kt + (t - tile_t) * LSTR;
            const float2 w = *reinterpret_cast<const float2 *>(rowp + lane * 8);
            s0 += w.x;
            s1 += w.y;
          }
          sbuf[si * kD + 2 * lane] += s0;
          sbuf[si * kD + 2 * lane + 1] += s1;
        }
      }
    } else {
      // ---- token importance: max over the group's heads in registers, exp2, sum over window queries
      float *imp = sbuf;
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        const int t = wt0 + 16 * s + c16;
        const bool edge = (wt0 + 16 * s + 15 > last_free);
        float sum = 0.f;
#pragma unroll
        for (int al = 0; al < AL; ++al) {
          float gm = -INFINITY;
#pragma unroll
          for (int i = 0; i < NP; ++i) {
            const int q = al * NP + i;
            gm = fmaxf(gm, fmaf(acc[s][q >> 2][q & 3], kScale2, -cn[q]));
          }
          if (edge && t > last_free + g + 4 * al) gm = -INFINITY;
          sum += __builtin_amdgcn_exp2f(gm);
        }
        sum += __shfl_xor(sum, 16);
        sum += __shfl_xor(sum, 32);
        if (g == 0) imp[wave * WT + 16 * s + c16] = (t < t_end) ? sum / (float)a.alpha : 0.f;
      }
      __syncthreads();
      // sentence sums over the unprotected part, and the optional per-token outputs / inputs
      const int64_t tok_col = (int64_t)lh * a.total_tokens + tok0;
      if (tid < ns) {
        const int lo = max(soff[tid], tile_t), hi = min(min(soff[tid + 1], p_start), tile_t + TT);
        float si = 0.f, sr = 0.f;
        for (int t = lo; t < hi; ++t) {
          si += imp[t - tile_t];
          if (a.tok_red) sr += a.tok_red[tok_col + t];
        }
        sbuf[TT + tid] += si;
        sbuf[TT + kChunkMaxSent + tid] += sr;
      }
      if (a.tok_imp) {
        for (int i = tid; i < TT && tile_t + i < t_end; i += 256) a.tok_imp[tok_col + tile_t + i] = imp[i];
      }
    }
    __syncthreads();  // the next tile overwrites kt / imp
  }

  if constexpr (!PASSB) {
    // ---- unit sentence embeddings, split into bf16 hi + lo, one wave per sentence
    for (int si = wave; si < ns && !a.no_pool; si += 4) {
      const float inv_len = 1.f / (float)(soff[si + 1] - soff[si]);
      const float m0 = sbuf[si * kD + 2 * lane] * inv_len, m1 = sbuf[si * kD + 2 * lane + 1] * inv_len;
      const float nrm = sqrtf(wave_sum(m0 * m0 + m1 * m1));
      const float inv = 1.f / (nrm + 1e-12f);
      const float u0 = m0 * inv, u1 = m1 * inv;
      const uint32_t h0 = f32_to_bf16_bits(u0), h1 = f32_to_bf16_bits(u1);
      const uint32_t l0 = f32_to_bf16_bits(u0 - bf16_bits_to_f32(h0)), l1 = f32_to_bf16_bits(u1 - bf16_bits_to_f32(h1));
      const int64_t o = ((int64_t)lh * a.total_sentences + sent_col0 + si) * (kD / 2) + lane;
      reinterpret_cast<uint32_t *>(a.ws.vhat_hi)[o] = h0 | (h1 << 16);
      reinterpret_cast<uint32_t *>(a.ws.vhat_lo)[o] = l0 | (l1 << 16);
    }
    // ---- merge the row statistics of the 4 waves and publish the chunk's partial
    // (in the key tile's buffer, which nobody reads after the last tile: with 160 query rows this keeps
    // the workgroup under half of the CU's LDS)
    static_assert(8 * R * sizeof(float) <= sizeof(kt), "the statistics of the 4 waves fit the key tile");
    float *wstat = reinterpret_cast<float *>(kt);
#pragma unroll
    for (int q = 0; q < SLP; ++q) {
      const float tot = row16_sum(lsum[q]);
      if (c16 == 0) {
        const int r = 16 * (q >> 2) + 4 * g + (q & 3);
        wstat[(wave * R + r) * 2] = ref[q];
        wstat[(wave * R + r) * 2 + 1] = tot;
      }
    }
    __syncthreads();
    for (int r = tid; r < R; r += 256) {
      float m = kRefInit;
#pragma unroll
      for (int w = 0; w < 4; ++w) m = fmaxf(m, wstat[(w * R + r) * 2]);
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) s += wstat[(w * R + r) * 2 + 1] * __builtin_amdgcn_exp2f(wstat[(w * R + r) * 2] - m);
      a.ws.stat_part[((int64_t)lh * a.ws.nr_max + c) * R + r] = make_float2(m, s);
    }
  } else {
    if (tid < ns) {
      const int len = min(soff[tid + 1], p_start) - soff[tid];
      const int64_t o = (int64_t)lh * a.total_sentences + sent_col0 + tid;
      a.ws.sent_imp[o] = len > 0 ? sbuf[TT + tid] / (float)len : 0.f;
      a.ws.sent_red[o] = len > 0 ? sbuf[TT + kChunkMaxSent + tid] / (float)len : 0.f;
    }
  }
  }  // item loop
}

template <int NP, int AL, bool PASSB>
hipError_t launch_one(const ScanArgs &a, hipStream_t st) {
  const int64_t items = (int64_t)a.n_layers * a.n_kv_heads * a.ws.nr_max;
  if (items == 0) return hipSuccess;
  const int64_t grid = items < 4096 ? items : 4096;  // grid-stride over the items
  hipLaunchKernelGGL((k_scan<NP, AL, PASSB>), dim3((unsigned)grid), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <bool PASSB>
hipError_t dispatch(const ScanArgs &a, hipStream_t st) {
#define SKIPKV_CASE(NP_, AL_) \
  if (a.rl.np == NP_ && a.rl.al == AL_) return launch_one<NP_, AL_, PASSB>(a, st);
  SKIPKV_CASE(4, 2)
  SKIPKV_CASE(4, 4)
  SKIPKV_CASE(4, 8)
  SKIPKV_CASE(8, 2)
  SKIPKV_CASE(8, 4)
  SKIPKV_CASE(5, 8)  // (256 fp32 query rows, the shape (8, 8), do not fit in LDS)
  SKIPKV_CASE(7, 2)
#undef SKIPKV_CASE
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_scan_stats(const ScanArgs &a, hipStream_t st) { return a.dtype == SKIPKV_BF16 ? launch_rows_stats(a, st) : dispatch<false>(a, st); }
hipError_t launch_scan_scores(const ScanArgs &a, hipStream_t st) { return a.dtype == SKIPKV_BF16 ? launch_rows_scores(a, st) : dispatch<true>(a, st); }

}  // namespace skipkv
