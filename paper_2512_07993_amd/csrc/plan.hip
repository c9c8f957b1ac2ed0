// Work decomposition for one compression step: cuts every sequence's sentence list into
// chunks (units of the key scan) and row blocks (units of the redundancy kernel), checks the
// sentence offsets, and decides per sequence which scan variant handles it.  Shared by all
// layers and heads of the batch, so it is tiny.
#include "common.h"

#include <algorithm>

namespace skipkv {

__global__ void k_plan_reset(PlanHeader *hdr) {
  if (threadIdx.x == 0) reset_header(hdr);
}

// End (exclusive sentence index) of the run of whole sentences that starts at sentence `start` and
// holds at most `cap` tokens and `max_sent` sentences: the largest e in (start, start + max_sent]
// with off[e] - off[start] <= cap, at least start + 1.
__device__ __forceinline__ int run_end(const int *off, int start, int n_sent, int cap, int max_sent) {
  int lo = start + 1, hi = min(n_sent, start + max_sent);
  const int limit = off[start] + cap;
  while (lo < hi) {  // invariant: the answer lies in [lo, hi]
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= limit) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Plans of sequences: WPS waves each, 4 / WPS sequences per block.  Chunks (two-pass scan) and spans (single-pass
// scan) are packed greedily: the longest run of whole sentences within the unit's token and sentence limits; a sentence
// longer than the token limit is a chunk of its own and as many spans as it needs.
//
// What bounds a plan: with few sequences the latency of the serial walks along the runs (an LDS read per step, 300 spans
// in 32 K tokens), so the two walks run side by side; with thousands of them (every head a sequence of its own) the
// atomic on the one word that hands out the ranges, 13 ns each, hence one for four sequences.  LDS and registers
// are the same for both forms: a wave takes what fits a quarter of the tables (kMaxSent<1> sentences; with cut sentences as
// many spans as a quarter holds, so that a sequence takes the same scan in every batch), longer
// sequences are done by the block afterwards.  Measured, against a block
// per sequence with both walks in one thread: 7168 sequences of 1.1 K tokens 95 -> 32 us, 4096 of 2.1 K 60 -> 23,
// 4 of 32 K 43 -> 28, 16 of 2-16 K 23 -> 17.  The walk over cut sentences has an LDS read per step too: with three, and a walk also for
// sequences with a sentence that no item holds, the plan of 8 K tokens of sentences of 129 took 32 us, now 24 (not cut: 14),
// of 4 K with some sentences of more than 512 17, now 10.  What only such sequences need stands behind the rest (k_plan of others 7.3 -> 6.7 us).
template <int WPS>
constexpr int kMaxSent = WPS == 4 ? SKIPKV_MAX_SENTENCES : SKIPKV_MAX_SENTENCES / 4 - 1;

struct PlanShared {
  int off[SKIPKV_MAX_SENTENCES + 1];
  // End of the chunk (span) that would start at each sentence; the walk along them replaces them, from the front,
  // by the first sentences of the chunks (spans) and a final n_sent.  Chunk k never starts before sentence k, so
  // what is replaced has been read.
  uint16_t chunk[SKIPKV_MAX_SENTENCES + 1];
  uint16_t span[SKIPKV_MAX_SENTENCES + 1];  // (with cut sentences: | (spans of the sentence - 1) << 13, and not replaced)
  // The spans of a sequence with sentences of several spans: first sentence, number of the piece of it << 13.  (A span
  // that is only there so that the pieces of a sentence come to lie in one item is empty: it begins where the next one does.)
  uint16_t pieces[kItemSpans * kFuseMaxItems + 4];
  struct Seq {
    int n_chunks, n_spans;
    unsigned long long counts, old;  // of the sequence, and drawn before it (packed as in the header)
  } seq[4];
  int later[4];  // a wave's sequence is left to the whole block
};

// b < 0: the group has no sequence (in this pass), but takes part in the barriers.
//
// Two launches are saved where calls are so small that launches are what they cost: a batch of one sequence needs
// no atomics, hence no header reset before (a.alone); and few statistics records are marked here instead of by
// k_plan_preset (a.preset: see launch_plan).
template <int WPS>
__device__ __forceinline__ void plan_sequences(const PlanArgs &a, PlanShared &sh, int b, int gt, int grp) {
  constexpr int G = 64 * WPS, PART = SKIPKV_MAX_SENTENCES / 4;
  static_assert(SKIPKV_MAX_SENTENCES < 1 << 13, "sentence indices are kept in 16 bits here, in 13 beside the number of a piece");
  int *s_off = sh.off + grp * PART;
  uint16_t *s_chunk = sh.chunk + grp * PART, *s_span = sh.span + grp * PART;
  constexpr int kPieces = kItemSpans * kFuseMaxItems / (4 / WPS);  // spans of a sequence that the group's part of the table holds
  uint16_t *s_pieces = sh.pieces + grp * (kPieces + 1);
  auto any = [](bool x) -> bool { return WPS == 4 ? __syncthreads_or(x) != 0 : __any(x) != 0; };
  auto sync = [] {
    if constexpr (WPS == 4) __syncthreads();
    else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // one wave: its LDS operations are in order
  };

  int tok0 = 0, n_tok = 0, sp = 0, n_sent = 0;
  bool cut = false;  // some sentence has several spans
  int most = 0;      // spans of a sequence like that, at most
  bool ok = b >= 0;
  if (ok) {
    tok0 = a.seq_off[b];
    n_tok = seq_tokens(a.seq_off, a.len, b);
    sp = a.sent_ptr[b];
    n_sent = seq_sentences(a.sent_ptr, a.cnt, b);
    const int32_t *off = a.sent_off + sp;
    const bool reject = n_sent > SKIPKV_MAX_SENTENCES || n_sent < 0;
    // explicit lengths and counts must fit the room that the CSR arrays describe
    bool bad = !reject && (n_tok < 0 || n_tok > a.seq_off[b + 1] - tok0 || n_sent > a.sent_ptr[b + 1] - sp - 1);
    bool longer = false;  // some sentence is longer than a span may be
    if (!reject && !bad) {
      // validation: o[0] = 0, o[S] = N, strictly ascending
      for (int s = gt; s <= n_sent; s += G) {
        const int o = off[s];
        s_off[s] = o;
        if (s < n_sent) {
          const int n = off[s + 1] - o;
          bad |= off[s + 1] <= o;
          longer |= n > kSpanCap;
        }
      }
      if (gt == 0) bad |= (off[0] != 0) | (off[n_sent] != n_tok) | (n_sent == 0 && n_tok != 0);
    }
    bad = any(bad);
    longer = any(longer);
    ok = !reject && !bad;
    bool later = false;
    if (__builtin_expect(longer && ok, false)) {
      bool fits_items = true;
      sync();
      for (int s = gt; s < n_sent; s += G) fits_items &= s_off[s + 1] - s_off[s] <= kItemSpans * kSpanCap;
      cut = !any(!fits_items);  // (else the sequence is the two-pass scan's: its spans are not looked for)
      // (no sequence gets more items than its tokens and sentences make of ordinary spans at most: that is what there is room for)
      most = min(kItemSpans * kFuseMaxItems, kItemSpans * ((2 * (n_tok / a.ws.span_cap + n_sent / kSpanMaxSent) + 1) / kItemSpans + 1));
      if (a.cut_item_tokens > 0) most = min(most, kItemSpans * (n_tok / a.cut_item_tokens));
      later = cut && most > kPieces;
      ok = !later;
    }
    if (WPS == 1 && gt == 0) sh.later[grp] = later;
    for (int lh = gt; lh < a.n_lh; lh += G) a.ws.head_redo[(int64_t)lh * a.batch + b] = 0;
    sync();
    if (ok) {
      // the greedy packing is a walk along s -> end(s); the ends are found for all sentences at
      // once, so that the (serial) walk is one LDS read per chunk
      // short spans only where they leave the sequence within the items that a head may have
      const int cap = 2 * ((n_tok + a.ws.span_cap - 1) / a.ws.span_cap + (n_sent + kSpanMaxSent - 1) / kSpanMaxSent) < kItemSpans * kFuseMaxItems ? a.ws.span_cap : kSpanCap;
      for (int s = gt; s < n_sent; s += G) {
        s_chunk[s] = (uint16_t)run_end(s_off, s, n_sent, kChunkCap, kChunkMaxSent);
        s_span[s] = (uint16_t)run_end(s_off, s, n_sent, cap, kSpanMaxSent);
      }
      if (__builtin_expect(cut, false))
        for (int s = gt; s < n_sent; s += G) s_span[s] |= (uint16_t)((s_off[s + 1] - s_off[s] - 1) / kSpanCap << 13);
    }
    sync();
    PlanShared::Seq &me = sh.seq[grp];
    constexpr int kOther = WPS == 4 ? 64 : 1;  // the thread of the second walk: another wave, or another lane in step
    if (ok && (gt == 0 || gt == kOther)) {
      uint16_t *at = gt == 0 ? s_span : s_chunk;
      int n = 0;
      if (__builtin_expect(gt == 0 && longer, false)) {
        bool fits = cut;
        for (int start = 0; start < n_sent && fits;) {
          const int x = at[start], more = x >> 13;  // spans of the sentence besides its first
          if (more > 0 && n % kItemSpans + more >= kItemSpans)  // on to the next item
            for (; n % kItemSpans != 0 && n < most; ++n) s_pieces[n] = (uint16_t)start;
          fits = n + more < most;
          for (int k = 0; k <= more && fits; ++k) s_pieces[n++] = (uint16_t)(start | k << 13);
          start = x & 0x1FFF;
        }
        if (fits) s_pieces[n] = (uint16_t)n_sent;
        else n = 0;  // the two-pass scan's
      } else {
        for (int start = 0; start < n_sent;) {
          const int e = at[start];
          at[n++] = (uint16_t)start;
          start = e;
        }
        at[n] = (uint16_t)n_sent;
        if (gt == 0 && n > kItemSpans * kFuseMaxItems) n = 0;
      }
      if (gt == 0) me.n_spans = n;
      else me.n_chunks = n;
    }
    sync();
    if (gt == 0) {
      unsigned long long counts = 0;
      if (ok) {
        const int n_items = (me.n_spans + kItemSpans - 1) / kItemSpans, nrb = (n_sent + kRowBlock - 1) / kRowBlock;
        const int rc = a.ws.run_chunks;  // whole runs: the sequence's chunks start at a multiple of their length
        counts = (unsigned long long)((me.n_chunks + rc - 1) / rc * rc) | ((unsigned long long)n_items << kHdrItemShift) | ((unsigned long long)nrb << kHdrRbShift);
      } else if (a.dev_status && !later) {
        atomicOr(a.dev_status, reject ? SKIPKV_DEV_TOO_MANY_SENT : SKIPKV_DEV_BAD_OFFSETS);
      }
      me.counts = counts;
    }
  } else if (gt == 0) {
    sh.seq[grp].counts = 0;
    if (WPS == 1) sh.later[grp] = 0;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    // one atomic draws the ranges of chunks, items and row blocks of the block's sequences
    unsigned long long sum = 0;
#pragma unroll
    for (int i = 0; i < 4 / WPS; ++i) sum += sh.seq[i].counts;
    unsigned long long old = 0;
    if (a.alone) {
      a.ws.hdr->ranges = sum;
      a.ws.hdr->n_unfused = sum != 0 && sh.seq[0].n_spans == 0 && sh.seq[0].n_chunks > 0;
      a.ws.hdr->abort = 0;
    } else if (sum) {
      old = atomicAdd(&a.ws.hdr->ranges, sum);
    }
#pragma unroll
    for (int i = 0; i < 4 / WPS; ++i) {
      sh.seq[i].old = old;
      old += sh.seq[i].counts;
    }
  }
  __syncthreads();
  if (b < 0) return;
  if (!ok) {
    if (gt == 0) {
      a.ws.chunk_base[b] = 0;
      a.ws.chunk_cnt[b] = 0;
      a.ws.rb_base[b] = 0;
      a.ws.rb_cnt[b] = 0;
      a.ws.seq_fused[b] = 1;  // nothing to scan either way
    }
    return;
  }
  const PlanShared::Seq &me = sh.seq[grp];
  const int n_chunks = me.n_chunks, n_spans = me.n_spans, n_items = (n_spans + kItemSpans - 1) / kItemSpans;
  const int base = hdr_chunks(me.old), ibase = hdr_items(me.old), rb0 = hdr_rowblocks(me.old);
  const bool fused = n_spans > 0 || n_chunks == 0;
  const int nrb = hdr_rowblocks(me.counts);
  if (gt == 0) {
    a.ws.chunk_base[b] = base;
    a.ws.chunk_cnt[b] = n_chunks;
    a.ws.seq_fused[b] = fused;
    if (!fused && n_chunks > 0 && !a.alone) atomicAdd(&a.ws.hdr->n_unfused, 1);
    a.ws.rb_base[b] = rb0;
    a.ws.rb_cnt[b] = nrb;
  }
  for (int i = gt; i < nrb; i += G) a.ws.rowblocks[rb0 + i] = RowBlock{b, i * kRowBlock};
  for (int j = gt; j < n_chunks; j += G) {  // one record per chunk
    const int s0 = s_chunk[j], e = s_chunk[j + 1];
    a.ws.chunks[base + j] = Chunk{b, s0, e - s0, s_off[s0], s_off[e] - s_off[s0], sp + s0, tok0, n_tok};
  }
  for (int j = gt; j < n_items; j += G) {  // one record per item: up to kItemSpans consecutive spans
    const int nsp = min(kItemSpans, n_spans - kItemSpans * j);
    int32_t *r = a.ws.item_rec + (int64_t)(ibase + j) * kItemRecInts;
    const uint16_t *at = (cut ? s_pieces : s_span) + kItemSpans * j;  // sentence, piece << 13 (s_span has no pieces)
    const int s0 = at[0] & 0x1FFF;
    r[kIrB] = b;
    r[kIrRec] = ibase + j;
    r[kIrTok0] = tok0;
    r[kIrNTok] = n_tok;
    r[kIrNItems] = n_items;
    r[kIrFirst] = ibase;
    r[kIrSoffIdx] = sp + s0;
    uint32_t ns = 0, pieces = 0;
    for (int w = 0; w <= kItemSpans; ++w) {
      const int x = at[min(w, nsp)], sw = x & 0x1FFF, piece = x >> 13;
      r[kIrT0 + w] = s_off[sw] + kSpanCap * piece;
      if (w < nsp) {
        // sentences that begin here; the next span may begin within the one that this one begins with
        const int y = at[w + 1], next = (y & 0x1FFF) + (y >> 13 ? 1 : 0);
        if (piece == 0) ns |= (uint32_t)(next - sw) << (8 * w);
        pieces |= piece;
      }
    }
    r[kIrNsp] = nsp | (pieces ? kIrCut : 0);
    r[kIrNs] = (int32_t)ns;
  }
  if (a.preset) {
    const int n16 = n_items * a.ws.rows / 2;
    for (int i = gt; i < a.n_lh * n16; i += G) {
      uint4 *dst = reinterpret_cast<uint4 *>(a.ws.item_stat + ((int64_t)(i / n16) * a.ws.ni_max + ibase) * a.ws.rows);
      dst[i % n16] = make_uint4(kRowNormUnset, 0u, kRowNormUnset, 0u);
    }
  }
}

template <int WPS>
__global__ void __launch_bounds__(256) k_plan(PlanArgs a) {
  __shared__ PlanShared sh;
  if constexpr (WPS == 4) {
    plan_sequences<4>(a, sh, blockIdx.x, threadIdx.x, 0);
  } else {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int b = blockIdx.x * 4 + wave;
    const bool mine = b < a.batch && seq_sentences(a.sent_ptr, a.cnt, b) <= kMaxSent<1>;
    plan_sequences<1>(a, sh, mine ? b : -1, lane, wave);
    for (int w = 0; w < 4; ++w) {  // those that were left, one after the other, by the whole block
      const int bl = blockIdx.x * 4 + w;
      if (bl >= a.batch) break;
      if (seq_sentences(a.sent_ptr, a.cnt, bl) <= kMaxSent<1> && !sh.later[w]) continue;
      __syncthreads();  // everybody is done with the tables
      plan_sequences<4>(a, sh, bl, threadIdx.x, 0);
    }
  }
}

// Marks the statistics records of all items of this step as "not written yet": the single-pass
// scan polls them.  The number of items is only known on the device, so the grid covers the
// capacity and the surplus exits.  grid = (x, LH); one thread writes two rows of a record at a time.
__global__ void __launch_bounds__(256) k_plan_preset(Workspace ws) {
  const int64_t n16 = (int64_t)hdr_items(ws.hdr->ranges) * ws.rows / 2;  // 16-byte pieces per head
  uint4 *dst = reinterpret_cast<uint4 *>(ws.item_stat + (int64_t)blockIdx.y * ws.ni_max * ws.rows);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (int64_t)gridDim.x * 256)
    dst[i] = make_uint4(kRowNormUnset, 0u, kRowNormUnset, 0u);
}

hipError_t launch_plan(const PlanArgs &args, hipStream_t st) {
  PlanArgs a = args;
  const int64_t cap16 = (int64_t)a.ws.ni_max * a.ws.rows / 2;
  a.alone = a.batch == 1;
  // up to about 32 records' pieces per thread of a plan block: cheaper than a launch of their own (us, whole
  // score call of 8 heads and 1152 tokens: bf16 38.5 -> 34.5, fp32 44.7 -> 40.1 without the two launches)
  a.preset = a.n_lh * cap16 <= 8192 * (int64_t)a.batch && a.batch < 1024;
  if (!a.alone && !a.hdr_reset) hipLaunchKernelGGL(k_plan_reset, dim3(1), dim3(64), 0, st, a.ws.hdr);
  if (a.batch > 0) {
    // A wave per sequence from where a block each would fill the chip (four blocks per CU), unless the sentences that
    // there is room for are so many on average that blocks would do their sequences one after the other.  us, a wave / a
    // block: 1024 sequences of 300 / 700 / 900 / 1100 / 3000 sentences 22 / 33 / 39 / 64 / 132, 29 / 32 / 34 / 36 / 56;  2048 of
    // 500: 31, 46;  4096 of 300 / 1020 / 1100: 34 / 55 / 103, 70 / 91 / 100.
    const int64_t most = a.batch < 2048 ? 640 : kMaxSent<1>;
    if (a.batch < 1024 || a.total_sentences > a.batch * most)
      hipLaunchKernelGGL(k_plan<4>, dim3(a.batch), dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL(k_plan<1>, dim3((a.batch + 3) / 4), dim3(256), 0, st, a);
    const int gx = (int)std::min<int64_t>((cap16 + 255) / 256, std::max(32, 8192 / std::max(1, a.n_lh)));  // ~8192 workgroups in all
    if (!a.preset && a.n_lh > 0 && cap16 > 0) hipLaunchKernelGGL(k_plan_preset, dim3(gx, a.n_lh), dim3(256), 0, st, a.ws);
  }
  return hipGetLastError();
}

}  // namespace skipkv
