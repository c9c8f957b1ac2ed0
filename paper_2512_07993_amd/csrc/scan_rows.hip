// Two-pass key scan of bf16 caches (Sec. 4.1 "Token Importance Score", Eq. 4, and the sentence embedding of
// Eq. 2 over the head's keys), for shapes whose logits cannot wait in registers for the head's normalisers
// (more than 64 query rows) and for whatever else the single-pass scan cannot take:
//   pass A   (reference, sum exp2) of every query row over a run of chunks, and the unit key mean of every
//            sentence;
//   pass B   a head's records merged into log2 of each row's normaliser (by every run for itself, or by k_row_norm before), the
//            logits again, I[t] = (1/alpha) sum_a max_i softmax, and its mean over every sentence.
//
// What bounds it.  With 160 query rows a 256-byte key costs 41 KFLOP and 160 exponentials: both passes are bound by
// the instructions that a SIMD can issue (pass A at 160 rows: about 1250 vector and 220 matrix instructions per 64-key
// tile and CU, 70 and 37 % of a SIMD's cycles at the 1.83 GHz that the chip's power allows such a load), not by HBM.  Products
// pinned among the exponentials of the 16 tokens before them, or fragments read three ahead, changed nothing.  Hence:
//   - a workgroup takes a RUN of up to kMaxRunChunks consecutive chunks of a sequence, so that its query fragments,
//     loaded once, stay in registers for it (no query tile in LDS);
//   - 8 waves; the rows are split over RS of them (2, 4, 8 for up to 16, 40, 64 slots per lane group) and a tile's
//     tokens over the other 8 / RS: 40 slots are four waves' ten, 10 of 12 in whole 16-row products;
//   - keys go HBM -> LDS directly in tiles of 64 rows, three tiles deep, two tiles ahead of the compute, one barrier
//     per tile; a chunk's sentence offsets travel with its tiles;
//   - sentence sums are matrix products of a 0/2 indicator with the transposed key tile, 32 dimensions and 16
//     sentences per wave, so that no wave waits for another one's sentences; the indicator's words come from two additions
//     and a three-way bit operation each;
//   - pass A's row sums are relative to a reference that the wave's first 16 tokens fix for each row: two fmas and one
//     exponential per logit.  Where a later logit is too far above it (2^100) a wave does its share once more by itself,
//     with references that follow the logits.  8 layers x 8 heads, 4 x 16 K tokens, 160 rows, whole score call: 962 us, with
//     such a jump every 4096 / 1024 / 256 tokens 1016 / 1170 / 1338;
//   - what the rare parts of pass A (first tile, ends of chunks, second try) need of the lane's number they compute
//     there: held over the tiles it went to scratch, whose loads wait for the tiles
//     in flight (whole call of the first shape below 10.6 ms instead of 10.0).
// Measured, pass A / pass B / k_row_norm in us, against one workgroup of 256 threads per chunk with the query tile in
// LDS and a running maximum per row, which this replaces:
//   48 layers x 8 heads, 4 x 32 K tokens, 160 rows (50 M keys, 12.9 GB):    7327 / 3926 / 196  ->  3980 / 3210 / 10
//     and where that took 4075 / 3280: 3910 / 3090 with the first tiles' loads in front of the loop (in it, a step without a tile made the compiler move every
//     sum at each tile) and the indicator as it is now (it took shifts and masks, 13 instructions for two words)
//   32 layers x 8 heads, 4 x 3-9 K tokens, 1 % long sentences, 64 rows:      995 /  711 /  23  ->   412 /  338 /  7
// The whole call of the first shape with one, four, up to sixteen chunks per run: 18.0, 11.2, 10.0 ms.  Pass B alone would be
// a little faster in either of two other shapes that pass A is slower in, measured while both took 4189 / 3193: half the waves
// with twice the rows each (256 threads) 4445 / 3110;  32x32x16 products with the rows in two halves 5675 / 2936, the
// logits of a tile no longer fit beside the fragments in pass A.
#include "scan_dev.h"

#include <algorithm>

namespace skipkv {

namespace {

constexpr int kWaves = 8;
constexpr int kTileRows = 64;           // keys per tile: 8 per wave
constexpr int kTileSlots = 3;           // tiles in LDS
constexpr int kAhead = kTileSlots - 1;  // tiles that are loaded ahead of the one computed on
constexpr int kTileLoads = 3;           // direct loads of a wave per tile: 2 x 4 rows and the chunk's offsets
constexpr int kGroupTok = 256;    // pass B: tokens whose importance is summed over the waves at a time

template <int NP, int AL>
struct RowsShape {
  static constexpr int SL = NP * AL;                             // (window query, head) slots of a lane group
  static constexpr int RS = SL <= 16 ? 2 : (SL <= 40 ? 4 : 8);   // waves that share the rows
  static constexpr int TH = kWaves / RS;                         // waves that share the tokens
  static constexpr int ALW = AL / RS;                            // window-query slots per wave
  static constexpr int SPW = NP * ALW;                           // used slots per wave
  static constexpr int NTW = (SPW + 3) / 4;                      // row tiles per wave
  static constexpr int RW = 16 * NTW;                            // query rows per wave
  static constexpr int R = RS * RW;                              // rows of the statistics arrays
  static constexpr int NSUB = 4 / TH;                            // 16-token sub-tiles of a tile per wave
  static constexpr int PG = RS == 8 ? 1 : 4;                     // pass B: lane groups whose parts of the importance go to LDS
  static_assert(AL % RS == 0, "whole window queries per wave");
};

// Where the rows of a head are: contiguous from base, or through a row map.
struct KeyRows {
  const char *base;
  ConstIntPtr map;      // paged cache, else nullptr
  int64_t pitch;        // bytes from a row to the next (of the same block)
  int64_t map_pitch;    // bytes per unit of the map
  int page_size;        // > 0: a power of two >= 16, consecutive slots of a block are one pitch apart
};

// Rows r0 .. r0+3 from token t0 of a sequence of which `last` + 1 rows (from t0) may be read (the others re-read row
// `last`) -> 1 KB at dst, swizzled as rows tile_row + r0 .. of their tile.  (Contiguous caches with a row pitch below
// 16 MB do this in place.)
__device__ __forceinline__ void issue_rows4(const KeyRows &kr, int t0, int last, int r0, int tile_row, int lane, char *dst) {
  const int sub = lane >> 4, r = min(r0 + sub, last);
  const uint32_t piece = (uint32_t)((lane & 15) ^ swz16((tile_row + r0 + sub) & 15)) << 4;
  if (kr.map == nullptr) {
    load_to_lds_16(kr.base + (int64_t)(t0 + r) * kr.pitch + piece, dst);
  } else if (kr.page_size > 0) {  // at most two blocks, consecutive slots in each
    const int jb = kr.page_size - (t0 & (kr.page_size - 1));  // rows before the next block begins
    const char *b0 = kr.base + (int64_t)kr.map[t0] * kr.map_pitch;
    const char *b1 = kr.base + (int64_t)kr.map[t0 + min(jb, last)] * kr.map_pitch - (int64_t)jb * kr.pitch;
    load_to_lds_16((r >= jb ? b1 : b0) + (int64_t)r * kr.pitch + piece, dst);
  } else {  // blocks of any size: every row is looked up, with scalar reads
    int m[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) m[u] = kr.map[t0 + min(r0 + u, last)];
    const int mine = sub == 0 ? m[0] : (sub == 1 ? m[1] : (sub == 2 ? m[2] : m[3]));
    load_to_lds_16(kr.base + (int64_t)mine * kr.map_pitch + piece, dst);
  }
}

__device__ __forceinline__ bf16x8 join_tr(i16x4 lo, i16x4 hi) {
  const uint2 l = __builtin_bit_cast(uint2, lo), h = __builtin_bit_cast(uint2, hi);
  return __builtin_bit_cast(bf16x8, make_uint4(l.x, l.y, h.x, h.y));
}

// The value that lane r of the lane's quad holds.
template <class T>
__device__ __forceinline__ T quad_lane(T v, int r) {  // (r is a constant once unrolled)
  const int x = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(T, r == 0   ? __builtin_amdgcn_mov_dpp(x, 0x00, 0xf, 0xf, true)
                               : r == 1 ? __builtin_amdgcn_mov_dpp(x, 0x55, 0xf, 0xf, true)
                               : r == 2 ? __builtin_amdgcn_mov_dpp(x, 0xAA, 0xf, 0xf, true)
                                        : __builtin_amdgcn_mov_dpp(x, 0xFF, 0xf, 0xf, true));
}

// Fields of a Chunk record as seen through ConstIntPtr.
enum ChunkRec : int { kChB = 0, kChS0, kChNs, kChT, kChLen, kChSoff, kChTok0, kChNTok, kChInts };
static_assert(sizeof(Chunk) == kChInts * 4, "a chunk is read as eight words");

// Chunks per run of a sequence of n chunks: the runs are of one length, the last one is not left with a short rest.
__device__ __forceinline__ int run_length(int n, int run_chunks) {
  const int runs = (n + run_chunks - 1) / run_chunks;
  return (n + runs - 1) / runs;
}

// (reference, sum) of query row r over n > 0 runs of a head, whose records begin at recs: merged in the sequence's order.
__device__ __forceinline__ float2 merge_records(const float2 *recs, int n, int R, int r) {
  float m = kRefInit, s = 0.f;
  for (int u = 0; u < n; u += 8) {
    float2 p[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) p[k] = recs[(int64_t)min(u + k, n - 1) * R + r];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (u + k >= n) break;
      const float nm = fmaxf(m, p[k].x);
      s = s * __builtin_amdgcn_exp2f(m - nm) + p[k].y * __builtin_amdgcn_exp2f(p[k].x - nm);
      m = nm;
    }
  }
  return make_float2(m, s);
}
// Records of the head of a sequence that has n_chunks > 0 chunks from cb on, and how many there are.
__device__ __forceinline__ const float2 *head_records(const ScanArgs &a, int lh, int cb, int n_chunks, int R, int &n) {
  const int rc = a.ws.run_chunks;
  n = (n_chunks + rc - 1) / rc;
  return a.ws.stat_part + ((int64_t)lh * a.ws.nr_max + cb / rc) * R;
}
__device__ __forceinline__ float log2_norm(float2 x) { return x.y > 0.f ? x.x + __builtin_amdgcn_logf(x.y) : INFINITY; }

template <int NP, int AL, bool PASSB, bool SIMPLE>
__global__ void __launch_bounds__(64 * kWaves, 4) k_scan_rows(ScanArgs a) {
  using SH = RowsShape<NP, AL>;
  constexpr int RS = SH::RS, TH = SH::TH, ALW = SH::ALW, SPW = SH::SPW, NTW = SH::NTW, RW = SH::RW, R = SH::R, NSUB = SH::NSUB, PG = SH::PG;
  constexpr int GT = kGroupTok;
  // pass A: sums of squares of the sentence sums [32][4 waves], row statistics [waves][RW][2], references [waves][RW]
  // pass B: importance parts [row part and lane group][GT], importance [GT]
  constexpr int NPART = PG * RS;
  constexpr int NF = PASSB ? (NPART + 1) * GT : 128 + 3 * kWaves * RW;
  __shared__ __align__(256) char kt[kTileSlots][kTileRows * 256];
  __shared__ int soffb[kTileSlots][64];  // offsets of the tile's chunk, the last one repeated (every wave loads the same)
  __shared__ __align__(16) float fbuf[NF];

  const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rh = wave % RS, th = wave / RS;  // the wave's share of the rows and of a tile's tokens
  // Fallback: only sequences and heads that the single-pass scan left, unless everything goes this way.
  if (!a.force_two_pass && a.ws.hdr->n_unfused == 0) return;
  const int n_lh = a.n_layers * a.n_kv_heads;
  const int run_chunks = a.ws.run_chunks, n_runs = hdr_chunks(a.ws.hdr->ranges) / run_chunks;
  const uint32_t n_items = (uint32_t)n_lh * (uint32_t)n_runs;
  const int n = a.n_q_heads / a.n_kv_heads;
  const ConstIntPtr chunks_c = (ConstIntPtr) reinterpret_cast<const int32_t *>(a.ws.chunks);
  const ConstIntPtr chunk_base_c = (ConstIntPtr)a.ws.chunk_base, chunk_cnt_c = (ConstIntPtr)a.ws.chunk_cnt;

  for (uint32_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    // ---- a run: chunks c0 .. c1 - 1 of a sequence, filed under the run_chunks places of the chunk list that the plan
    // keeps for it.  Runs are counted from the sequence's first chunk, wherever its chunks stand in the list: that is up to
    // the order in which the plan's blocks drew their ranges, and a head's sums must not depend on it.
    int lh, run;
    two_pass_item(item, n_runs, lh, run);
    const int b = chunks_c[(int64_t)run * run_chunks * kChInts + kChB];
    const int cb = chunk_base_c[b], n_chunks = chunk_cnt_c[b], len = run_length(n_chunks, run_chunks);
    const int c0 = cb + (run - cb / run_chunks) * len, c1 = min(c0 + len, cb + n_chunks);
    const ConstIntPtr ch0 = chunks_c + (int64_t)c0 * kChInts;
    int n_tiles = 0;
    for (int c = c0; c < c1; ++c) n_tiles += (chunks_c[(int64_t)c * kChInts + kChLen] + kTileRows - 1) / kTileRows;
    if (!a.force_two_pass && a.ws.seq_fused[b] && !a.ws.head_redo[(int64_t)lh * a.batch + b]) continue;  // done by the single-pass scan
    const int l = lh / a.n_kv_heads, h = lh % a.n_kv_heads;
    const int tok0 = ch0[kChTok0], n_tok = ch0[kChNTok], t_first = ch0[kChT];
    const int last_free = n_tok - a.alpha;  // keys t <= last_free are visible to every window query
    KeyRows kr;
    kr.map = !SIMPLE && a.row_map ? (ConstIntPtr)a.row_map + tok0 : nullptr;
    kr.base = static_cast<const char *>(a.k) + ((int64_t)l * a.stride_layer + (int64_t)h * a.stride_head + (!SIMPLE && a.row_map ? 0 : (int64_t)tok0 * a.stride_tok)) * 2;
    kr.pitch = a.stride_tok * 2;
    kr.map_pitch = a.map_stride * 2;
    kr.page_size = (a.page_size >= 16 && (a.page_size & (a.page_size - 1)) == 0) ? a.page_size : 0;

    // lane constants of the LDS addressing, as in the single-pass scan (computed for each run: they need not outlive its tiles)
    const int ol = opaque(lane), ac = ol & 15, ag = ol >> 4;
    const uint32_t b_off = ac * 256 + (((4 * ag) ^ swz16(ac)) << 4);
    const int tr_row = 4 * ag + (ac >> 2);
    const uint32_t tr_off = tr_row * 256 + (((((ac >> 1) & 1) ^ swz16(tr_row)) & 15) << 4) + ((ac & 1) << 3);

    // ---- load stream: tiles of the run in order, chunk by chunk.  A tile's loads come in two parts (part j: rows
    // 4j .. 4j+3 of the wave's eight; the second one also the chunk's offsets, and on to the next tile), so that they
    // can be spread over the compute: issued in one go by all waves they queue up at the CU's address unit.  Rows past
    // a chunk's end re-read its last row, and tiles past the run its last tile's (nobody looks at either): no
    // branch, and the same count every time.
    int lc, lt, lend, lns;
    const int32_t *lso;
    const uint32_t v_piece = (uint32_t)(ac ^ swz16(8 * (wave & 1) + ag)) << 4;
    auto load_chunk = [&](int c) {
      const ConstIntPtr r = chunks_c + (int64_t)c * kChInts;
      lt = r[kChT];
      lend = lt + r[kChLen];
      lso = a.sent_off + r[kChSoff];
      lns = r[kChNs];
    };
    auto issue = [&](int slot, int j) {
      char *dst = kt[slot] + wave * 2048 + j * 1024;
      const int t0 = min(lt + 8 * wave, lend - 1), last = lend - 1 - t0;
      if constexpr (SIMPLE)
        load_to_lds_16_sbase(scalar64(kr.base + (int64_t)t0 * kr.pitch), __umul24((uint32_t)min(4 * j + (lane >> 4), last), (uint32_t)kr.pitch) + (v_piece ^ (uint32_t)(swz16(4 * j) << 4)), dst);
      else
        issue_rows4(kr, t0, last, 4 * j, 8 * (wave & 1), opaque(lane), dst);
      if (j == 1) {
        load_to_lds_4_sbase(scalar64(lso), (uint32_t)min(lane, lns) * 4u, &soffb[slot][0]);
        lt += kTileRows;
        if (lt >= lend && lc + 1 < c1) load_chunk(++lc);
      }
    };
    // slot q = 4 T + j of the wave: window query aq = g + 4 (rh ALW + q / NP), head q % NP
    auto slot_aq = [&](int q) { return g + 4 * (rh * ALW + q / NP); };
    auto slot_used = [&](int q) { return q < SPW && q % NP < n && slot_aq(q) < a.alpha; };
    auto slot_row = [&](int q) { return 16 * (q >> 2) + 4 * g + (q & 3); };
    [[maybe_unused]] float lsum[SPW];                   // pass A: the slots' sums
    [[maybe_unused]] float cn[SPW];                     // pass B: log2 normaliser of the slot's row (+inf: unused slot)
    [[maybe_unused]] float *row_ref = fbuf + 128 + 2 * kWaves * RW + wave * RW;  // pass A: the rows' references
    if constexpr (!PASSB) {
      if (lane < RW) row_ref[lane] = kRefInit;  // (kept by a row that sees no token of the wave)
    }
#pragma unroll
    for (int q = 0; q < SPW; ++q) {
      if constexpr (!PASSB) lsum[q] = 0.f;
    }
    const int p_start = n_tok - min(a.protect, n_tok);  // first protected token

    // Pass A keeps a row's statistics relative to a reference of its own, its largest logit among the wave's first 16 tokens:
    // two fmas and one exponential per logit; a lane group's references are four LDS words per row tile.  Should a row's
    // sum then lie outside what fp32 holds comfortably, the wave does its share of the run once more (below).
    [[maybe_unused]] int my_first = -1;  // becomes 0 once the wave has seen a token
    [[maybe_unused]] int t_ref = 0;      // ... and this is the first one
    [[maybe_unused]] bool not_finite = false;  // some sentence of the wave's half of the chunks has no finite sum
    lc = c0;
    load_chunk(c0);
    // ---- the wave's query fragments: lane (row c16 of a tile, head-dim slice g), as the A operand wants them
    bf16x8 afr[NTW][4];
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
#pragma unroll
      for (int T = 0; T < NTW; ++T) {
        // row c16 of a tile is register (c16 & 3) of lane group c16 / 4 in the output
        const int slot = 4 * T + (c16 & 3), gq = c16 >> 2;
        const int al = rh * ALW + slot / NP, i = slot % NP, aq = gq + 4 * al;
        const bool used = slot < SPW && i < n && aq < a.alpha;
        const int64_t row = (((int64_t)ql * q_batch + qb) * q_heads + (qh * n + (used ? i : 0))) * a.alpha + (used ? aq : 0);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          uint4 v = *reinterpret_cast<const uint4 *>(qbase + row * 256 + g * 64 + kk * 16);
          if (!used) v = make_uint4(0, 0, 0, 0);
          afr[T][kk] = __builtin_bit_cast(bf16x8, v);
        }
      }
    }
    // ---- compute stream
    int cc = c0, ct = t_first, c_t0 = t_first;
    int cend = ct + ch0[kChLen], ns = ch0[kChNs], col = ch0[kChSoff] - b;
    f32x4 pool[2];     // pass A: sentence key sums: slots 16 (wave / 4) + 4g + r, dimensions 16 (2 (wave % 4) + jj) + c16
    float sum_i = 0.f, sum_r = 0.f;  // pass B: thread (sentence tid / 16, part tid % 16)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) pool[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
    asm volatile("" ::: "memory");
    lds_barrier();  // all waves are done with the run before
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      issue(i, 0);
      issue(i, 1);
    }
    if constexpr (PASSB) {
      // log2 of the normaliser of every query row: from the records of the head's runs, merged while the first tiles arrive, as many
      // threads to a row as there are, unless a kernel has done that (scan_norms_apart).
      constexpr int kParts = 64 * kWaves / R;
      float *norm = fbuf + NPART * GT;  // (the tiles' importance takes this place behind another barrier)
      static_assert(R <= GT && 2 * kParts * R <= NPART * GT, "a place for each row, and for each of its parts");
      if (a.norms_apart) {
        if (tid < R) norm[tid] = a.ws.row_norm[((int64_t)lh * a.batch + b) * R + tid];
      } else {
        int n_rec;
        const float2 *recs = head_records(a, lh, cb, n_chunks, R, n_rec);
        const int share = (n_rec + kParts - 1) / kParts, r = tid % R, p0 = tid / R * share;
        float2 *parts = reinterpret_cast<float2 *>(fbuf);
        if (tid < kParts * R) parts[tid] = p0 < n_rec ? merge_records(recs + (int64_t)p0 * R, min(share, n_rec - p0), R, r) : make_float2(kRefInit, 0.f);
        asm volatile("" ::: "memory");
        lds_barrier();
        asm volatile("" ::: "memory");
        if (tid < R) {
          float m = kRefInit, s = 0.f;
#pragma unroll
          for (int p = 0; p < kParts; ++p) m = fmaxf(m, parts[p * R + tid].x);
#pragma unroll
          for (int p = 0; p < kParts; ++p) s += parts[p * R + tid].y * __builtin_amdgcn_exp2f(parts[p * R + tid].x - m);
          norm[tid] = log2_norm(make_float2(m, s));
        }
      }
      asm volatile("" ::: "memory");
      lds_barrier();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int q = 0; q < SPW; ++q) cn[q] = slot_used(q) ? norm[rh * RW + slot_row(q)] : INFINITY;
    }
    int slot = 0;
    for (int i = 0; i < n_tiles; ++i) {
      wait_vm<(kAhead - 1) * kTileLoads>();
      asm volatile("" ::: "memory");
      lds_barrier();  // the tile's rows are there for all waves, and all are done with the tile before it
      asm volatile("" ::: "memory");
      const int fill = slot == 0 ? kTileSlots - 1 : slot - 1;
      auto prefetch = [&](int j) { issue(fill, j); };
      const uint32_t tile_a = lds_addr(kt[slot]);
      const int *soff = soffb[slot];
      slot = slot + 1 == kTileSlots ? 0 : slot + 1;
      const bool chunk_done = ct + kTileRows >= cend;

      // ---- logits: acc[s][T][j] = row 4g + j of the wave's row tile T, token c16 of its sub-tile s
      const int wt = ct + 16 * th * NSUB;  // the wave's first token
      const uint32_t brow = tile_a + th * NSUB * 4096 + b_off;
      f32x4 acc[NSUB][NTW];
      auto logits = [&](int s) {
#pragma unroll
        for (int T = 0; T < NTW; ++T) acc[s][T] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const bf16x8 bfr = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>((uintptr_t)((brow + s * 4096) ^ (kk << 4)));
#pragma unroll
          for (int T = 0; T < NTW; ++T) acc[s][T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr[T][kk], bfr, acc[s][T], 0, 0, 0);
        }
      };
      const bool edge = wt + 16 * NSUB - 1 > last_free;  // some key is hidden from some window query

      if constexpr (!PASSB) {
        if (!edge && my_first == 0) {
#pragma unroll
          for (int s = 0; s < NSUB; ++s) {
            logits(s);
            if (s == 0) prefetch(0);
          }
          float live[NSUB];  // rows past the chunk's end count nothing
#pragma unroll
          for (int s = 0; s < NSUB; ++s) live[s] = wt + 16 * s + c16 < cend ? 1.f : 0.f;
#pragma unroll
          for (int T = 0; T < NTW; ++T) {
            const f32x4 ref = *reinterpret_cast<const f32x4 *>(row_ref + 16 * T + 4 * g);
#pragma unroll
            for (int s = 0; s < NSUB; ++s)
#pragma unroll
              for (int q = 4 * T; q < SPW && q < 4 * T + 4; ++q)
                lsum[q] = fmaf(__builtin_amdgcn_exp2f(fmaf(acc[s][T][q & 3], kScale2, -ref[q & 3])), live[s], lsum[q]);
          }
        } else {
          prefetch(0);
#pragma unroll
          for (int s = 0; s < NSUB; ++s) {
            if (wt + 16 * s >= cend) continue;
            logits(s);
            const int sl = opaque(lane), sc = sl & 15, sg = sl >> 4;  // (lane constants are not kept over the tiles for this)
            const int t = wt + 16 * s + sc, lf = last_free + sg + 4 * rh * ALW;
#pragma unroll
            for (int q = 0; q < SPW; ++q) {
              float x = acc[s][q >> 2][q & 3] * kScale2;
              if (!(t < cend && t <= lf + 4 * (q / NP))) x = -INFINITY;
              acc[s][q >> 2][q & 3] = x;
            }
            if (my_first < 0) {  // the wave's first 16 tokens fix the references
              my_first = 0;
              t_ref = wt + 16 * s;
#pragma unroll
              for (int q = 0; q < SPW; ++q) {
                const float m = fmaxf(row16_max_fast(acc[s][q >> 2][q & 3]), kRefInit);
                row_ref[16 * (q >> 2) + 4 * sg + (q & 3)] = m;  // (all 16 lanes of a row the same: no branch)
              }
            }
#pragma unroll
            for (int q = 0; q < SPW; ++q) lsum[q] += __builtin_amdgcn_exp2f(acc[s][q >> 2][q & 3] - row_ref[16 * (q >> 2) + 4 * sg + (q & 3)]);
          }
        }
        prefetch(1);
        // ---- sentence sums: [16 slots x 32 tokens] indicator (ones written as 2.0, a single bit; the unit
        // normalisation removes the factor) times [32 tokens x 16 dimensions]: waves 0-3 take the chunk's first 16
        // sentences, waves 4-7 the others (if there are any), each 32 of the 128 dimensions.  Lane group g brings
        // tokens 4g .. 4g+3 of two 16-token stages.
        const int pw = wave & 3, u = wave >> 2;
        if (!a.no_pool && ns > 16 * u) {
          // Offsets past the chunk's last one repeat it: empty slots.  Two 16-bit fields to a word, a token each: bit 14 of
          // 0x4000 + token - first is set from the sentence's first token on, that of 0x4000 + token - end from its end on
          const int g4 = opaque(4 * g);  // (no register over the tiles for what follows from it)
          const uint32_t s_lo = (uint32_t)min(max(soff[16 * u + c16] - ct, 0), kTileRows), s_hi = (uint32_t)min(max(soff[16 * u + c16 + 1] - ct, 0), kTileRows);
          const uint32_t tok = __umul24((uint32_t)g4, 0x10001u) + 0x40014000u;  // tokens 4g, 4g + 1
          const uint32_t from = tok - (s_lo << 16 | s_lo), past = tok - (s_hi << 16 | s_hi);
          bf16x8 trv[2][2];
#pragma unroll
          for (int w = 0; w < 2; ++w)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
              const uint32_t ta = ((tile_a + tr_off) ^ ((2 * pw + jj) << 5)) + w * 8192;
              trv[w][jj] = join_tr(lds_read_tr16(ta), lds_read_tr16(ta + 4096));
            }
#pragma unroll
          for (int w = 0; w < 2; ++w) {
            uint32_t ind[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {  // the lane's sentence over tokens 4g + 2 (s % 2) and the next of stage 2w + s / 2
              const uint32_t at = (uint32_t)(32 * w + 16 * (s >> 1) + 2 * (s & 1)) * 0x10001u;
              ind[s] = (from + at) & ~(past + at) & 0x40004000u;
            }
            const bf16x8 av = __builtin_bit_cast(bf16x8, make_uint4(ind[0], ind[1], ind[2], ind[3]));
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) pool[jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, trv[w][jj], pool[jj], 0, 0, 0);
          }
        }
        if (!a.no_pool && chunk_done) {
          // ---- unit sentence embeddings as bf16 hi + lo.  The dimensions of a row are stored as the waves
          // hold them: position 32 pw + 2 c + jj is dimension 16 (2 pw + jj) + c; every embedding of a head
          // is written by this kernel, so cosines are not affected.
          float *sq = fbuf;  // [slot][pw]
          const int el = opaque(lane), ec = el & 15, eg = el >> 4;  // (lane constants are not kept over the tiles for this)
          // A quad's lanes each look after one sentence of their lane group and hand its values round.  Sums are brought to
          // the size of a mean by a power of two, so that their squares leave fp32 no sooner than a mean's.
          const int si = 16 * u + 4 * eg + (ec & 3), len = soff[si + 1] - soff[si];  // 0 past the last sentence
          const float scale = __builtin_amdgcn_ldexpf(1.f, __builtin_clz(len | 1) - 33);
          if (ns > 16 * u) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float by = quad_lane(scale, r);
#pragma unroll
              for (int jj = 0; jj < 2; ++jj) pool[jj][r] *= by;
              const float v = row16_sum_fast(fmaf(pool[0][r], pool[0][r], pool[1][r] * pool[1][r]));
              sq[4 * (16 * u + 4 * eg + r) + pw] = v;
            }
          }
          asm volatile("" ::: "memory");
          lds_barrier();
          asm volatile("" ::: "memory");
          if (ns > 16 * u) {
            const float4 ss4 = *reinterpret_cast<const float4 *>(sq + 4 * si);
            const float ss = ((ss4.x + ss4.y) + ss4.z) + ss4.w;
            not_finite = not_finite || __any(len > 0 && !(ss < INFINITY));
            // mean / (|mean| + eps), both sides times 2 len scale (ones were written as 2.0)
            const float inv = 1.f / (sqrtf(ss) + 2e-12f * (float)len * scale);
            const int64_t o = ((int64_t)lh * a.total_sentences + col + 16 * u) * (kD / 2) + 16 * pw;
            uint32_t *dhi = reinterpret_cast<uint32_t *>(a.ws.vhat_hi) + o, *dlo = reinterpret_cast<uint32_t *>(a.ws.vhat_lo) + o;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float by = quad_lane(inv, r);
              const float u0 = pool[0][r] * by, u1 = pool[1][r] * by;
              const uint32_t hi = pack_bf16x2(u0, u1);
              const uint32_t lo = pack_bf16x2(u0 - __uint_as_float(hi << 16), u1 - __uint_as_float(hi & 0xFFFF0000u));
              if (quad_lane(len, r) > 0) {
                dhi[(4 * eg + r) * (kD / 2) + ec] = hi;
                dlo[(4 * eg + r) * (kD / 2) + ec] = lo;
              }
            }
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) pool[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        }
      } else {
        // ---- token importance: max over the group's heads in registers, exp2, sum over the wave's window queries
        float *parts = fbuf, *imp = fbuf + NPART * GT;
        const int goff = (ct - c_t0) % GT;  // the tile's place in its group of GT tokens
#pragma unroll
        for (int s = 0; s < NSUB; ++s) {
          logits(s);
          if (s == 0) prefetch(0);
        }
#pragma unroll
        for (int s = 0; s < NSUB; ++s) {
          float sum = 0.f;
#pragma unroll
          for (int al = 0; al < ALW; ++al) {
            float gm = -INFINITY;
#pragma unroll
            for (int i2 = 0; i2 < NP; ++i2) {
              const int q = al * NP + i2;
              gm = fmaxf(gm, fmaf(acc[s][q >> 2][q & 3], kScale2, -cn[q]));
            }
            if (edge && wt + 16 * s + c16 > last_free + g + 4 * (rh * ALW + al)) gm = -INFINITY;
            sum += __builtin_amdgcn_exp2f(gm);
          }
          if constexpr (PG == 1) {
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 32);
            if (g == 0) parts[rh * GT + goff + 16 * (th * NSUB + s) + c16] = sum;
          } else {
            parts[(4 * rh + g) * GT + goff + 16 * (th * NSUB + s) + c16] = sum;
          }
        }
        prefetch(1);
        if (chunk_done || goff + kTileRows == GT) {
          // the parts of the importance are added in a fixed order, then the sentences' sums over their
          // unprotected part
          const int g0 = ct - goff, g1 = min(cend, g0 + GT);
          asm volatile("" ::: "memory");
          lds_barrier();
          asm volatile("" ::: "memory");
          if (tid < GT) {
            float tot = 0.f;
#pragma unroll
            for (int p = 0; p < NPART; ++p) tot += parts[p * GT + tid];
            imp[tid] = g0 + tid < g1 ? tot / (float)a.alpha : 0.f;
          }
          asm volatile("" ::: "memory");
          lds_barrier();
          asm volatile("" ::: "memory");
          const int64_t tok_col = (int64_t)lh * a.total_tokens + tok0;
          static_assert(kChunkMaxSent * 16 == 64 * kWaves && GT <= 64 * kWaves, "16 lanes per sentence of a chunk, one thread per token of a group");
          const int si = tid >> 4, sub = tid & 15;
          if (si < ns) {
            const int lo = max(soff[si], g0), hi = min(min(soff[si + 1], p_start), g1);
            for (int t = lo + sub; t < hi; t += 16) {
              sum_i += imp[t - g0];
              if (a.tok_red) sum_r += a.tok_red[tok_col + t];
            }
          }
          if (a.tok_imp && tid < GT && g0 + tid < g1) a.tok_imp[tok_col + g0 + tid] = imp[tid];
          if (chunk_done) {
            sum_i = row16_sum_fast(sum_i);
            if (a.tok_red) sum_r = row16_sum_fast(sum_r);
            if (si < ns && sub == 0) {
              const int len = min(soff[si + 1], p_start) - soff[si];
              const int64_t o = (int64_t)lh * a.total_sentences + col + si;
              a.ws.sent_imp[o] = len > 0 ? sum_i / (float)len : 0.f;
              a.ws.sent_red[o] = len > 0 ? sum_r / (float)len : 0.f;
            }
            sum_i = sum_r = 0.f;
          }
        }
      }
      ct += kTileRows;
      if (ct >= cend && cc + 1 < c1) {
        ++cc;
        const ConstIntPtr r = chunks_c + (int64_t)cc * kChInts;
        c_t0 = ct = r[kChT];
        cend = ct + r[kChLen];
        ns = r[kChNs];
        col = r[kChSoff] - b;
      }
    }  // tiles

    if constexpr (!PASSB) {
      if (not_finite) {
        // An infinite or NaN key: 0 times it is NaN, so the products have carried it into sentences that do not hold it.
        // The embeddings of the half are formed again from each sentence's own rows alone; every wave writes its 32 dimensions.
        const int ln = opaque(lane), pw = wave & 3, u = wave >> 2, d0 = 32 * (ln >> 4) + (ln & 15);
        for (int c = c0; c < c1; ++c) {
          const ConstIntPtr r = chunks_c + (int64_t)c * kChInts;
          const int32_t *off = a.sent_off + r[kChSoff];
          for (int si = 16 * u; si < min(r[kChNs], 16 * u + 16); ++si) {
            float s0 = 0.f, s1 = 0.f;
            const int t1 = off[si + 1], len = t1 - off[si];
            for (int t = off[si]; t < t1; ++t) {
              const char *key = kr.base + (kr.map ? (int64_t)kr.map[t] * kr.map_pitch : (int64_t)t * kr.pitch) + d0 * 2;
              s0 += bf16_bits_to_f32(*reinterpret_cast<const uint16_t *>(key));
              s1 += bf16_bits_to_f32(*reinterpret_cast<const uint16_t *>(key + 32));
            }
            const float scale = 1.f / (float)len, m0 = s0 * scale, m1 = s1 * scale;
            const float inv = 1.f / (sqrtf(wave_sum(fmaf(m0, m0, m1 * m1))) + 1e-12f);
            const uint32_t hi = pack_bf16x2(m0 * inv, m1 * inv);
            const uint32_t lo = pack_bf16x2(m0 * inv - __uint_as_float(hi << 16), m1 * inv - __uint_as_float(hi & 0xFFFF0000u));
            const int64_t o = ((int64_t)lh * a.total_sentences + r[kChSoff] - b + si) * (kD / 2) + ln;
            if (ln >> 4 == pw) {
              reinterpret_cast<uint32_t *>(a.ws.vhat_hi)[o] = hi;
              reinterpret_cast<uint32_t *>(a.ws.vhat_lo)[o] = lo;
            }
          }
        }
      }
      bool doubt = false;
#pragma unroll
      for (int q = 0; q < SPW; ++q) {
        lsum[q] = row16_sum_fast(lsum[q]);
        // rows of padding hold zero queries, and a window query that does not see the wave's first token sees none of its tokens
        doubt = doubt || (slot_used(q) && my_first == 0 && t_ref <= last_free + slot_aq(q) && !(lsum[q] > kMinRowSum && lsum[q] < kMaxRowSum));  // also catches NaN and infinity
      }
      if (__any(doubt)) {
        // The wave's share of the run once more, with references that follow the logits.  Its keys come straight from
        // memory in the layout of the matrix product: no other wave is needed (the others wait for the records).
        const int ln = opaque(lane), lc16 = ln & 15, lg = ln >> 4;  // nothing of this is kept in registers over the tiles
        float m[SPW];
#pragma unroll
        for (int q = 0; q < SPW; ++q) {
          m[q] = kRefInit;
          lsum[q] = 0.f;
        }
        for (int c = c0; c < c1; ++c) {
          const ConstIntPtr r = chunks_c + (int64_t)c * kChInts;
          const int e = r[kChT] + r[kChLen];
          for (int t0 = r[kChT] + 16 * th * NSUB; t0 < e; t0 += kTileRows) {
#pragma unroll 1
            for (int s = 0; s < NSUB; ++s) {
              const int t = t0 + 16 * s + lc16, row = min(t, e - 1);
              const char *key = kr.base + (kr.map ? (int64_t)kr.map[row] * kr.map_pitch : (int64_t)row * kr.pitch) + lg * 64;
              f32x4 x[NTW];
#pragma unroll
              for (int T = 0; T < NTW; ++T) x[T] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int kk = 0; kk < 4; ++kk) {
                const bf16x8 bfr = *reinterpret_cast<const bf16x8 *>(key + kk * 16);
#pragma unroll
                for (int T = 0; T < NTW; ++T) x[T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr[T][kk], bfr, x[T], 0, 0, 0);
              }
#pragma unroll
              for (int q = 0; q < SPW; ++q) {
                const float y = t < e && t <= last_free + lg + 4 * (rh * ALW + q / NP) ? x[q >> 2][q & 3] * kScale2 : -INFINITY;
                const float nm = fmaxf(m[q], row16_max_fast(y));
                lsum[q] = lsum[q] * __builtin_amdgcn_exp2f(m[q] - nm) + __builtin_amdgcn_exp2f(y - nm);
                m[q] = nm;
              }
            }
          }
        }
#pragma unroll
        for (int q = 0; q < SPW; ++q) {
          lsum[q] = row16_sum_fast(lsum[q]);
          row_ref[16 * (q >> 2) + 4 * lg + (q & 3)] = m[q];
        }
      }
      // ---- the run's record; rows of waves that shared the tokens are merged
      float2 *out = a.ws.stat_part + ((int64_t)lh * a.ws.nr_max + run) * R;
      float *wstat = fbuf + 128;
#pragma unroll
      for (int q = 0; q < SPW; ++q) {
        const float2 rec = make_float2(row_ref[slot_row(q)], lsum[q]);
        *reinterpret_cast<float2 *>(wstat + 2 * (wave * RW + slot_row(q))) = rec;  // (all 16 lanes of a row the same)
      }
      asm volatile("" ::: "memory");
      lds_barrier();
      asm volatile("" ::: "memory");
      if (tid < R) {  // (rows past the used slots hold whatever: nobody reads them)
        const int w = tid / RW, r = tid % RW;
        float m = kRefInit;
#pragma unroll
        for (int p = 0; p < TH; ++p) m = fmaxf(m, wstat[2 * ((w + RS * p) * RW + r)]);
        float s = 0.f;
#pragma unroll
        for (int p = 0; p < TH; ++p) {
          const float *x = wstat + 2 * ((w + RS * p) * RW + r);
          s += x[1] * __builtin_amdgcn_exp2f(x[0] - m);
        }
        out[tid] = make_float2(m, s);
      }
    }
  }  // items
  wait_vm<0>();  // the loads past the last tile still write LDS that the workgroup is about to give up
}

// log2 of the softmax normaliser of every query row of a head, for pass B to read.
__global__ void __launch_bounds__(256) k_row_norm(ScanArgs a, int R) {
  const int lhb = blockIdx.x, lh = lhb / a.batch, b = lhb % a.batch;
  if (!a.force_two_pass && a.ws.seq_fused[b] && !a.ws.head_redo[lhb]) return;  // the single-pass scan computed these itself
  const int r = threadIdx.x;
  if (r >= R || a.ws.chunk_cnt[b] == 0) return;
  int n_rec;
  const float2 *recs = head_records(a, lh, a.ws.chunk_base[b], a.ws.chunk_cnt[b], R, n_rec);
  a.ws.row_norm[(int64_t)lhb * R + r] = log2_norm(merge_records(recs, n_rec, R, r));
}

template <int NP, int AL, bool PASSB>
hipError_t launch_rows(const ScanArgs &a, hipStream_t st) {
  static_assert(RowsShape<NP, AL>::R <= 256, "one thread per row merges the records");
  if (a.ws.rows2 != RowsShape<NP, AL>::R) return hipErrorInvalidValue;
  const int64_t items = (int64_t)a.n_layers * a.n_kv_heads * a.ws.nr_max;
  if (items == 0) return hipSuccess;
  // Eight workgroups to a place on the chip balance the passes where there is work for them.  Where they are only the fallback they
  // mostly find nothing to do, and a launch of fewer workgroups is over sooner, which all but large calls notice; unless sentences are
  // so long on average that many do not fit the single pass.  Whole score call, us, 1024 / 4096 workgroups:
  //   sentences of 4-64 tokens (nothing to do), 1.1 M keys 110 / 111    2.1 M 201 / 204    4.2 M 358 / 362    16.8 M 1236 / 1241
  //   1 % of them longer than 512               1.1 M 177 / 177    2.1 M 294 / 292    8.4 M 1009 / 962    16.8 M 1901 / 1777
  //   half of 257, half of 129                  6.1 M 823 / 776
  //   80 % of 129, 20 % of 20                   0.5 M 137 / 136    1.5 M 279 / 254    2.1 M 326 / 291    3.6 M 520 / 460
  const int64_t keys = (int64_t)a.n_layers * a.n_kv_heads * a.total_tokens;
  const bool many = a.force_two_pass || keys >= 6000000 || (keys >= 1000000 && a.total_tokens >= 64 * (int64_t)a.total_sentences);
  const dim3 grid((unsigned)std::min<int64_t>(items, many ? 4096 : 1024));
  if (a.row_map == nullptr && a.stride_tok * 2 < (1 << 24))  // lane offsets by a 24-bit multiply
    hipLaunchKernelGGL((k_scan_rows<NP, AL, PASSB, true>), grid, dim3(64 * kWaves), 0, st, a);
  else
    hipLaunchKernelGGL((k_scan_rows<NP, AL, PASSB, false>), grid, dim3(64 * kWaves), 0, st, a);
  return hipGetLastError();
}

template <bool PASSB>
hipError_t dispatch(const ScanArgs &a, hipStream_t st) {
#define SKIPKV_CASE(NP_, AL_) \
  if (a.rl.np == NP_ && a.rl.al == AL_) return launch_rows<NP_, AL_, PASSB>(a, st);
  SKIPKV_CASE(4, 2)
  SKIPKV_CASE(4, 4)
  SKIPKV_CASE(4, 8)
  SKIPKV_CASE(8, 2)
  SKIPKV_CASE(8, 4)
  SKIPKV_CASE(8, 8)
  SKIPKV_CASE(5, 8)
  SKIPKV_CASE(7, 2)
#undef SKIPKV_CASE
  return hipErrorInvalidValue;
}

}  // namespace

// Chunks per run of `seqs` sequences (of all heads) of some `tokens` tokens each: the least of
//   the runs that a CU does one after the other x (their chunks + 0.9 for the start, which another run half hides)
//   + 0.75 x the chunks of the last ones, when CUs run idle (+ 2 where a run has its CU to itself and hides nothing),
// in chunks of some 240 tokens, and among those within 1 % of it the shortest; but four chunks where there is a sequence
// for every CU, which costs nothing there and leaves short sequences whole, whatever else is in the batch.  Pass A + pass B in us with 1, 3, 6, 16
// chunks, and with the length chosen here:
//   384 sequences of 4096 tokens, 160 rows:          420  291  273  258    271
//   552 of 1253, 96 rows:                            173  134  132  131    140
//   8 of 32000, 160 rows:                             90   73   83  171     74
//   1024 of 3000-9000, 64 rows:                     1050  753  707  763    761
//   480 of 700-5000, 256 rows:                       389  305  327  399    286
//   1536 of 32896, 160 rows:                       11446 7764 6960 6498   6516
// (With eight runs for every workgroup slot of the chip instead, shortest runs for all but the largest calls, the first two
// took 435 and 173; the kernels before, a workgroup per chunk, 365 and 148.)
int scan_run_chunks(int dtype, int64_t seqs, int64_t tokens) {
  if (dtype != SKIPKV_BF16) return 1;
  const int64_t n = std::max<int64_t>(1, (tokens + 239) / 240);
  auto cost = [&](int64_t rc) {  // in twentieths of a chunk
    const int64_t per_seq = (n + rc - 1) / rc, len = (n + per_seq - 1) / per_seq, runs = seqs * per_seq;
    return (runs + 255) / 256 * (20 * len + 18) + 15 * len + (runs <= 256 ? 40 : 0);
  };
  int64_t best = cost(1);
  for (int rc = 2; rc <= kMaxRunChunks; ++rc) best = std::min(best, cost(rc));
  int rc = 1;
  while (cost(rc) * 100 > best * 101) ++rc;
  return seqs >= 256 ? std::max(rc, 4) : rc;
}

int scan_two_pass_rows(const RowLayout &rl, int dtype) {
  if (dtype != SKIPKV_BF16) return rl.rows;
#define SKIPKV_CASE(NP_, AL_) \
  if (rl.np == NP_ && rl.al == AL_) return RowsShape<NP_, AL_>::R;
  SKIPKV_CASE(4, 8)
  SKIPKV_CASE(8, 4)
  SKIPKV_CASE(8, 8)
  SKIPKV_CASE(5, 8)
#undef SKIPKV_CASE
  return rl.rows;  // up to 64 rows: as the single-pass scan lays them out
}

hipError_t launch_rows_stats(const ScanArgs &a, hipStream_t st) { return dispatch<false>(a, st); }
hipError_t launch_rows_scores(const ScanArgs &a, hipStream_t st) { return dispatch<true>(a, st); }

// Whether a kernel between the passes merges the records of a head.  If not, every run of pass B does it for itself, which is
// quadratic in the runs, but hidden and done by eight threads a row (64 rows; 160 rows: three, 256: two) where all runs have a place on the
// chip, and saves calls that leave nothing to the passes a launch.  Whole score call, us, one thread a row / all of them / a
// kernel, by the rows, layers x heads, the tokens of one sequence (runs of a head, of the call):
//   64    1 x 4, 33 K (135, 540): 152 / 113 / 140    2 x 8, 131 K (112, 1792): 524 / 413 / 441    8 x 8, 131 K (56, 3584): 1154 / 1111 / 1125
//   160   1 x 4, 33 K: 167 / 149 / 157    2 x 8, 33 K (45, 720): 180 / 172 / 174    2 x 8, 131 K: 601 / 536 / 511    8 x 8, 33 K (27, 1728):
//         431 / 422 / 419    8 x 8, 131 K: 1476 / 1432 / 1411    32 x 8, 16 K (10, 2560): 707 / 707 / 700
// (nr_max is about 2.2 times the runs.)  The fp32 passes read the kernel's result.
bool scan_norms_apart(const ScanArgs &a) {
  return a.dtype == SKIPKV_F32 || (a.ws.rows2 > 64 && (int64_t)a.n_layers * a.n_kv_heads * a.ws.nr_max > 2400);
}

hipError_t launch_row_norm(const ScanArgs &a, hipStream_t st) {
  const int blocks = a.n_layers * a.n_kv_heads * a.batch;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_row_norm, dim3(blocks), dim3(256), 0, st, a, a.ws.rows2);
  return hipGetLastError();
}

}  // namespace skipkv
