// In-place compaction of K and V (Alg. 1, eviction line): row k of every head becomes the
// row kept_idx[k] it had before.  Pure byte movement.
//
// Because kept_idx is strictly ascending, kept_idx[k] >= k: a row is only ever moved towards
// the front.  One wave owns one (head, K-or-V) stream and walks it front to back in tiles; all
// loads of a tile are complete before its first store, and everything a later tile reads lies
// behind everything already written, so no row is overwritten before it has been read.  The
// leading rows with kept_idx[k] == k are not touched at all.
//
// What bounds it is memory: 5.7 TB/s read and written on large caches.
#include "common.h"

#include <type_traits>

namespace skipkv {

namespace {
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Rows of large caches are read once and written once before anybody comes back to them: they are moved past the caches, and
// displace neither each other nor what the next kernels need.  Small ones are found in the memory-side cache again by
// what follows the call (the next call at the latest).  Whole call, us, ordinary / past the caches, by the rows' bytes in K and V:
//   one sequence, 4096 rows kept:   16 MB 83 / 98   64 MB 92 / 119   128 MB 132 / 141   192 MB 153 / 153   256 MB 181 / 174
//                                   512 MB 306 / 278
//   per-head ranges, 1024 kept:     128 MB 109 / 106   512 MB 305 / 288   2 GB 1058 / 1015
constexpr int64_t kStreamBytes = 192ll << 20;

// 16 bytes that nobody comes back to soon (STREAM), or ordinary ones.
template <bool STREAM>
__device__ __forceinline__ u32x4 load16(const char *p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
  return *reinterpret_cast<const u32x4 *>(p);
}
template <bool STREAM>
__device__ __forceinline__ void store16(char *p, u32x4 x) {
  if constexpr (STREAM) __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(p));
  else *reinterpret_cast<u32x4 *>(p) = x;
}

// Paged cache (PAGED): rows live in block slots.  Sources come pre-translated (src_rows: slot row of
// kept_idx[k], written by k_kept_rows below), destinations are read from the row map one coalesced
// load per tile, issued right before the tile's row loads.  Logical positions still only move
// forward and distinct logical rows are distinct slots, so the order argument above holds.
//
// A stream: the rows of K or of V of a head of a sequence, and where they go.
template <int ROWB, bool PAGED>
struct Stream {
  char *base;            // first row of the sequence (paged: the head's base)
  int64_t pitch;         // paged: of the units of the row map
  const int32_t *kept;   // the head's row of indices
  const int32_t *srcs;   // what the row loads are addressed with
  const int32_t *rmap;   // paged: slot rows of the sequence
  int nl, room;          // rows kept; rows of the sequence (contiguous cache: a source index is one of them)
  bool valid;

  __device__ __forceinline__ Stream(const CompactArgs &a, uint32_t sid) {
    constexpr int ESZ = ROWB / kD;
    // the arguments in one go, and what they point to (else there are waits for a few of them at a time, all along the way)
    asm volatile("" ::"s"(a.k), "s"(a.v), "s"(a.stride_layer), "s"(a.stride_head), "s"(a.stride_tok), "s"(a.seq_off), "s"(a.kept_idx), "s"(a.new_len));
    const uint32_t lhb = sid >> 1, lh = lhb / (uint32_t)a.batch, b = lhb - lh * (uint32_t)a.batch;
    nl = a.new_len[lhb];
    const int t0 = a.seq_off[b], t1 = a.seq_off[b + 1];
    const bool bad = PAGED && a.seq_bad[b];
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t l = lh / (uint32_t)a.n_kv_heads, h = lh - l * (uint32_t)a.n_kv_heads;
    base = static_cast<char *>((sid & 1) ? a.v : a.k) + ((int64_t)l * a.stride_layer + (int64_t)h * a.stride_head + (PAGED ? 0 : (int64_t)t0 * a.stride_tok)) * ESZ;
    pitch = (PAGED ? a.map_stride : a.stride_tok) * ESZ;
    kept = a.kept_idx + (int64_t)lhb * a.kept_stride;
    srcs = PAGED ? a.src_rows + (int64_t)lhb * a.src_stride : kept;
    rmap = PAGED ? a.row_map + t0 : nullptr;
    room = t1 - t0;
    // An invalid block table: leave the sequence alone.  A head that kept everything because its inputs could not be trusted reports
    // its full length, which its row of indices may not even hold: nothing to move, and nothing to read past the row.
    valid = !bad && nl <= a.kept_stride && !(PAGED && nl > a.src_stride);
  }
};

// Whether a stream's rows are moved past the caches: where the call's rows are so many (kStreamBytes).  A row of indices is often much
// longer than what is kept, so that the host only knows that they may be.  Here: if they were with every head as long as the
// stream's own (rows of shorter ones displace little), and are by the lengths of eight heads spread over the call, which are loaded
// together with its own.  The call alone, us, by the list's pitch / like this: 512 streams of 1024 rows in lists of 2000: 57 / 42, 8192 of
// 64: 38 / 33 (lists of as many: 42, 33).
struct Spread {
  int len[8];
  __device__ __forceinline__ explicit Spread(const CompactArgs &a) {
    typedef const __attribute__((address_space(4))) int32_t *ConstIntPtr;  // constant while the kernel runs: scalar loads
    const ConstIntPtr new_len = (ConstIntPtr)a.new_len;
    const uint32_t heads = (uint32_t)(a.n_layers * a.n_kv_heads * a.batch);
#pragma unroll
    for (uint32_t i = 0; i < 8; ++i) len[i] = new_len[(uint32_t)(((uint64_t)(i * 0x9E3779B9u) * heads) >> 32)];
    __builtin_amdgcn_sched_barrier(0);  // (all of them under way, and nothing waits for them yet)
  }
  __device__ __forceinline__ bool past_the_caches(const CompactArgs &a, int nl, int row_bytes) const {
    int64_t rows = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) rows += len[i] <= a.kept_stride ? max(len[i], 0) : 0;
    return min(rows, (int64_t)8 * nl) * ((int64_t)a.n_layers * a.n_kv_heads * a.batch) * 2 * row_bytes > 8 * kStreamBytes;
  }
};
struct NoSpread {
  __device__ __forceinline__ explicit NoSpread(const CompactArgs &) {}
  __device__ __forceinline__ bool past_the_caches(const CompactArgs &, int, int) const { return false; }
};

// SL: bytes of a row that a wave moves.  The argument above holds for every byte column of a stream by
// itself, so a stream may be split into ROWB / SL waves that know nothing of each other; launch_compact
// says when.
template <int ROWB, int SL, bool PAGED, bool STREAM>
__device__ __forceinline__ void move_slice(const Stream<ROWB, PAGED> &x, char *base, int lane) {
  constexpr int PPR = SL / 16;     // 16-byte pieces per row slice
  constexpr int RPI = 64 / PPR;    // rows moved by one wave-wide instruction
  constexpr int U = 8;             // instructions in flight per tile
  const int64_t pitch = x.pitch;
  const int32_t *kept = x.kept, *srcs = x.srcs, *rmap = x.rmap;
  const int nl = x.nl, room = x.room;

  // first row that actually moves
  int first = nl;
  for (int k0 = 0; k0 < nl; k0 += 64) {
    const int k = k0 + lane;
    const unsigned long long moved = __ballot(k < nl && kept[k] != k);
    if (moved) {
      first = k0 + __ffsll((long long)moved) - 1;
      break;
    }
  }

  // Software pipeline, two tiles deep.  Tile i's loads may be issued before tile i-1's stores
  // (a tile only reads rows at or behind its own first row, a tile's stores only write rows of
  // that tile), so the wave always has one tile of loads and one tile of stores in flight; the
  // only ordering kept is that a tile's own loads have landed before its stores.  Vector memory
  // operations complete in issue order, which lets a counted wait express exactly that.  The
  // tile's source indices come in with one coalesced load, a tile ahead of their use.
  const int sub = lane / PPR, piece = lane % PPR;
  constexpr int TR = U * RPI;  // rows per tile
  constexpr int NI = (TR + 63) / 64;  // index loads per tile: lane i of load n holds row 64 n + i
  static_assert(NI <= 2 && (NI == 1 || U * RPI == 128), "instructions 0..3 take their rows from the first load, 4..7 from the second");
  auto load_idx = [&](int k0) -> int {  // unconditional (clamped), so that it always counts as one outstanding load
    const int i = srcs[min(k0 + lane, nl - 1)];
    return PAGED ? i : max(0, min(i, room - 1));  // never address a row outside the sequence, whatever the indices say
  };
  auto load_dst = [&](int k0) -> int {  // paged: slot rows of the tile's destinations (same rule)
    return PAGED ? rmap[min(k0 + lane, nl - 1)] : 0;
  };
  if (first >= nl) return;
  // The two tiles are written out as named registers (A0..A7, B0..B7): arrays carried around the
  // loop end up in scratch memory with this compiler.
  static_assert(U == 8, "the tiles below are spelled out for 8 instructions");
#define SKIPKV_EACH(X, T) X(T, 0) X(T, 1) X(T, 2) X(T, 3) X(T, 4) X(T, 5) X(T, 6) X(T, 7)
#define SKIPKV_DECL(T, u) u32x4 T##u;
  // always U loads per tile: rows past the end re-read the last kept row (index loads are clamped)
#define SKIPKV_LOAD(T, u) \
  T##u = load16<STREAM>(base + (int64_t)__shfl(NI == 2 && u >= 4 ? idx2_##T : idx_##T, (u * RPI + sub) & 63) * pitch + piece * 16);
  // destination row of the lane's piece: position in the sequence, or (paged) its slot row; the shuffle
  // is taken by all lanes, outside any condition
#define SKIPKV_DROW(T, u) const int64_t dr_##u = PAGED ? (int64_t)__shfl(NI == 2 && u >= 4 ? dst2_##T : dst_##T, (u * RPI + sub) & 63) : (int64_t)(ks + u * RPI + sub);
#define SKIPKV_STORE(T, u) store16<STREAM>(base + dr_##u * pitch + piece * 16, T##u);
#define SKIPKV_STORE_TAIL(T, u) \
  if (ks + u * RPI + sub < nl) store16<STREAM>(base + dr_##u * pitch + piece * 16, T##u);
#define SKIPKV_STORE_TILE(T, K0)        \
  {                                     \
    const int ks = (K0);                \
    SKIPKV_EACH(SKIPKV_DROW, T)         \
    if (ks + TR <= nl) {                \
      SKIPKV_EACH(SKIPKV_STORE, T)      \
    } else {                            \
      SKIPKV_EACH(SKIPKV_STORE_TAIL, T) \
    }                                   \
  }
  // Wait until the loads of the tile about to be stored have landed.  Behind them in the queue
  // are the previous tile's U stores (none for the first tile), NI index loads and the next
  // tile's U loads (paged: plus the NI loads of the next tile's destination rows, NX of them).  The next tile is always loaded, also past the end (clamped, one tile of
  // wasted reads per stream): unconditional loads keep the counts exact and the registers in place.
  SKIPKV_EACH(SKIPKV_DECL, A)
  SKIPKV_EACH(SKIPKV_DECL, B)
  constexpr int NX = PAGED ? NI : 0;
  int idx_A = load_idx(first), idx2_A = NI == 2 ? load_idx(first + 64) : 0;
  int idx_B = load_idx(first + TR), idx2_B = NI == 2 ? load_idx(first + TR + 64) : 0;
  int dst_A = load_dst(first), dst2_A = NI == 2 ? load_dst(first + 64) : 0, dst_B = 0, dst2_B = 0;
  SKIPKV_EACH(SKIPKV_LOAD, A)
  for (int k0 = first;; k0 += 2 * TR) {
    idx_A = load_idx(k0 + 2 * TR);
    if constexpr (NI == 2) idx2_A = load_idx(k0 + 2 * TR + 64);
    dst_B = load_dst(k0 + TR);
    if constexpr (NI == 2) dst2_B = load_dst(k0 + TR + 64);
    SKIPKV_EACH(SKIPKV_LOAD, B)
    if (k0 != first)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * U + NI + NX) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(U + NI + NX) : "memory");
    SKIPKV_STORE_TILE(A, k0)
    if (k0 + TR >= nl) break;
    idx_B = load_idx(k0 + 3 * TR);
    if constexpr (NI == 2) idx2_B = load_idx(k0 + 3 * TR + 64);
    dst_A = load_dst(k0 + 2 * TR);
    if constexpr (NI == 2) dst2_A = load_dst(k0 + 2 * TR + 64);
    SKIPKV_EACH(SKIPKV_LOAD, A)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * U + NI + NX) : "memory");
    SKIPKV_STORE_TILE(B, k0 + TR)
    if (k0 + 2 * TR >= nl) break;
  }
#undef SKIPKV_EACH
#undef SKIPKV_DECL
#undef SKIPKV_LOAD
#undef SKIPKV_STORE
#undef SKIPKV_DROW
#undef SKIPKV_STORE_TAIL
#undef SKIPKV_STORE_TILE
}

// LARGE: the rows may be so many that they are moved past the caches.
template <int ROWB, int SL, bool PAGED, bool LARGE>
__global__ void __launch_bounds__(256) k_compact(CompactArgs a) {
  constexpr int NS = ROWB / SL;  // waves per stream
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t wid = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave, sid = wid / NS;
  if (sid >= 2 * (int64_t)a.n_layers * a.n_kv_heads * a.batch) return;
  const std::conditional_t<LARGE, Spread, NoSpread> all(a);
  const Stream<ROWB, PAGED> x(a, (uint32_t)sid);
  if (!x.valid) return;
  char *base = x.base + (int)(wid % NS) * SL;
  if (LARGE && all.past_the_caches(a, x.nl, ROWB)) move_slice<ROWB, SL, PAGED, true>(x, base, lane);
  else move_slice<ROWB, SL, PAGED, false>(x, base, lane);
}

// The same by a workgroup of eight waves per slice of a stream, which moves eight tiles at a time: all rows of a step have
// landed in registers before the first of them is stored, so no wave overwrites what another one still has to read, and a
// step's loads may pass the stores of the one before, which lie in front of everything they read.  For few streams,
// whose chains of tiles would otherwise be most of the time (launch_compact says when).
template <int ROWB, int SL, bool PAGED, bool STREAM>
__device__ __forceinline__ void move_steps(const Stream<ROWB, PAGED> &x, char *base, int first, int wave, int lane) {
  constexpr int PPR = SL / 16;     // 16-byte pieces per row slice
  constexpr int RPI = 64 / PPR;    // rows moved by one wave-wide instruction
  constexpr int U = 8;             // instructions per wave and step
  constexpr int TR = U * RPI;      // rows per wave and step
  const int sub = lane / PPR, piece = lane % PPR, nl = x.nl;
  int src[U], dst[U];
  auto load_rows = [&](int k0) {  // (clamped: rows past the end are the last one)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(k0 + wave * TR + u * RPI + sub, nl - 1);
      src[u] = x.srcs[k];
      if constexpr (PAGED) dst[u] = x.rmap[k];
      else {
        src[u] = max(0, min(src[u], x.room - 1));
        dst[u] = k;
      }
    }
  };
  if (first < nl) load_rows(first);
  for (int k0 = first; k0 < nl; k0 += 8 * TR) {
    u32x4 v[U];
    char *to[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] = load16<STREAM>(base + (int64_t)src[u] * x.pitch + piece * 16);
      to[u] = base + (int64_t)dst[u] * x.pitch + piece * 16;
    }
    load_rows(k0 + 8 * TR);
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7])::"memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k0 + wave * TR + u * RPI + sub < nl) store16<STREAM>(to[u], v[u]);
  }
}

template <int ROWB, int SL, bool PAGED, bool LARGE>
__global__ void __launch_bounds__(512) k_compact_steps(CompactArgs a, int step_rows) {
  constexpr int NS = ROWB / SL;  // workgroups per stream
  constexpr int SCAN = 4;        // indices per thread of one look for the first row that moves
  constexpr int SHORT = 64;      // slices of streams that are too short for this: of as few streams' otherwise (launch_compact)
  __shared__ int first_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const std::conditional_t<LARGE, Spread, NoSpread> all(a);
  const Stream<ROWB, PAGED> x(a, blockIdx.x / NS);
  if (!x.valid) return;
  const int nl = x.nl, at_byte = (int)(blockIdx.x % NS) * SL;
  if (__builtin_expect(nl < step_rows, false)) {
    if (wave < SL / SHORT) move_slice<ROWB, SHORT, PAGED, false>(x, x.base + at_byte + wave * SHORT, lane);
    return;
  }

  int first = nl;
  for (int k0 = 0; k0 < nl; k0 += 512 * SCAN) {
    if (tid == 0) first_s = nl;
    __syncthreads();
    int mine = nl, at[SCAN];
#pragma unroll
    for (int j = 0; j < SCAN; ++j) at[j] = x.kept[min(k0 + 512 * j + tid, nl - 1)];  // (all of them before the first is looked at)
#pragma unroll
    for (int j = SCAN - 1; j >= 0; --j) {
      const int k = k0 + 512 * j + tid;
      if (k < nl && at[j] != k) mine = k;
    }
    if (mine < nl) atomicMin(&first_s, mine);
    __syncthreads();
    first = first_s;
    if (first < nl) break;
    __syncthreads();
  }
  if (LARGE && all.past_the_caches(a, nl, ROWB)) move_steps<ROWB, SL, PAGED, true>(x, x.base + at_byte, first, wave, lane);
  else move_steps<ROWB, SL, PAGED, false>(x, x.base + at_byte, first, wave, lane);
}

// Paged cache: src_rows[head, k] = slot row of the head's kept token k, for k < new_len (one wave
// per head; shared by the K and the V stream of the head).
__global__ void __launch_bounds__(256) k_kept_rows(CompactArgs a) {
  const int64_t lhb = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (lhb >= (int64_t)a.n_layers * a.n_kv_heads * a.batch) return;
  const int b = (int)(lhb % a.batch), lane = threadIdx.x & 63;
  if (a.seq_bad[b]) return;
  const int32_t *kept = a.kept_idx + lhb * a.kept_stride;
  const int32_t *rmap = a.row_map + a.seq_off[b];
  int32_t *out = a.src_rows + lhb * a.src_stride;
  const int nl = min(min(a.new_len[lhb], a.src_stride), a.kept_stride);
  const int room = a.seq_off[b + 1] - a.seq_off[b];
  for (int k = lane; k < nl; k += 64) out[k] = rmap[max(0, min(kept[k], room - 1))];
}

template <int ROWB, int SL, bool LARGE>
void launch_slices(const CompactArgs &a, int64_t streams, hipStream_t st) {
  const unsigned grid = (unsigned)((streams * (ROWB / SL) + 3) / 4);
  if (a.row_map)
    hipLaunchKernelGGL((k_compact<ROWB, SL, true, LARGE>), dim3(grid), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((k_compact<ROWB, SL, false, LARGE>), dim3(grid), dim3(256), 0, st, a);
}

// The caller's row of indices bounds the rows.  (Slices of 64 bytes are for so few streams that, where the bound is beyond kStreamBytes,
// it is beyond kStepRowsLong, too: those move in steps.)
template <int ROWB, int SL>
void launch_slices(const CompactArgs &a, int64_t streams, hipStream_t st) {
  if (SL > 64 && streams * a.kept_stride * ROWB > kStreamBytes) launch_slices<ROWB, SL, (SL > 64)>(a, streams, st);
  else launch_slices<ROWB, SL, false>(a, streams, st);
}

template <int ROWB, bool LARGE>
void launch_steps(const CompactArgs &a, int64_t streams, int step_rows, hipStream_t st) {
  constexpr int SL = 128;
  const dim3 grid((unsigned)(streams * (ROWB / SL)));
  if (a.row_map)
    hipLaunchKernelGGL((k_compact_steps<ROWB, SL, true, LARGE>), grid, dim3(512), 0, st, a, step_rows);
  else
    hipLaunchKernelGGL((k_compact_steps<ROWB, SL, false, LARGE>), grid, dim3(512), 0, st, a, step_rows);
}

template <int ROWB>
void launch_steps(const CompactArgs &a, int64_t streams, int step_rows, hipStream_t st) {
  if (streams * a.kept_stride * ROWB > kStreamBytes) launch_steps<ROWB, true>(a, streams, step_rows, st);
  else launch_steps<ROWB, false>(a, streams, step_rows, st);
}

}  // namespace

// A stream is a serial chain of tiles, so with few streams the chip waits for memory.  Long chains of few streams are
// therefore moved eight tiles at a time by workgroups of eight waves, in slices of 128 bytes.  The call alone, us, a wave
// per slice / this, by streams and rows kept:
//   bf16       600           1024          2500          4096           3000 (of 12000)   16000
//     8        7.4 / 7.6     8.2 / 8.0     15.3 / 11.1   21.7 / 13.5    17.6 / 12.2       118 / 49
//     64       7.5 / 8.6     9.4 / 9.5     24.4 / 18.1   36.1 / 24.1    28.8 / 21.8       262 / 106
//     128      7.7 / 9.6     11.8 / 11.8   28.7 / 29.6   41.3 / 40.4    39.3 / 35.7       289 / 192
//     256      12.9 / 13.0   21.6 / 21.7   53.8 / 53.1   97.1 / 88.1    81.6 / 70.9
//     512      -             38.3 / 41.2   -             175 / 174
//   paged 64   17.9 / 19.2   23.5 / 22.3   54.5 / 46.7   76.9 / 62.7    63.9 / 54.3
//   paged 256  24.6 / 24.3   35.9 / 35.4   79.0 / 78.0   144 / 135      124 / 114
//   fp32 rows are twice as long: 64 streams of them behave like 128 of bf16
// Slices of 64 bytes take this up to twice as long from 64 streams on, and whole rows half as much again at 8.  Streams are
// counted in columns of 256 bytes.  The host goes by the caller's row of indices, which bounds the rows; a stream that turns out to keep
// fewer rows than the lines below is moved by a wave per slice all the same (128 streams of 600 rows in lists of 3000, us: in steps 9.6,
// like this 7.7, lists of 600 8.5).
constexpr int64_t kStepColumns = 64, kStepRows = 1024, kStepColumnsLong = 256, kStepRowsLong = 2560;

// Otherwise rows are split into slices of 128 or 64 bytes (half a cache line: the least that a wave should take) as long as that makes no more
// than 1024 waves, four per CU.  More waves than that gain nothing and the smaller pieces cost: whole step of 8 heads
// per layer and 4224 tokens, us, with rows in 1 / 2 / 4 / 8 slices:
//   bf16   32 streams: 154 / 116 / 97    128: 208 / 165 / 148    256: 288 / 217 / 199    512: 370 / 362 / 406
//          768: 455 / 476 / 498    8192: 2333 / 2299 / 2573
//   fp32   16 streams: 111 / 103 / 92 / 88    64: 333 / 235 / 191 / 176    256: 592 / 442 / 386 / 418
hipError_t launch_compact(const CompactArgs &a, hipStream_t st) {
  const int64_t heads = (int64_t)a.n_layers * a.n_kv_heads * a.batch, streams = 2 * heads;
  if (streams == 0) return hipSuccess;
  if (a.row_map) hipLaunchKernelGGL(k_kept_rows, dim3((unsigned)((heads + 3) / 4)), dim3(256), 0, st, a);
  const int64_t fit = 1024 / streams;  // slices that make at most 1024 waves
  const int64_t columns = streams * (a.dtype == SKIPKV_BF16 ? 1 : 2);
  const int64_t step_rows = columns <= kStepColumns ? kStepRows : kStepRowsLong;
  if (columns <= kStepColumnsLong && a.kept_stride >= step_rows) {
    // Budgets that whole sentences fill leave a list a little short.  And two waves of a workgroup of eight are slower at more than some 160
    // columns than waves by themselves: rather steps, there, too.
    const int fewest = (int)(columns > 160 || step_rows == kStepRows ? kStepRows * 7 / 8 : step_rows);
    if (a.dtype == SKIPKV_BF16) launch_steps<256>(a, streams, fewest, st);
    else launch_steps<512>(a, streams, fewest, st);
  } else if (a.dtype == SKIPKV_BF16) {
    if (fit >= 4) launch_slices<256, 64>(a, streams, st);
    else if (fit >= 2) launch_slices<256, 128>(a, streams, st);
    else launch_slices<256, 256>(a, streams, st);
  } else {
    if (fit >= 8) launch_slices<512, 64>(a, streams, st);
    else if (fit >= 4) launch_slices<512, 128>(a, streams, st);
    else if (fit >= 2) launch_slices<512, 256>(a, streams, st);
    else launch_slices<512, 512>(a, streams, st);
  }
  return hipGetLastError();
}

}  // namespace skipkv
