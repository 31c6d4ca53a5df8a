// gfx950 kernels and entry points of the C ABI that move KV tokens between
// the page pools and dense token-major buffers, bit for bit:
// gather_kernel: paged tokens out into a dense buffer (the read-back of the
//   paged KV cache);
// scatter_kernel: new tokens into their pages (a decode append or a prefill
//   chunk), the write path of the cache;
// page_copy_kernel: whole-page copies (the copy of copy-on-write).
// Pool layouts: K pages [H][D/E][16][E] (E elements per 16 bytes), V pages
// [H][D][16] with token slots permuted as below.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "halo_internal.h"

using namespace halo;

namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// V pages keep the tokens of a dim row in the slot order 0-3, 8-11, 4-7,
// 12-15 (bits 2 and 3 of the index swapped; the map is its own inverse).
__device__ __forceinline__ int v_token_at_slot(int s) { return (s & 3) | ((s & 4) << 1) | ((s & 8) >> 1); }

// ---------------------------------------------------------------- gather

struct GatherArgs {
  const void* pool;
  const int32_t* page_ids;
  const int32_t* seq_page_indptr;
  const int32_t* seq_len;
  const int64_t* out_token_offset;
  void* out;
  int32_t* error_flag;
  int64_t num_pool_pages;
  int32_t num_seqs;
  int32_t num_kv_heads;
  int32_t head_dim;
  int32_t v_layout;
};

// The last index s < n with indptr[s] <= x, for a nondecreasing indptr with
// indptr[0] <= x (wave-uniform x): the wave compares 64 evenly spaced
// entries at once and keeps the bracket that holds the answer, so up to 4095
// entries take two rounds of loads where a binary search takes twelve.
__device__ __forceinline__ int last_at_or_below(const int32_t* indptr, int n, int64_t x, int lane) {
  int lo = 0, len = n;
  while (len > 64) {
    const int stride = (len + 63) / 64;
    const int off = lane * stride;
    const bool hit = off < len && indptr[lo + off] <= x;
    const uint64_t mask = __ballot(hit);
    const int top = 63 - __clzll(mask);          // lane 0 always hits
    lo += top * stride;
    len = min(stride, len - top * stride);
  }
  const bool hit = lane < len && indptr[lo + lane] <= x;
  const uint64_t mask = __ballot(hit);
  return lo + 63 - __clzll(mask);
}

// Tiles t_begin .. t_end - 1 by one wave; `stage`: its LDS buffer. The two
// kinds of loads and stores are two loops: in one, the compiler merges them and
// drops the non-temporal hint.
template <typename W, int D, bool STREAM>
__device__ __forceinline__ void gather_run(const GatherArgs& a, u32x4_t* stage, int first, int64_t t_begin,
                                           int64_t t_end, int lane) {
  constexpr int E = 16 / (int)sizeof(W);   // elements per 16-byte vector
  constexpr int VPT = D / E;               // vectors per token and head
  constexpr int NV = 16 * VPT / 64;        // vectors per lane for a tile
  constexpr int ROW = D + E;               // staged row, in words (16-byte aligned)
  const int H = a.num_kv_heads;
  const int64_t row = (int64_t)H * D;      // output elements per token
  const W* pool = static_cast<const W*>(a.pool);
  W* out = static_cast<W*>(a.out);
  W* st = reinterpret_cast<W*>(stage);
  // indptr[0] <= first + t_begin / H, so the search returns a sequence in
  // [0, num_seqs); the walk below stops at num_seqs - 1 at the latest, since
  // every slot is < indptr[num_seqs]
  int seq = last_at_or_below(a.seq_page_indptr, a.num_seqs, first + t_begin / H, lane);
  int base = a.seq_page_indptr[seq], next = a.seq_page_indptr[seq + 1];
  for (int64_t tl = t_begin; tl < t_end; ++tl) {
    const int slot = first + (int)(tl / H), h = (int)(tl % H);
    while (slot >= next) {             // later sequences (empty ones are passed over)
      ++seq;
      base = next;
      next = a.seq_page_indptr[seq + 1];
    }
    const int len = a.seq_len[seq];
    const int pid = a.page_ids[slot];
    if (len < 0 || next - base != (len + 15) / 16 || pid < 0 || pid >= a.num_pool_pages) {
      if (lane == 0 && a.error_flag) a.error_flag[0] = 1;
      continue;
    }
    const int t0 = (slot - base) * 16;
    const int n = min(16, len - t0);
    const W* src = pool + ((int64_t)pid * H + h) * 16 * D;
    u32x4_t v[NV];
    const u32x4_t* src16 = reinterpret_cast<const u32x4_t*>(src) + lane;
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = STREAM ? __builtin_nontemporal_load(src16 + 64 * i) : src16[64 * i];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int idx = lane + 64 * i;
      if (!a.v_layout) {             // K: vector idx = (dims j*E.., token t)
        const int j = idx / 16, t = idx % 16;
        *reinterpret_cast<u32x4_t*>(st + t * ROW + j * E) = v[i];
      } else {                       // V: vector idx = (dim c, slots part*E..)
        const int c = idx / (16 / E), part = idx % (16 / E);
        const W* e = reinterpret_cast<const W*>(&v[i]);
#pragma unroll
        for (int q = 0; q < E; ++q) st[v_token_at_slot(part * E + q) * ROW + c] = e[q];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    W* dst = out + (a.out_token_offset[seq] + t0) * row + (int64_t)h * D;
    for (int idx = lane; idx < n * VPT; idx += 64) {
      const int tok = idx / VPT, j = idx % VPT;
      const u32x4_t x = *reinterpret_cast<const u32x4_t*>(st + tok * ROW + j * E);
      u32x4_t* to = reinterpret_cast<u32x4_t*>(dst + tok * row + j * E);
      if constexpr (STREAM) __builtin_nontemporal_store(x, to);
      else *to = x;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// The (page slot, head) tiles of all sequences, in order, are cut into equal
// contiguous runs, one per wave, so a few long sequences among many short
// ones spread over the whole grid. A wave finds the sequence of its first
// tile by binary search over seq_page_indptr and walks forward from there.
// Per tile it reads the tile in its stored order with 16-byte loads
// (coalesced), stages it token-major in its own LDS buffer ([16][D + E]
// words, rows 16-byte aligned) and writes the tile's tokens as dense rows,
// 16 bytes per lane. K vectors hold E dims of one token and move whole; V
// vectors hold one dim of E tokens and are split into single words on the
// way into LDS. W is an unsigned word of the element's width, so every bit
// pattern (NaN payloads included) moves unchanged. Bound by HBM: tiles are
// read and rows written once. A launch of more than kGatherCached bytes reads
// and writes past the caches (64 sequences of 256-2048 tokens, K and V, 595 MB:
// 134 -> 124.4 us, 4.8 TB/s, a device copy's rate; 128 MB each, and a copy that
// reads the rows next: 218 -> 214 us, after other work 241 -> 227). Tiles and
// rows of smaller launches may stay in the last-level cache, for this call and
// for the reader of the rows. K and V of 8 / 32 / 60 MB each, gathered and then
// copied: cached 21.9 / 45.7 / 92.8 us, rows past the caches 22.9 / 50.7 / 102;
// after other work 24.8 / 66.7 / 128 and 28.5 / 77.4 / 130. (The gather alone,
// its tiles still cached: 9.3 / 24.8 / 48.3 and 9.3 / 23.8 / 41.4.)
constexpr int64_t kGatherCached = (int64_t)64 << 20;
template <typename W, int D>
__global__ __launch_bounds__(256) void gather_kernel(GatherArgs a) {
  constexpr int E = 16 / (int)sizeof(W);
  __shared__ u32x4_t stage[4][16 * (D + E) / E];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int H = a.num_kv_heads;

  // page-list slots first .. last-1 are tiled; first need not be 0 (a
  // slice of a larger page list)
  const int first = a.seq_page_indptr[0];
  const int64_t total = ((int64_t)a.seq_page_indptr[a.num_seqs] - first) * H;
  const int64_t waves = (int64_t)gridDim.x * 4;
  const int64_t per = (total + waves - 1) / waves;
  const int64_t w_id = (int64_t)blockIdx.x * 4 + wave;
  const int64_t t_begin = w_id * per;
  const int64_t t_end = min(total, t_begin + per);
  if (t_begin >= t_end) return;
  if (total * 16 * D * (int64_t)sizeof(W) > kGatherCached)
    gather_run<W, D, true>(a, stage[wave], first, t_begin, t_end, lane);
  else
    gather_run<W, D, false>(a, stage[wave], first, t_begin, t_end, lane);
}

// ---------------------------------------------------------------- write path

// Up to two (pool, input) pairs written by one launch: the K and V pools of
// one append share the page lists and the launch.
struct ScatterArgs {
  void* pool[2];
  const void* in[2];
  int32_t v_layout[2];
  const int32_t* page_ids;
  const int32_t* seq_page_indptr;
  const int32_t* seq_start;
  const int32_t* seq_count;
  const int64_t* in_token_offset;
  int32_t* error_flag;
  int64_t num_pool_pages;
  int32_t num_seqs;
  int32_t num_kv_heads;
  int32_t n_pairs;
  int32_t seq_blocks;    // workgroups by sequence (partly touched pages)
  int32_t seq_split;     // of them per sequence: 1, or one for each pool
  int32_t tile_blocks;   // workgroups per pool for the whole pages' tiles
};
// Sequences whose tiles one workgroup sums.
constexpr int kTileSeqs = 4096;

// A whole tile (16 tokens of one head): read from the dense input with 16-byte
// loads, transposed in the wave's own LDS buffer and written in stored order,
// 16 bytes per lane.
template <typename W, int D>
struct TileWriter {
  static constexpr int E = 16 / (int)sizeof(W);   // elements per 16-byte vector
  static constexpr int VPT = D / E;               // vectors per token and head
  static constexpr int NV = 16 * VPT / 64;        // vectors per lane for a tile
  static constexpr int KROW = 17;                 // K staging: vector (j, t) at j * KROW + t
  // V staging: the tile in stored order, [D][16] elements, row c held at row
  // c ^ ((c / E) & RMASK): the rows written by one instruction (dims
  // j*E + q of four dim groups j) then fall in different 32-byte bank groups.
  static constexpr int RMASK = 128 / (16 * (int)sizeof(W)) - 1;
  static constexpr int BUF = VPT * KROW > D * 16 / E ? VPT * KROW : D * 16 / E;   // 16-byte vectors

  static __device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // This lane's vectors of a tile: K in input order (dims fastest); V with the
  // token fastest across lanes, so that one instruction's 16 lanes of a dim
  // group fill the 16 slots of one staged row.
  template <bool V>
  static __device__ __forceinline__ void load(const W* src, int64_t row, u32x4_t (&v)[NV], int lane) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int idx = lane + 64 * i;
      const int tok = V ? idx % 16 : idx / VPT, j = V ? idx / 16 : idx % VPT;
      v[i] = *reinterpret_cast<const u32x4_t*>(src + tok * row + j * E);
    }
  }

  template <bool V>
  static __device__ __forceinline__ void store(const u32x4_t (&v)[NV], W* dst, u32x4_t* kst, int lane) {
    if constexpr (!V) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int idx = lane + 64 * i, tok = idx / VPT, j = idx % VPT;
        kst[j * KROW + tok] = v[i];
      }
      wave_sync();
#pragma unroll
      for (int i = 0; i < NV; ++i) {    // K: [D/E][16][E], vector idx = (j, t)
        const int idx = lane + 64 * i;
        *reinterpret_cast<u32x4_t*>(dst + idx * E) = kst[(idx / 16) * KROW + idx % 16];
      }
    } else {
      W* vst = reinterpret_cast<W*>(kst);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int idx = lane + 64 * i, tok = idx % 16, j = idx / 16;
        const int slot = v_token_at_slot(tok);   // the permutation is its own inverse
        const W* e = reinterpret_cast<const W*>(&v[i]);
#pragma unroll
        for (int q = 0; q < E; ++q) vst[((j * E + q) ^ (j & RMASK)) * 16 + slot] = e[q];
      }
      wave_sync();
#pragma unroll
      for (int i = 0; i < NV; ++i) {    // V: [D][16], vector idx = (dim c, slot group)
        const int idx = lane + 64 * i, c = idx / (16 / E), part = idx % (16 / E);
        *reinterpret_cast<u32x4_t*>(dst + idx * E) =
            *reinterpret_cast<const u32x4_t*>(vst + (c ^ ((c / E) & RMASK)) * 16 + part * E);
      }
    }
    wave_sync();
  }
};

// n < 16 (or unaligned) tokens of one page, every head, written straight from
// the input by the whole workgroup: 16-byte vectors for K, whose vector (dim
// group, token) holds one token; single elements of 8-byte loads for V, whose
// slots interleave tokens. Other slots are never written. src: the first of
// the tokens (dense rows of H * D elements); t: its slot in the page.
template <typename W, int D, bool V>
__device__ __forceinline__ void write_part_page(const W* __restrict__ src, W* __restrict__ page, int n, int t, int H) {
  constexpr int E = 16 / (int)sizeof(W);
  constexpr int VPT = D / E;
  constexpr int kUnroll = 4;   // loads in flight per thread before their stores
  const int threads = 256;
  if constexpr (!V) {
    const int per_tok = H * VPT, total = n * per_tok;
    for (int i0 = threadIdx.x; i0 < total; i0 += kUnroll * threads) {
      u32x4_t v[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int idx = i0 + u * threads;
        if (idx < total) v[u] = *reinterpret_cast<const u32x4_t*>(src + (int64_t)idx * E);
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int idx = i0 + u * threads;
        if (idx >= total) break;
        const int tok = idx / per_tok, hv = idx % per_tok;   // hv = head * VPT + dim group
        *reinterpret_cast<u32x4_t*>(page + ((int64_t)hv * 16 + t + tok) * E) = v[u];
      }
    }
  } else {
    typedef W wvec_t __attribute__((ext_vector_type(8 / (int)sizeof(W))));
    constexpr int EV = 8 / (int)sizeof(W);
    const int total = n * (H * D / EV);   // token fastest: neighbouring lanes write one dim row
    for (int i0 = threadIdx.x; i0 < total; i0 += kUnroll * threads) {
      wvec_t v[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int idx = i0 + u * threads;
        if (idx < total) {
          const int tok = idx % n, hc = idx / n;
          v[u] = *reinterpret_cast<const wvec_t*>(src + (int64_t)tok * H * D + hc * EV);
        }
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int idx = i0 + u * threads;
        if (idx >= total) break;
        const int tok = idx % n, hc = idx / n;
        W* dst = page + (int64_t)hc * EV * 16 + v_token_at_slot(t + tok);
#pragma unroll
        for (int q = 0; q < EV; ++q) dst[q * 16] = v[u][q];
      }
    }
  }
}

// Pages touched by tokens start .. start + count - 1 of one sequence: a first
// and a last one that may be partial, and nfull whole pages from slot f0.
struct PageRange {
  int first, last, f0, nfull;
  bool head, tail;   // the first / last page is partly touched (last != first)
  __device__ __forceinline__ PageRange(int start, int count) {
    const int end = start + count;
    first = start / 16;
    last = (end - 1) / 16;
    head = (start & 15) != 0 || end < 16 * (first + 1);
    tail = last > first && (end & 15) != 0;
    f0 = first + (head ? 1 : 0);
    nfull = last - (tail ? 1 : 0) - f0 + 1;
  }
};

// The inverse of the gather: tokens start .. start + count - 1 of each
// sequence are written from the dense input into their (page, head) tiles.
//
// What bounds it: a decode append is a chain of dependent loads (the
// sequence's range and page list, then the page id beside the token) and one
// store; a chunk is an HBM copy. The host knows neither, the ranges being on
// the device, so the grid has two kinds of workgroups:
//  * one for each sequence and pool, or, where they are so many that the chip
//    takes them in several rounds, one for each sequence and both pools,
//    launched first: its partly touched first and last pages, all heads at
//    once. An append costs one short chain, and no workgroup of this kind looks
//    at another sequence.
//  * tile_blocks per pool for the whole pages: each sums the whole-page tiles
//    of all sequences and its waves take equal shares of them, so one long
//    range among many short ones spreads over the chip. Without a whole page it
//    ends after the sum.
// Kernel times against a grid of equal workgroups per sequence (bf16, d 128, 8
// heads, K and V): 240 appends and 16 chunks of 64-512 tokens 66 -> 18 us, 992
// appends and 32 chunks 298 -> 58 us, 32 ragged chunks 27 -> 20 us, 64 appends
// 5.2 -> 4.0 us, 1024 appends 15.2 -> 13.2; 32 aligned chunks of 512 tokens after
// other work 42.3 -> 40.6 us (fp32 74.1 -> 71.6), written again and again 22.0 ->
// 23.5 (fp32 48.7 -> 48.5).
template <typename W, int D, bool V>
__device__ __forceinline__ void scatter_seq(const ScatterArgs& a, int z, int first_seq, int stride) {
  const int H = a.num_kv_heads;
  const int64_t row = (int64_t)H * D;      // input elements per token
  const W* in = static_cast<const W*>(a.in[z]);
  W* pool = static_cast<W*>(a.pool[z]);
  for (int seq = first_seq; seq < a.num_seqs; seq += stride) {
    const int start = a.seq_start[seq], count = a.seq_count[seq];
    const int base = a.seq_page_indptr[seq], next = a.seq_page_indptr[seq + 1];
    const int64_t off = a.in_token_offset[seq];
    if (count <= 0) continue;
    if (start < 0 || (int64_t)start + count > (int64_t)(next - base) * 16) {
      if (z == 0 && threadIdx.x == 0 && a.error_flag) a.error_flag[0] = 1;
      continue;
    }
    const PageRange r(start, count);
#pragma nounroll
    for (int side = 0; side < 2; ++side) {
      if (!(side ? r.tail : r.head)) continue;
      const int pslot = side ? r.last : r.first;
      const int pid = a.page_ids[base + pslot];
      if (pid < 0 || pid >= a.num_pool_pages) {
        if (threadIdx.x == 0 && a.error_flag) a.error_flag[0] = 1;
        continue;
      }
      const int lo = max(start, pslot * 16), hi = min(start + count, pslot * 16 + 16);
      write_part_page<W, D, V>(in + (off + (lo - start)) * row, pool + (int64_t)pid * H * 16 * D, hi - lo,
                               lo - pslot * 16, H);
    }
  }
}

// Inclusive sum over the lanes of a wave: shifts by 1, 2, 4 and 8 inside each
// row of 16 lanes, then the last lane of a row to the next row (rows 1 and 3)
// and lane 31 to the upper half.
__device__ __forceinline__ int wave_inclusive_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return x;
}

// The range of one sequence, and its whole-page tiles (none where the range
// does not fit its page list: its own workgroup flags that).
struct SeqRange {
  int start, base, tiles, f0;
  int64_t off;
  __device__ __forceinline__ SeqRange(const ScatterArgs& a, int seq) {
    start = a.seq_start[seq];
    const int count = a.seq_count[seq];
    base = a.seq_page_indptr[seq];
    const int next = a.seq_page_indptr[seq + 1];
    off = a.in_token_offset[seq];
    const PageRange r(start, count);
    f0 = r.f0;
    const bool fits = count > 0 && start >= 0 && (int64_t)start + count <= (int64_t)(next - base) * 16;
    tiles = fits ? r.nfull * a.num_kv_heads : 0;
  }
};

// Whole pages: the tiles of up to kTileSeqs sequences, shared equally by the
// waves. Up to 64 sequences every wave sums by itself, one sequence per lane,
// and finds its tiles in the lanes' registers, without a barrier or a second
// look at the metadata (32 chunks of 512 tokens, K and V: 30.6 us; by the
// workgroup 33.5); it takes every turns-th tile, so that neighbouring waves
// move neighbouring heads of one page (32 fp32 chunks of 512 tokens after other
// work: 83 us with contiguous runs, 72 so). More are summed by the workgroup,
// thread i those of sequences i, i + 256, ..., in LDS (1024 appends: 18 us,
// against 22.7 when every wave sums all of them), and a wave takes a contiguous
// run. A sequence with fewer than 16 new tokens has no whole page: only its
// count is read.
template <typename W, int D, bool V>
__device__ __forceinline__ void scatter_tiles(const ScatterArgs& a, int z, int s0, int n_seqs, int turn, int turns,
                                              u32x4_t* stage, int (&sums)[260], int wave, int lane) {
  const int H = a.num_kv_heads;
  const int64_t row = (int64_t)H * D;
  const bool by_wave = n_seqs <= 64;
  int mine = 0, l_start = 0, l_base = 0, l_f0 = 0, upto, total;
  int64_t l_off = 0;
  if (by_wave) {
    if (lane < n_seqs) {
      const SeqRange r(a, s0 + lane);
      mine = r.tiles;
      l_start = r.start;
      l_base = r.base;
      l_f0 = r.f0;
      l_off = r.off;
    }
    if (!__any(mine > 0)) return;
    upto = wave_inclusive_sum(mine);
    total = __builtin_amdgcn_readlane(upto, 63);
  } else {
    constexpr int kAhead = 4;   // counts in flight per thread
    for (int i0 = threadIdx.x; i0 < n_seqs; i0 += kAhead * 256) {
      int count[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) count[u] = i0 + 256 * u < n_seqs ? a.seq_count[s0 + i0 + 256 * u] : 0;
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (count[u] >= 16) mine += SeqRange(a, s0 + i0 + 256 * u).tiles;
    }
    if (!__syncthreads_or(mine)) return;
    upto = wave_inclusive_sum(mine);
    if (lane == 63) sums[256 + wave] = upto;
    __syncthreads();
    total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      upto += w < wave ? sums[256 + w] : 0;
      total += sums[256 + w];
    }
    sums[threadIdx.x] = upto;
    __syncthreads();
  }
  const int per = (int)(((int64_t)total + turns - 1) / turns);
  int k = by_wave ? turn : (int)min((int64_t)total, (int64_t)turn * per);
  const int k_end = by_wave ? total : (int)min((int64_t)total, (int64_t)k + per);
  while (k < k_end) {
    int t, n, base, f0;
    int64_t at;   // dense row of the sequence's token 0
    if (by_wave) {
      const int lo = __popcll(__ballot(upto <= k));   // the lane whose sequence holds tile k
      t = k - (lo ? __builtin_amdgcn_readlane(upto, lo - 1) : 0);
      n = __builtin_amdgcn_readlane(mine, lo);
      base = __builtin_amdgcn_readlane(l_base, lo);
      f0 = __builtin_amdgcn_readlane(l_f0, lo);
      at = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(l_off >> 32), lo) << 32) |
                     (uint32_t)__builtin_amdgcn_readlane((int)l_off, lo)) -
           __builtin_amdgcn_readlane(l_start, lo);
    } else {
      int lo = 0;   // the thread whose sequences hold tile k
#pragma unroll
      for (int j = 0; j < 4; ++j) lo += __popcll(__ballot(sums[64 * j + lane] <= k));
      t = k - (lo ? sums[lo - 1] : 0);
      t = __builtin_amdgcn_readfirstlane(t);
      int seq = s0 + lo;
      SeqRange r(a, seq);
      while (t >= r.tiles) {
        t -= r.tiles;
        seq += 256;
        r = SeqRange(a, seq);
      }
      n = r.tiles;
      base = r.base;
      f0 = r.f0;
      at = r.off - r.start;
    }
    // tiles t .. t_end - 1 of one sequence, heads innermost
    const int t_end = by_wave ? t + 1 : min(n, t + (k_end - k));
    k += by_wave ? turns : t_end - t;
    const W* in = static_cast<const W*>(a.in[z]) + at * row;
#pragma nounroll
    for (; t < t_end; ++t) {
      const int pslot = f0 + t / H, h = t % H;
      const int pid = a.page_ids[base + pslot];
      u32x4_t v[TileWriter<W, D>::NV];
      TileWriter<W, D>::template load<V>(in + (int64_t)pslot * 16 * row + (int64_t)h * D, row, v, lane);
      if (pid < 0 || pid >= a.num_pool_pages) {
        if (lane == 0 && a.error_flag) a.error_flag[0] = 1;
        continue;
      }
      TileWriter<W, D>::template store<V>(v, static_cast<W*>(a.pool[z]) + ((int64_t)pid * H + h) * 16 * D, stage, lane);
    }
  }
}

template <typename W, int D>
__global__ __launch_bounds__(256) void scatter_kernel(ScatterArgs a) {
  __shared__ u32x4_t stage[4][TileWriter<W, D>::BUF];
  __shared__ int sums[260];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  if ((int)blockIdx.x < a.seq_blocks) {
    // (z, then the following ones up to z_end: one pool, or all)
    int z = (int)blockIdx.x % a.seq_split;
    const int z_end = z + a.n_pairs / a.seq_split;
    const int seq = (int)blockIdx.x / a.seq_split, stride = a.seq_blocks / a.seq_split;
#pragma nounroll
    for (; z < z_end; ++z) {
      if (a.v_layout[z]) scatter_seq<W, D, true>(a, z, seq, stride);
      else scatter_seq<W, D, false>(a, z, seq, stride);
    }
    return;
  }
  const int z = ((int)blockIdx.x - a.seq_blocks) % a.n_pairs;
  const int tb = ((int)blockIdx.x - a.seq_blocks) / a.n_pairs;   // of a.tile_blocks for this pool
  const int groups = (a.num_seqs + kTileSeqs - 1) / kTileSeqs;
  for (int g = tb % groups; g < groups; g += a.tile_blocks) {
    // the workgroups of this group, and this one's turn among them
    const int of = a.tile_blocks >= groups ? (a.tile_blocks - g + groups - 1) / groups : 1;
    const int s0 = g * kTileSeqs, n = min(a.num_seqs - s0, kTileSeqs);
    const int turn = tb / groups * 4 + wave;
    if (a.v_layout[z]) scatter_tiles<W, D, true>(a, z, s0, n, turn, of * 4, stage[wave], sums, wave, lane);
    else scatter_tiles<W, D, false>(a, z, s0, n, turn, of * 4, stage[wave], sums, wave, lane);
    __syncthreads();   // the sums are overwritten for the next group
  }
}

struct PageCopyArgs {
  void* pool;
  const int32_t* src_pages;
  const int32_t* dst_pages;
  int32_t* error_flag;
  int64_t num_pool_pages;
  int64_t page_vecs;   // 16-byte units of one page (all heads)
  int32_t num_pages;
};

// Copy whole pages (every head) of one pool, 16 bytes per lane, grid-stride
// over (page, unit). Pages with an id out of range are skipped and flagged.
__global__ __launch_bounds__(256) void page_copy_kernel(PageCopyArgs a) {
  const int64_t total = (int64_t)a.num_pages * a.page_vecs;
  u32x4_t* pool = static_cast<u32x4_t*>(a.pool);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = i / a.page_vecs, u = i - k * a.page_vecs;
    const int src = a.src_pages[k], dst = a.dst_pages[k];
    if (src < 0 || src >= a.num_pool_pages || dst < 0 || dst >= a.num_pool_pages) {
      if (u == 0 && a.error_flag) a.error_flag[0] = 1;
      continue;
    }
    pool[dst * a.page_vecs + u] = pool[src * a.page_vecs + u];
  }
}

// ---------------------------------------------------------------- host side

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

halo_status_t hip_check(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HALO_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
  return HALO_OK;
}

}  // namespace

extern "C" halo_status_t halo_kv_page_gather(const void* pool, const halo_attn_params_t* params,
                                             halo_pool_kind_t pool_kind, const int32_t* page_ids,
                                             const int32_t* seq_page_indptr, const int32_t* seq_len,
                                             const int64_t* out_token_offset, int32_t num_seqs, void* out,
                                             int32_t* error_flag, void* stream) {
  clear_error();
  if (!params) return fail(HALO_ERR_INVALID_ARGUMENT, "params must not be NULL");
  if (num_seqs < 0) return fail(HALO_ERR_INVALID_ARGUMENT, "num_seqs must be >= 0");
  if (num_seqs == 0) return HALO_OK;
  if (!pool || !page_ids || !seq_page_indptr || !seq_len || !out_token_offset || !out)
    return fail(HALO_ERR_INVALID_ARGUMENT, "pool, page_ids, seq_page_indptr, seq_len, out_token_offset, out "
                                           "must not be NULL");
  if (params->head_dim != 64 && params->head_dim != 128)
    return fail(HALO_ERR_UNSUPPORTED, "head_dim must be 64 or 128");
  if (params->page_size != 16) return fail(HALO_ERR_UNSUPPORTED, "page_size must be 16");
  if (params->num_kv_heads < 1) return fail(HALO_ERR_INVALID_ARGUMENT, "num_kv_heads must be >= 1");
  if (pool_kind != HALO_POOL_K && pool_kind != HALO_POOL_V)
    return fail(HALO_ERR_INVALID_ARGUMENT, "pool_kind must be HALO_POOL_K or HALO_POOL_V");
  GatherArgs g{pool, page_ids, seq_page_indptr, seq_len, out_token_offset, out, error_flag,
               params->num_pool_pages, num_seqs, params->num_kv_heads, params->head_dim,
               pool_kind == HALO_POOL_V ? 1 : 0};
  hipStream_t st = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  if (!aligned16(pool) || !aligned16(out))
    return fail(HALO_ERR_INVALID_ARGUMENT, "pool and out must be 16-byte aligned");
  // 2048 workgroups of four waves; each wave takes an equal run of tiles.
  const dim3 grid(2048);
  const bool d128 = params->head_dim == 128;
  if (params->kv_dtype == HALO_BF16) {
    if (d128) hipLaunchKernelGGL((gather_kernel<uint16_t, 128>), grid, dim3(256), 0, st, g);
    else hipLaunchKernelGGL((gather_kernel<uint16_t, 64>), grid, dim3(256), 0, st, g);
  } else if (params->kv_dtype == HALO_F32) {
    if (d128) hipLaunchKernelGGL((gather_kernel<uint32_t, 128>), grid, dim3(256), 0, st, g);
    else hipLaunchKernelGGL((gather_kernel<uint32_t, 64>), grid, dim3(256), 0, st, g);
  } else {
    return fail(HALO_ERR_UNSUPPORTED, "kv_dtype must be HALO_F32 or HALO_BF16");
  }
  return hip_check("gather launch");
}

namespace {

// Shared checks and launch of the scatter entry points (n_pairs = 1 or 2).
halo_status_t launch_scatter(const halo_attn_params_t* params, ScatterArgs g, int n_pairs, void* stream) {
  if (params->head_dim != 64 && params->head_dim != 128)
    return fail(HALO_ERR_UNSUPPORTED, "head_dim must be 64 or 128");
  if (params->page_size != 16) return fail(HALO_ERR_UNSUPPORTED, "page_size must be 16");
  if (params->num_kv_heads < 1) return fail(HALO_ERR_INVALID_ARGUMENT, "num_kv_heads must be >= 1");
  if (params->kv_dtype != HALO_BF16 && params->kv_dtype != HALO_F32)
    return fail(HALO_ERR_UNSUPPORTED, "kv_dtype must be HALO_F32 or HALO_BF16");
  for (int z = 0; z < n_pairs; ++z)
    if (!aligned16(g.pool[z]) || !aligned16(g.in[z]))
      return fail(HALO_ERR_INVALID_ARGUMENT, "pools and inputs must be 16-byte aligned");
  g.num_pool_pages = params->num_pool_pages;
  g.num_kv_heads = params->num_kv_heads;
  g.n_pairs = n_pairs;
  hipStream_t st = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  // A workgroup per sequence and pool, or for both pools from 257 sequences on
  // (512 appends 9.8 -> 8.6 us, 1024 15.9 -> 13.2; 128 4.9 -> 5.0, 64 4.0 -> 4.5;
  // 992 appends and 32 chunks, whose last pages then come one after the other,
  // 39.6 -> 42.8), grid-stride past 65536 sequences, and
  // 512 of four waves for the whole pages: with 1024 a batch of appends waits
  // for them (64 sequences: 4.3 -> 4.7 us), with 256 a chunk's copies have
  // too few loads in flight (32 chunks of 512 tokens: 30.8 -> 39 us).
  constexpr int kTileBlocks = 512;
  g.seq_split = g.num_seqs > 256 ? 1 : n_pairs;
  g.seq_blocks = std::min(g.num_seqs, 65536) * g.seq_split;
  g.tile_blocks = kTileBlocks / n_pairs;
  const dim3 grid(g.seq_blocks + kTileBlocks);
  const bool d128 = params->head_dim == 128;
  if (params->kv_dtype == HALO_BF16) {
    if (d128) hipLaunchKernelGGL((scatter_kernel<uint16_t, 128>), grid, dim3(256), 0, st, g);
    else hipLaunchKernelGGL((scatter_kernel<uint16_t, 64>), grid, dim3(256), 0, st, g);
  } else {
    if (d128) hipLaunchKernelGGL((scatter_kernel<uint32_t, 128>), grid, dim3(256), 0, st, g);
    else hipLaunchKernelGGL((scatter_kernel<uint32_t, 64>), grid, dim3(256), 0, st, g);
  }
  return hip_check("scatter launch");
}

}  // namespace

extern "C" halo_status_t halo_kv_page_scatter(void* pool, const halo_attn_params_t* params,
                                              halo_pool_kind_t pool_kind, const int32_t* page_ids,
                                              const int32_t* seq_page_indptr, const int32_t* seq_start,
                                              const int32_t* seq_count, const int64_t* in_token_offset,
                                              int32_t num_seqs, const void* in, int32_t* error_flag,
                                              void* stream) {
  clear_error();
  if (!params) return fail(HALO_ERR_INVALID_ARGUMENT, "params must not be NULL");
  if (num_seqs < 0) return fail(HALO_ERR_INVALID_ARGUMENT, "num_seqs must be >= 0");
  if (num_seqs == 0) return HALO_OK;
  if (!pool || !page_ids || !seq_page_indptr || !seq_start || !seq_count || !in_token_offset || !in)
    return fail(HALO_ERR_INVALID_ARGUMENT, "pool, page_ids, seq_page_indptr, seq_start, seq_count, "
                                           "in_token_offset, in must not be NULL");
  if (pool_kind != HALO_POOL_K && pool_kind != HALO_POOL_V)
    return fail(HALO_ERR_INVALID_ARGUMENT, "pool_kind must be HALO_POOL_K or HALO_POOL_V");
  ScatterArgs g{};
  g.pool[0] = pool;
  g.in[0] = in;
  g.v_layout[0] = pool_kind == HALO_POOL_V ? 1 : 0;
  g.page_ids = page_ids;
  g.seq_page_indptr = seq_page_indptr;
  g.seq_start = seq_start;
  g.seq_count = seq_count;
  g.in_token_offset = in_token_offset;
  g.error_flag = error_flag;
  g.num_seqs = num_seqs;
  return launch_scatter(params, g, 1, stream);
}

extern "C" halo_status_t halo_kv_page_scatter_kv(void* k_pool, void* v_pool, const halo_attn_params_t* params,
                                                 const int32_t* page_ids, const int32_t* seq_page_indptr,
                                                 const int32_t* seq_start, const int32_t* seq_count,
                                                 const int64_t* in_token_offset, int32_t num_seqs,
                                                 const void* k_in, const void* v_in, int32_t* error_flag,
                                                 void* stream) {
  clear_error();
  if (!params) return fail(HALO_ERR_INVALID_ARGUMENT, "params must not be NULL");
  if (num_seqs < 0) return fail(HALO_ERR_INVALID_ARGUMENT, "num_seqs must be >= 0");
  if (num_seqs == 0) return HALO_OK;
  if (!k_pool || !v_pool || !page_ids || !seq_page_indptr || !seq_start || !seq_count || !in_token_offset ||
      !k_in || !v_in)
    return fail(HALO_ERR_INVALID_ARGUMENT, "k_pool, v_pool, page_ids, seq_page_indptr, seq_start, seq_count, "
                                           "in_token_offset, k_in, v_in must not be NULL");
  ScatterArgs g{};
  g.pool[0] = k_pool;
  g.pool[1] = v_pool;
  g.in[0] = k_in;
  g.in[1] = v_in;
  g.v_layout[0] = 0;
  g.v_layout[1] = 1;
  g.page_ids = page_ids;
  g.seq_page_indptr = seq_page_indptr;
  g.seq_start = seq_start;
  g.seq_count = seq_count;
  g.in_token_offset = in_token_offset;
  g.error_flag = error_flag;
  g.num_seqs = num_seqs;
  return launch_scatter(params, g, 2, stream);
}

extern "C" halo_status_t halo_kv_page_copy(void* pool, const halo_attn_params_t* params,
                                           const int32_t* src_pages, const int32_t* dst_pages,
                                           int32_t num_pages, int32_t* error_flag, void* stream) {
  clear_error();
  if (!params) return fail(HALO_ERR_INVALID_ARGUMENT, "params must not be NULL");
  if (num_pages < 0) return fail(HALO_ERR_INVALID_ARGUMENT, "num_pages must be >= 0");
  if (num_pages == 0) return HALO_OK;
  if (!pool || !src_pages || !dst_pages)
    return fail(HALO_ERR_INVALID_ARGUMENT, "pool, src_pages, dst_pages must not be NULL");
  if (params->head_dim != 64 && params->head_dim != 128)
    return fail(HALO_ERR_UNSUPPORTED, "head_dim must be 64 or 128");
  if (params->page_size != 16) return fail(HALO_ERR_UNSUPPORTED, "page_size must be 16");
  if (params->num_kv_heads < 1) return fail(HALO_ERR_INVALID_ARGUMENT, "num_kv_heads must be >= 1");
  int elt;
  if (params->kv_dtype == HALO_BF16) elt = 2;
  else if (params->kv_dtype == HALO_F32) elt = 4;
  else return fail(HALO_ERR_UNSUPPORTED, "kv_dtype must be HALO_F32 or HALO_BF16");
  if (!aligned16(pool)) return fail(HALO_ERR_INVALID_ARGUMENT, "pool must be 16-byte aligned");
  const int64_t page_bytes = (int64_t)params->num_kv_heads * 16 * params->head_dim * elt;
  PageCopyArgs g{pool, src_pages, dst_pages, error_flag, params->num_pool_pages, page_bytes / 16, num_pages};
  hipStream_t st = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  const int64_t want = ((int64_t)num_pages * g.page_vecs + 255) / 256;
  const int blocks = (int)std::min<int64_t>(std::max<int64_t>(want, 1), 4096);
  hipLaunchKernelGGL(page_copy_kernel, dim3(blocks), dim3(256), 0, st, g);
  return hip_check("page copy launch");
}
