// The word-topic counts by partition of the cells (gfx950).
//
// Counted in token order, the word table takes one device-wide atomic per
// distinct cell of every chunk of tokens, executed on the memory side (about
// 30 G/s on MI355X: 12.3M of them, 0.4 ms, for the 16.8M-token corpus at K =
// 1024, though the draw fills 1.7M cells).  Here every cell belongs to one
// workgroup, which counts it in LDS and stores it once:
//
//   split   each workgroup takes a chunk of tokens, sorts their cells by bucket
//           (the top bits of the cell index times an odd constant, so that the
//           frequent words' cells spread evenly) in LDS, and writes them out
//           as one contiguous run with the buckets' offsets in it; it also
//           clears its share of the table;
//   cells   workgroup p takes bucket p's piece of every chunk's run and sums
//           it in an LDS hash table, then stores each cell's count.
//
// An entry of a run is the cell's hash without its bucket bits, and in their
// place the number of the chunk's tokens it stands for, less one: pieces much
// longer than the mean hold a frequent word's favourite topics, and their equal
// entries are merged, 64 at a time, so that one cell does not hold up its
// bucket's workgroup.
// The runs and offsets need 4 bytes per token and 2 per chunk and bucket.
// They lie in the document table, which is written after them (its rows whole
// by count_docs_kernel, or cleared and added to by count_doc_ids_kernel): the
// call overwrites both tables in any case, so it needs no workspace.
//
// Measured on MI355X at 16.8M tokens, K = 1024, V = 100,000: split 122 us (600
// MB read and written, 5 TB/s: the copy rate), cells 111 us: 52 for reading the
// pieces (64 bytes each on average), 20 for the table, 40 for the 1.7M single
// stores.
//
// A bucket's table holds 8,192 cells, 2.1M or 4.2M in all.  Where the topics
// fill more (a sampler's first sweeps over a large corpus: near-uniform topics),
// tokens that find no slot are added in memory.  Their walk over 32 taken slots
// cost more than that addition: once one token has been through it, the others
// of the bucket try four.  16.8M uniform topics (6.6M cells) 692 -> 590 us, 50M
// (12.4M cells) 1,553 -> 1,058, 7.9M over 256 buckets (2.8M cells) 315 -> 209; over
// the word index, without the partition, these took 632, 1,325 and 314.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "config.hpp"
#include "counts.hpp"

namespace LDA_NS {
namespace {

constexpr int kSplitThreads = 512;
constexpr int kCellThreads = 1024;
constexpr int kCellSlots = 8192;        // hash slots of a bucket (64 KiB of LDS)
constexpr int kMerges = 4;              // cells merged per 64 entries of a long piece
constexpr int kCellProbes = 32;         // probes before a token goes to memory
constexpr int kFullProbes = 4;          // ... once the table is full (a token has)
constexpr uint32_t kCellMul = 2654435761u;  // odd: a bijection mod 2^32

// Inverse of an odd number mod 2^32 (Newton: each step doubles the bits).
constexpr uint32_t inverse32(uint32_t a) {
  uint32_t x = a;
  for (int i = 0; i < 5; ++i) x *= 2u - a * x;
  return x;
}
static_assert(kCellMul * inverse32(kCellMul) == 1u, "the inverse of kCellMul");

// Chunks of kSplitThreads PER tokens, 2^BITS buckets.
template <int PER, int BITS>
struct CellSplit {
  static constexpr int kChunk = kSplitThreads * PER;
  static constexpr int kBuckets = 1 << BITS;
  // the mean length of a piece, and the lanes of `cells` that share one
  static constexpr int kPiece = kChunk / kBuckets;
  static constexpr int kLanes = 2 * kPiece;
  // pieces longer than this are merged; the bits of an entry's cell
  static constexpr uint32_t kLong = kLanes;
  static constexpr uint32_t kLow = (1u << (32 - BITS)) - 1u;
  static_assert(BITS >= 6, "an entry counts up to 64 tokens");
  static_assert(kBuckets <= kSplitThreads && kBuckets % 64 == 0 && kChunk < (1 << 16), "offsets are 16 bits wide");
  static_assert(kLanes >= 8 && kLanes <= 64 && (kLanes & (kLanes - 1)) == 0, "lanes per piece");
  static int64_t chunks(int64_t N) { return (N + kChunk - 1) / kChunk; }
  // scratch in bytes: the runs (whole chunks but for the last), the offsets
  static int64_t bytes(int64_t N) { return 4 * N + 2 * chunks(N) * (kBuckets + 1); }
};

// doc_id null: documents given as offsets (every token has one).
template <int PER, int BITS>
__global__ __launch_bounds__(kSplitThreads) void count_split_kernel(
    const int32_t *__restrict__ doc_id, const int32_t *__restrict__ word_id,
    const int32_t *__restrict__ z, int64_t N, int32_t M, int32_t V, int32_t K,
    uint32_t *__restrict__ runs, uint16_t *__restrict__ offs, int32_t *__restrict__ nwk,
    int64_t cells) {
  using S = CellSplit<PER, BITS>;
  __shared__ uint32_t sorted[S::kChunk];
  __shared__ uint8_t times[S::kChunk];      // merged pieces: tokens per entry
  __shared__ uint32_t start[S::kBuckets];
  __shared__ uint32_t len[S::kBuckets];     // entries, once merged
  __shared__ uint32_t out[S::kBuckets];     // where they go in the run
  __shared__ uint32_t part[kSplitThreads / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (t < S::kBuckets) start[t] = 0;
  const int64_t c0 = (int64_t)blockIdx.x * S::kChunk;
  uint32_t h[PER];
  bool ok[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int64_t n = c0 + (int64_t)i * kSplitThreads + t;
    int32_t d = 0, w = -1, k = -1;
    if (n < N) {
      if (doc_id) d = doc_id[n];
      w = word_id[n];
      k = z[n];
    }
    ok[i] = (uint32_t)d < (uint32_t)M && (uint32_t)w < (uint32_t)V && (uint32_t)k < (uint32_t)K;
    h[i] = ((uint32_t)w * (uint32_t)K + (uint32_t)k) * kCellMul;
  }
  {
    // this workgroup's share of the table, cleared while the loads are out:
    // 16-byte stores at 16-byte boundaries, the ends by single stores
    const int64_t head = (int64_t)((16u - (reinterpret_cast<uintptr_t>(nwk) & 15u)) & 15u) / 4;
    const int64_t h0 = head < cells ? head : cells;
    const int64_t quads = (cells - h0) / 4, tail0 = h0 + 4 * quads;
    const int64_t per = (quads + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * per, hi = lo + per < quads ? lo + per : quads;
    int4 *body = reinterpret_cast<int4 *>(nwk + h0);
    for (int64_t i = lo + t; i < hi; i += kSplitThreads) body[i] = int4{0, 0, 0, 0};
    if (blockIdx.x == 0) {
      if (t < h0) nwk[t] = 0;
      if (t < cells - tail0) nwk[tail0 + t] = 0;
    }
  }
  __syncthreads();
  uint32_t rank[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i)
    rank[i] = ok[i] ? atomicAdd(&start[h[i] >> (32 - BITS)], 1u) : 0u;
  __syncthreads();
  // exclusive scan of one value per thread, and their total
  const auto scan = [&](uint32_t v, uint32_t &total) {
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t up = __shfl_up(incl, d);
      if (lane >= d) incl += up;
    }
    if (lane == 63) part[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < kSplitThreads / 64; ++i) {
      const uint32_t p = part[i];
      before += i < wave ? p : 0u;
      total += p;
    }
    __syncthreads();
    return before + incl - v;
  };
  uint32_t tokens;
  const uint32_t count = t < S::kBuckets ? start[t] : 0u;
  const uint32_t at = scan(count, tokens);
  if (t < S::kBuckets) {
    start[t] = at;
    len[t] = count;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (ok[i]) sorted[start[h[i] >> (32 - BITS)] + rank[i]] = h[i];
  __syncthreads();
  // merge the long pieces, one wavefront each
  for (int b0 = wave * 64; b0 < S::kBuckets; b0 += kSplitThreads) {
    uint64_t longs = __builtin_amdgcn_ballot_w64(len[b0 + lane] > S::kLong);
    while (longs) {
      const int b = b0 + __builtin_ctzll(longs);
      longs &= longs - 1;
      const uint32_t from = start[b], n = len[b];
      uint32_t to = from;
      for (uint32_t i = 0; i < n; i += 64) {
        const bool in = i + lane < n;
        const uint32_t e = in ? sorted[from + i + lane] : 0u;
        // the cells of up to kMerges of the first entries, merged if repeated
        uint64_t rest = __builtin_amdgcn_ballot_w64(in), left = rest;
        for (int m = 0; m < kMerges && left; ++m) {
          const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)e, __builtin_ctzll(left));
          const uint64_t same = __builtin_amdgcn_ballot_w64(in && e == first);
          left &= ~same;
          if (same & (same - 1)) {
            rest &= ~same;
            if (lane == 0) {
              sorted[to] = first;
              times[to] = (uint8_t)(__builtin_popcountll(same) - 1);
            }
            ++to;
          }
        }
        // the other entries as they are
        if ((rest >> lane) & 1) {
          const uint32_t j = to + (uint32_t)__builtin_popcountll(rest & ((1ull << lane) - 1ull));
          sorted[j] = e;
          times[j] = 0;
        }
        to += (uint32_t)__builtin_popcountll(rest);
      }
      if (lane == 0) len[b] = to - from;
    }
  }
  __syncthreads();
  uint32_t total;
  const uint32_t now = t < S::kBuckets ? len[t] : 0u;
  const uint32_t put = scan(now, total);
  uint16_t *mine = offs + (int64_t)blockIdx.x * (S::kBuckets + 1);
  if (t < S::kBuckets) {
    out[t] = put;
    mine[t] = (uint16_t)put;
  }
  if (t == 0) mine[S::kBuckets] = (uint16_t)total;
  __syncthreads();
  for (uint32_t i = t; i < tokens; i += kSplitThreads) {
    const uint32_t e = sorted[i], b = e >> (32 - BITS), j = i - start[b];
    // (a merged piece's places past its entries still hold the old ones)
    const bool was_long = (b + 1 < S::kBuckets ? start[b + 1] : tokens) - start[b] > S::kLong;
    if (j < len[b])
      runs[c0 + out[b] + j] = (e & S::kLow) | (was_long ? (uint32_t)times[i] << (32 - BITS) : 0u);
  }
}

// `n` more tokens of the cell with low hash bits `low`: counted in the LDS
// table from `slot` on, or, where none of PROBES slots takes it, in memory
// (true).
template <int PROBES>
__device__ __forceinline__ bool cell_spills(uint32_t *keys, uint32_t *cnt, uint32_t low,
                                            uint32_t slot, uint32_t n) {
  for (int probe = 0; probe < PROBES; ++probe) {
    uint32_t k = __hip_atomic_load(&keys[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (k == kCountEmpty) k = atomicCAS(&keys[slot], kCountEmpty, low);
    if (k == kCountEmpty || k == low) {
      atomicAdd(&cnt[slot], n);
      return false;
    }
    slot = (slot + 1) & (kCellSlots - 1);
  }
  return true;
}

// Workgroup p sums bucket p of every chunk and stores its cells (adds them if
// some of its tokens had to be counted in memory: a cell may then be in both).
// (8 wavefronts per SIMD, so that two such workgroups share a CU: 107 us against
// 140 without the attribute, whose scalar registers allowed one.)
template <int PER, int BITS>
__global__ __launch_bounds__(kCellThreads) __attribute__((amdgpu_waves_per_eu(8)))
void count_cells_kernel(
    const uint32_t *__restrict__ runs, const uint16_t *__restrict__ offs, uint32_t chunks,
    int32_t *__restrict__ nwk) {
  using S = CellSplit<PER, BITS>;
  constexpr int kAhead = 4;                           // pieces in flight per lane
  constexpr int kGroups = kCellThreads / S::kLanes;   // pieces side by side
  constexpr int kSlotShift = 32 - BITS - 13;
  static_assert(kCellSlots == 1 << 13 && kSlotShift >= 0, "slot: the top 13 low bits");
  __shared__ uint32_t keys[kCellSlots];
  __shared__ uint32_t cnt[kCellSlots];
  __shared__ uint32_t spilled;
  const int t = threadIdx.x;
  const int lane = t & (S::kLanes - 1), group = t / S::kLanes;
  const uint32_t p = blockIdx.x;
  for (int s = t; s < kCellSlots; s += kCellThreads) {
    keys[s] = kCountEmpty;
    cnt[s] = 0;
  }
  if (t == 0) spilled = 0;
  __syncthreads();
  const auto cell_of = [&](uint32_t low) {
    return (size_t)(((p << (32 - BITS)) | low) * inverse32(kCellMul));
  };
  // (run positions and offsets are below 2^32: N < 2^31)
  const auto pieces = [&](uint32_t g0, auto full) {
    const auto add = [&](uint32_t e) {
      const uint32_t low = e & S::kLow, n = (e >> (32 - BITS)) + 1u;
      if (cell_spills<full.value ? kFullProbes : kCellProbes>(keys, cnt, low, low >> kSlotShift,
                                                              n)) {
        atomicAdd(&nwk[cell_of(low)], (int32_t)n);
        if (!full.value) spilled = 1;
      }
    };
    uint32_t from[kAhead], left[kAhead], e[kAhead], seen[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const uint32_t g = g0 + (uint32_t)u * kGroups + group;
      from[u] = left[u] = 0;
      if (g < chunks) {
        const uint16_t *o = offs + g * (uint32_t)(S::kBuckets + 1) + p;
        const uint32_t lo = o[0], hi = o[1];
        from[u] = g * (uint32_t)S::kChunk + lo + lane;
        left[u] = hi > lo + lane ? hi - lo - lane : 0u;  // entries from this lane's first on
      }
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) e[u] = left[u] ? runs[from[u]] : 0u;
    // Most tokens' cells are in the table already, at their first slot: those
    // slots are read together (one LDS round trip), the rest taken one by one.
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      seen[u] = __hip_atomic_load(&keys[(e[u] & S::kLow) >> kSlotShift], __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (left[u]) {
        const uint32_t low = e[u] & S::kLow;
        if (seen[u] == low)
          atomicAdd(&cnt[low >> kSlotShift], (e[u] >> (32 - BITS)) + 1u);
        else
          add(e[u]);
        // (a piece longer than its lanes)
        for (uint32_t i = S::kLanes; i < left[u]; i += S::kLanes) add(runs[from[u] + i]);
      }
  };
  const auto overflows = [&] {
    return __hip_atomic_load(&spilled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0;
  };
  uint32_t g0 = 0;
  for (; g0 < chunks && !overflows(); g0 += kGroups * kAhead) pieces(g0, std::false_type());
  for (; g0 < chunks; g0 += kGroups * kAhead) pieces(g0, std::true_type());
  __syncthreads();
  const bool sum = spilled != 0;
  for (int s = t; s < kCellSlots; s += kCellThreads) {
    const uint32_t low = keys[s];
    if (low != kCountEmpty) {
      const size_t cell = cell_of(low);
      if (sum)
        atomicAdd(&nwk[cell], (int32_t)cnt[s]);
      else
        nwk[cell] = (int32_t)cnt[s];
    }
  }
}

}  // namespace
}  // namespace LDA_NS
