// RR collection layout and greedy maximum coverage on gfx950.
//
// Compaction (scan of set sizes, then a gather) turns the node pool written by
// the samplers into a flat CSR of sets in set-id order.  A counting sort of
// that CSR (histogram, scan, scatter) builds the node -> sets inverted index;
// its histogram is also the initial coverage count of every node.  The greedy
// of Algorithm 1 then runs on the device without host round
// trips: per step one argmax kernel packs (count, ~id) into a 64-bit key so
// that a single atomicMax selects the largest count with ties to the lowest
// id, and one cover kernel marks the chosen node's uncovered sets and
// decrements the counts of their members.
#include <string.h>

#include <algorithm>
#include <mutex>

#include "engine.hpp"

namespace tim {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 16;
constexpr int kTile = kThreads * kItems;

__device__ __forceinline__ unsigned long long block_sum_u64(unsigned long long x, unsigned long long* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  if (lane == 0) red[wv] = x;
  __syncthreads();
  unsigned long long t = 0;
  for (int w = 0; w < kThreads / 64; ++w) t += red[w];
  __syncthreads();
  return t;
}

// Exclusive block scan of 64-bit values (T threads, red[T / 64]).
template <int T = kThreads>
__device__ __forceinline__ unsigned long long block_excl_scan(unsigned long long x, unsigned long long* red,
                                                              unsigned long long* total) {
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  unsigned long long incl = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) red[wv] = incl;
  __syncthreads();
  unsigned long long carry = 0, all = 0;
  for (int w = 0; w < T / 64; ++w) {
    if (w < wv) carry += red[w];
    all += red[w];
  }
  __syncthreads();
  *total = all;
  return carry + incl - x;
}

__global__ __launch_bounds__(kThreads) void scan_tile_sums(const uint32_t* in, uint64_t len,
                                                           unsigned long long* tile_sums) {
  __shared__ unsigned long long red[kThreads / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kTile;
  unsigned long long s = 0;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const uint64_t j = base + (uint64_t)i * kThreads + threadIdx.x;
    if (j < len) s += in[j];
  }
  s = block_sum_u64(s, red);
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = s;
}

__global__ __launch_bounds__(kThreads) void scan_tile_offsets(unsigned long long* tile_sums, uint64_t ntiles,
                                                              int64_t* out, uint64_t len) {
  __shared__ unsigned long long red[kThreads / 64];
  unsigned long long carry = 0;
  for (uint64_t base = 0; base < ntiles; base += kThreads) {
    const uint64_t j = base + threadIdx.x;
    const unsigned long long x = j < ntiles ? tile_sums[j] : 0ull;
    unsigned long long total;
    const unsigned long long ex = block_excl_scan(x, red, &total);
    if (j < ntiles) tile_sums[j] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) out[len] = (int64_t)carry;
}

__global__ __launch_bounds__(kThreads) void scan_apply(const uint32_t* in, uint64_t len,
                                                       const unsigned long long* tile_off, int64_t* out) {
  __shared__ unsigned long long red[kThreads / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kTile + (uint64_t)threadIdx.x * kItems;
  uint32_t v[kItems];
  unsigned long long s = 0;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    v[i] = (base + i < len) ? in[base + i] : 0u;
    s += v[i];
  }
  unsigned long long total;
  unsigned long long run = tile_off[blockIdx.x] + block_excl_scan(s, red, &total);
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    if (base + i < len) out[base + i] = (int64_t)run;
    run += v[i];
  }
}

__global__ void compact_kernel(const int32_t* pool, const uint64_t* set_start, const uint32_t* set_len,
                               const int64_t* out_off, int32_t* out_nodes, uint64_t nsets) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; s < nsets; s += stride) {
    const int32_t* from = pool + set_start[s];
    int32_t* to = out_nodes + out_off[s];
    const uint32_t len = set_len[s];
    for (uint32_t i = 0; i < len; ++i) to[i] = from[i];
  }
}

// flag[0] |= 1 if any node id of the collection lies outside [0, n).
__global__ void check_ids_kernel(const int32_t* nodes, uint64_t total, int64_t n, unsigned int* flag) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride)
    bad |= nodes[i] < 0 || (int64_t)nodes[i] >= n;
  if (bad) atomicOr(flag, 1u);
}

__global__ void set_sizes_kernel(const int64_t* set_off, uint32_t* sizes, uint64_t nsets) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; s < nsets; s += stride)
    sizes[s] = (uint32_t)(set_off[s + 1] - set_off[s]);
}

// Counters that many blocks update with device atomics sit one per 128-byte
// line (32 words apart): atomics on different words of one line wait for each
// other.  The counting sort's per-bucket counts and cursors took 0.45 ms more
// per TIM+ step on the 1M-node graph packed 32 to a line.
constexpr int kLinePad = 32;

__global__ void unpad_u32(const uint32_t* in, uint32_t* out, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[(size_t)i * kLinePad];
}

__global__ void zero_u32(uint32_t* p, uint64_t len) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += stride) p[i] = 0u;
}

__global__ void zero_u8(uint8_t* p, uint64_t len) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += stride) p[i] = 0u;
}

__global__ void zero_u64(unsigned long long* p, uint64_t len) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += stride) p[i] = 0ull;
}

// ---- views of a collection: set s has len(s) nodes from nodes[start(s)] ----
struct CsrSets {  // flat CSR (caller collections, resident prefixes)
  const int64_t* off;
  const int32_t* nodes;
  __device__ __forceinline__ int64_t start(uint64_t s) const { return off[s]; }
  __device__ __forceinline__ uint32_t len(uint64_t s) const { return (uint32_t)(off[s + 1] - off[s]); }
};
struct PoolSets {  // node pool as the samplers leave it (per-set start and size)
  const uint64_t* st;
  const uint32_t* ln;
  const int32_t* nodes;
  __device__ __forceinline__ int64_t start(uint64_t s) const { return (int64_t)st[s]; }
  __device__ __forceinline__ uint32_t len(uint64_t s) const { return ln[s]; }
};

// ---- per-tile aggregation of node updates in LDS ----
// A tile's updates to the same node (hub nodes recur in many RR sets) are
// summed in an LDS open-addressing table (at most about half full for a tile
// of typical sets) and reach device memory as one atomic per distinct node
// per tile.  A node that finds no free slot among the first kAggProbes of its
// probe sequence falls back to direct atomics: a tile holding a set larger
// than the table (a set reaching a giant component) fills it, and without
// the bound every later entry would scan the whole table.  Probe sequences
// are fixed per node and slots are never freed within a tile, so a node is
// either in the table for all of its entries of the tile or for none.
constexpr int kAggLog = 12;
constexpr int kAgg = 1 << kAggLog;
constexpr int kAggProbes = 32;
constexpr int kTileSets = 128;      // sets per tile (set-tiled kernels)
constexpr int kHistTileSets = 256;  // sets per tile of the counts pass (at most kThreads)
static_assert(kTileSets <= kThreads && kHistTileSets <= kThreads, "a tile's sets are carried one per thread");
constexpr int kTileEntries = 2048;  // entries per tile (flat histogram)

// lg: the table's size in use, 2^lg <= kAgg slots.
__device__ __forceinline__ int agg_slot(uint32_t* keys, uint32_t u, bool insert, int lg = kAggLog) {
  const uint32_t key = u + 1u;
  const uint32_t mask = (1u << lg) - 1u;
  uint32_t pos = (u * 0x9E3779B1u) >> (32 - lg);
  for (int i = 0; i < kAggProbes; ++i) {
    const uint32_t cur = keys[pos];
    if (cur == key) return (int)pos;
    if (cur == 0u) {
      if (!insert) return -1;
      const uint32_t old = atomicCAS(&keys[pos], 0u, key);
      if (old == 0u || old == key) return (int)pos;
    }
    pos = (pos + 1u) & mask;
  }
  return -1;
}

// Clears the first `slots` (a multiple of 4) slots of a table.
__device__ __forceinline__ void agg_clear(uint32_t* a, uint32_t* b, int slots = kAgg) {
  uint4* a4 = reinterpret_cast<uint4*>(a);
  uint4* b4 = reinterpret_cast<uint4*>(b);
  for (int i = threadIdx.x; i < slots / 4; i += blockDim.x) {
    a4[i] = make_uint4(0u, 0u, 0u, 0u);
    if (b) b4[i] = make_uint4(0u, 0u, 0u, 0u);
  }
}

// Block-wide prefix of the sizes of a tile's sets: thread t < kTileSets
// carries set t (len 0 if it takes no part); afterwards s_pre[t] is the first
// tile position of set t, s_pre[kTileSets] the tile total, and s_start[t] its
// first entry in the collection.
template <int TS = kTileSets>
__device__ __forceinline__ void tile_prefix(uint32_t len, int64_t start, int64_t* s_start, int64_t* s_pre,
                                            uint32_t* s_wtot) {
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  uint32_t incl = len;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) s_wtot[wv] = incl;
  __syncthreads();
  uint32_t carry = 0;
  for (int w = 0; w < wv; ++w) carry += s_wtot[w];
  if (threadIdx.x < TS) {
    s_start[threadIdx.x] = start;
    s_pre[threadIdx.x + 1] = carry + incl;
  }
  if (threadIdx.x == 0) s_pre[0] = 0;
  __syncthreads();
}

// Position of tile entry e among the tile's sets: the set j with
// s_pre[j] <= e < s_pre[j+1].
__device__ __forceinline__ int tile_set_of(const int64_t* s_pre, int ns, int64_t e) {
  int lo = 0, hi = ns - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_pre[mid] <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <int TS = kTileSets>
struct TileShared {
  int64_t start[TS];
  int64_t pre[TS + 1];
  uint32_t wtot[kThreads / 64];
  uint32_t key[kAgg], cnt[kAgg];
};

// Tiles without entries (a greedy step's cover pass mostly meets tiles whose
// sets are all covered already) skip the LDS table altogether.  Smaller
// tiles still aggregate: the nodes they share are hubs, whose direct atomics
// would contend across the chip.
constexpr int64_t kAggMin = 1;

// Adds (sign +1) or subtracts the memberships of the tile's listed sets (prefix
// from tile_prefix) to cnt, skipping node `skip`.
// The table in use for a tile of `tot` entries: at least twice as many slots
// as entries (256 to kAgg), so that a tile of few entries, as most tiles of
// the cover pass are, clears and scans few slots.
__device__ __forceinline__ int agg_log_for(int64_t tot) {
  int lg = 8;
  while (lg < kAggLog && (int64_t(1) << lg) < 2 * tot) ++lg;
  return lg;
}

template <bool kAdd, int TS = kTileSets>
__device__ __forceinline__ void tile_apply(const int32_t* nodes, TileShared<TS>& t, int64_t skip, uint32_t* cnt) {
  const int64_t tot = t.pre[TS];
  const bool agg = tot >= kAggMin;
  const int lg = agg_log_for(tot);
  if (agg) {
    agg_clear(t.key, t.cnt, 1 << lg);
    __syncthreads();
  }
  for (int64_t e = threadIdx.x; e < tot; e += kThreads) {
    const int j = tile_set_of(t.pre, TS, e);
    const int32_t u = nodes[t.start[j] + (e - t.pre[j])];
    if (u == skip) continue;
    const int slot = agg ? agg_slot(t.key, (uint32_t)u, true, lg) : -1;
    if (slot >= 0) atomicAdd(&t.cnt[slot], 1u);
    else if (kAdd) atomicAdd(&cnt[u], 1u);
    else atomicSub(&cnt[u], 1u);
  }
  if (agg) {
    __syncthreads();
    for (int i = threadIdx.x; i < (1 << lg); i += kThreads) {
      if (t.key[i]) {
        if (kAdd) atomicAdd(&cnt[t.key[i] - 1u], t.cnt[i]);
        else atomicSub(&cnt[t.key[i] - 1u], t.cnt[i]);
      }
    }
  }
  __syncthreads();
}

// cnt[u] += number of sets containing u, over the entries [set_off[0], total)
// of a CSR (a caller's offsets may be a slice of a larger collection's, whose
// first set does not start at entry 0).
__global__ __launch_bounds__(kThreads) void hist_flat_kernel(const int64_t* set_off, const int32_t* nodes,
                                                             uint64_t total, uint32_t* cnt) {
  __shared__ uint32_t s_key[kAgg], s_cnt[kAgg];
  for (uint64_t t0 = (uint64_t)set_off[0] + (uint64_t)blockIdx.x * kTileEntries; t0 < total;
       t0 += (uint64_t)gridDim.x * kTileEntries) {
    agg_clear(s_key, s_cnt);
    __syncthreads();
    const uint64_t t1 = min(t0 + (uint64_t)kTileEntries, total);
    for (uint64_t e = t0 + threadIdx.x; e < t1; e += kThreads) {
      const uint32_t u = (uint32_t)nodes[e];
      const int slot = agg_slot(s_key, u, true);
      if (slot >= 0) atomicAdd(&s_cnt[slot], 1u);
      else atomicAdd(&cnt[u], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kAgg; i += kThreads)
      if (s_key[i]) atomicAdd(&cnt[s_key[i] - 1u], s_cnt[i]);
    __syncthreads();
  }
}

// cnt[u] += number of sets containing u, in tiles of sets.
// (Larger tiles than the other passes: the LDS table's clear and scan are
// spread over twice the entries, and more hub repeats meet in it.)
template <class V>
__global__ __launch_bounds__(kThreads) void hist_sets_kernel(V sets, uint64_t nsets, uint32_t* cnt) {
  constexpr int TS = kHistTileSets;
  __shared__ TileShared<TS> t;
  for (uint64_t s0 = (uint64_t)blockIdx.x * TS; s0 < nsets; s0 += (uint64_t)gridDim.x * TS) {
    const int ns = (int)min((uint64_t)TS, nsets - s0);
    uint32_t len = 0;
    int64_t start = 0;
    if (threadIdx.x < ns) {
      start = sets.start(s0 + threadIdx.x);
      len = sets.len(s0 + threadIdx.x);
    }
    tile_prefix<TS>(len, start, t.start, t.pre, t.wtot);
    tile_apply<true, TS>(sets.nodes, t, -1, cnt);
  }
}

// inv_sets[inv_off[u] ..] = the sets containing u, in no particular order.
template <class V>
__global__ __launch_bounds__(kThreads) void scatter_kernel(V sets, uint64_t nsets, const int64_t* inv_off,
                                                           uint32_t* fill, uint32_t* inv_sets) {
  __shared__ TileShared<> t;
  __shared__ uint32_t s_base[kAgg];
  for (uint64_t s0 = (uint64_t)blockIdx.x * kTileSets; s0 < nsets; s0 += (uint64_t)gridDim.x * kTileSets) {
    const int ns = (int)min((uint64_t)kTileSets, nsets - s0);
    agg_clear(t.key, t.cnt);
    uint32_t len = 0;
    int64_t start = 0;
    if (threadIdx.x < ns) {
      start = sets.start(s0 + threadIdx.x);
      len = sets.len(s0 + threadIdx.x);
    }
    tile_prefix(len, start, t.start, t.pre, t.wtot);
    const int64_t tot = t.pre[kTileSets];
    for (int64_t e = threadIdx.x; e < tot; e += kThreads) {
      const int j = tile_set_of(t.pre, kTileSets, e);
      const int slot = agg_slot(t.key, (uint32_t)sets.nodes[t.start[j] + (e - t.pre[j])], true);
      if (slot >= 0) atomicAdd(&t.cnt[slot], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kAgg; i += kThreads) {
      if (t.key[i]) s_base[i] = atomicAdd(&fill[t.key[i] - 1u], t.cnt[i]);
      t.cnt[i] = 0u;
    }
    __syncthreads();
    for (int64_t e = threadIdx.x; e < tot; e += kThreads) {
      const int j = tile_set_of(t.pre, kTileSets, e);
      const uint32_t u = (uint32_t)sets.nodes[t.start[j] + (e - t.pre[j])];
      const uint32_t sid = (uint32_t)(s0 + (uint64_t)j);
      const int slot = agg_slot(t.key, u, false);
      uint64_t pos;
      if (slot >= 0) pos = (uint64_t)inv_off[u] + s_base[slot] + atomicAdd(&t.cnt[slot], 1u);
      else pos = (uint64_t)inv_off[u] + atomicAdd(&fill[u], 1u);
      inv_sets[pos] = sid;
    }
    __syncthreads();
  }
}

// ---- counting sort of the entries by node range ----
//
// The counts pass above adds one device atomic per distinct node of every
// tile, about two for every three entries on the large collections, and
// device atomics to scattered addresses top out far below the memory's
// bandwidth.  With a workspace, the index is built instead by a counting sort
// in two levels: the entries are first moved into buckets of 2^shift
// consecutive node ids (one atomic per bucket and tile of sets), then each
// chunk of a bucket counts its nodes, and places its sets, in LDS, with one
// device atomic per distinct node and chunk (none for a bucket of one chunk).
// Counts and index are those of the direct passes: only the order of the sets
// within a node's list differs, and no step of the greedy depends on it.
// Buckets of 8192 nodes (32 KB of LDS counters per chunk): the fewer the
// buckets, the longer the runs each tile of sets writes into one bucket.
// Chunks of 16384 entries give the per-bucket passes four times the blocks of
// 65536-entry chunks, for one more atomic per node present in each extra chunk:
// the index and greedy run about 7% faster on a 1M-node graph.
constexpr int kBucketShiftMin = 13, kBucketShiftMax = 13;
// Collections of at most kDirectCounts entries are counted by the direct pass:
// the sort's eight launches cost more than its atomics save (0.7M entries: 2%
// of the 1.15 ms of a TIM+ run on 15K nodes; at 1 to 2M entries the sort gains 1% on
// stored sets of 300K nodes).
constexpr uint64_t kDirectCounts = 1ull << 20;
constexpr int kBucketMax = 8192;             // buckets (LDS counters per tile of sets)
constexpr uint32_t kBucketChunk = 1u << 14;  // entries per block of the per-bucket passes

constexpr int kSortThreads = 512;    // sets per tile of the sort at most, one per thread
constexpr int kSortWindow = 4096;    // entries per window of a tile
constexpr unsigned kSortBlocks = 1024;

enum SortPass { kSortCount, kSortMove, kSortMoveIds };

// kSortCount: fill[b * kLinePad] += entries of the collection in bucket b.
// Otherwise moves every entry (and its set id) into its bucket, fill counting
// those moved.  A block walks over tiles of ts sets in windows of kSortWindow
// entries.  An entry's set is the number of set starts up to it: a bit per entry
// and the starts before each 64 of them.  The entry's place in its bucket is what
// its LDS counter returns, after those of the windows before.  Bounded by LDS and
// latency between barriers, not by the entries' bytes.  Against tiles of 256 sets
// with a binary search for every entry's set, twice for a move, the one-step run on
// the 1M-node graph takes 0.7 ms for the count (1.27 before) and 1.4 ms for the
// move (2.5).  512 threads of 90 to 120 registers are better than 1024 (25.4 against
// 25.7 ms for that run), registers cut to 64 for twice the wavefronts worse (27.4).
template <class V, SortPass PASS>
__global__ __launch_bounds__(kSortThreads) void bucket_sort_kernel(V sets, uint64_t nsets, int ts, int shift, int nb,
                                                                   const int64_t* boff, uint32_t* fill, uint32_t* bu,
                                                                   uint32_t* bs) {
  constexpr int NW = kSortThreads / 64;
  constexpr int NC = kSortWindow / 64;  // 64-entry chunks of a window, one per lane of a wavefront
  constexpr int PW = NC / NW;           // chunks per wavefront
  static_assert(NC == 64, "a wavefront scans the chunks of a window");
  __shared__ unsigned long long red[NW];
  __shared__ unsigned long long s_marks[NC];
  __shared__ int64_t s_delta[kSortThreads];
  __shared__ uint32_t s_id[PASS == kSortMoveIds ? kSortThreads : 1];
  __shared__ uint32_t s_rank[NC], s_seen;
  __shared__ uint32_t h[kBucketMax];  // the window's entries per bucket, then where they go
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const uint64_t ntiles = (nsets + (uint64_t)ts - 1) / (uint64_t)ts;
  if (PASS == kSortCount)
    for (int i = tid; i < nb; i += kSortThreads) h[i] = 0u;
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint64_t s = tile * (uint64_t)ts + (uint64_t)tid;
    unsigned long long len = 0;
    int64_t start = 0;
    if (tid < ts && s < nsets) {
      len = sets.len(s);
      start = sets.start(s);
    }
    // entries (low 40 bits) and non-empty sets (above) before this one
    unsigned long long all;
    const unsigned long long ex = block_excl_scan<kSortThreads>(len | (len ? 1ull << 40 : 0ull), red, &all);
    const uint64_t tot = all & ((1ull << 40) - 1ull), e0 = ex & ((1ull << 40) - 1ull);
    if (len) {
      s_delta[ex >> 40] = start - (int64_t)e0;
      if (PASS == kSortMoveIds) s_id[ex >> 40] = (uint32_t)s;
    }
    uint32_t seen = 0;  // sets that started before the window
    for (uint64_t w0 = 0; w0 < tot; w0 += kSortWindow) {
      if (tid < NC) s_marks[tid] = 0ull;
      if (PASS != kSortCount)
        for (int i = tid; i < nb; i += kSortThreads) h[i] = 0u;
      __syncthreads();
      if (len && e0 >= w0 && e0 - w0 < kSortWindow) atomicOr(&s_marks[(e0 - w0) / 64], 1ull << ((e0 - w0) % 64));
      __syncthreads();
      if (wv == 0) {
        const uint32_t x = (uint32_t)__popcll(s_marks[lane]);
        uint32_t inc = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t y = __shfl_up(inc, o, 64);
          if (lane >= o) inc += y;
        }
        s_rank[lane] = seen + inc - x;
        if (lane == 63) s_seen = seen + inc;
      }
      __syncthreads();
      seen = s_seen;
      uint32_t u[PW], rk[PW], at[PW];
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const int ch = i * NW + wv;
        const uint64_t e = w0 + (uint64_t)(ch * 64 + lane);
        u[i] = rk[i] = at[i] = 0u;
        if (e < tot) {
          rk[i] = s_rank[ch] + (uint32_t)__popcll(s_marks[ch] & (~0ull >> (63 - lane))) - 1u;
          u[i] = (uint32_t)sets.nodes[s_delta[rk[i]] + (int64_t)e];
        }
      }
#pragma unroll
      for (int i = 0; i < PW; ++i)
        if (w0 + (uint64_t)((i * NW + wv) * 64 + lane) < tot) at[i] = atomicAdd(&h[u[i] >> shift], 1u);
      __syncthreads();
      if (PASS == kSortCount) continue;
      for (int i = tid; i < nb; i += kSortThreads)
        if (h[i]) h[i] = (uint32_t)boff[i] + atomicAdd(&fill[(size_t)i * kLinePad], h[i]);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        if (w0 + (uint64_t)((i * NW + wv) * 64 + lane) < tot) {
          const uint32_t pos = h[u[i] >> shift] + at[i];
          bu[pos] = u[i];
          if (PASS == kSortMoveIds) bs[pos] = s_id[rk[i]];
        }
      }
      __syncthreads();
    }
  }
  if (PASS == kSortCount) {
    __syncthreads();
    for (int i = tid; i < nb; i += kSortThreads)
      if (h[i]) atomicAdd(&fill[(size_t)i * kLinePad], h[i]);
  }
}

// Chunks of kBucketChunk entries per bucket: cstart[b] is bucket b's first
// chunk, cstart[nb] their number, cb[c] the bucket of chunk c.
__global__ __launch_bounds__(kThreads) void bucket_chunks_kernel(const int64_t* boff, int nb, uint32_t* cstart,
                                                                 uint32_t* cb) {
  __shared__ unsigned long long red[kThreads / 64];
  unsigned long long carry = 0;
  for (int base = 0; base < nb; base += kThreads) {
    const int b = base + (int)threadIdx.x;
    const unsigned long long len = b < nb ? (unsigned long long)(boff[b + 1] - boff[b]) : 0ull;
    const unsigned long long ch = (len + kBucketChunk - 1) / kBucketChunk;
    unsigned long long total;
    const unsigned long long ex = block_excl_scan(ch, red, &total);
    if (b < nb) {
      const uint32_t c0 = (uint32_t)(carry + ex);
      cstart[b] = c0;
      for (uint32_t j = 0; j < (uint32_t)ch; ++j) cb[c0 + j] = (uint32_t)b;
    }
    carry += total;
  }
  if (threadIdx.x == 0) cstart[nb] = (uint32_t)carry;
}

// The bucket, first entry and end of chunk blockIdx.x; false past the last chunk.
__device__ __forceinline__ bool chunk_of(const int64_t* boff, const uint32_t* cstart, const uint32_t* cb, int nb,
                                         uint32_t& b, int64_t& e0, int64_t& e1, bool& alone) {
  const uint32_t c = blockIdx.x;
  if (c >= cstart[nb]) return false;
  b = cb[c];
  e0 = boff[b] + (int64_t)(c - cstart[b]) * kBucketChunk;
  e1 = min(e0 + (int64_t)kBucketChunk, boff[b + 1]);
  alone = cstart[b + 1] - cstart[b] == 1u;
  return true;
}

constexpr int kCountThreads = 512;

// cnt of the chunk's node range: stored where the chunk is its bucket's only
// one, else added with one atomic per node present.
// (0.34 ms for the one-step run on the 1M-node graph; with a 4-byte load per entry
// and 256 threads 0.61.)
__global__ __launch_bounds__(kCountThreads) void bucket_count_kernel(const uint32_t* bu, const int64_t* boff,
                                                                const uint32_t* cstart, const uint32_t* cb, int nb,
                                                                int shift, int64_t n, uint32_t* cnt) {
  __shared__ __align__(16) uint32_t lc[1 << kBucketShiftMax];
  uint32_t b;
  int64_t e0, e1;
  bool alone;
  if (!chunk_of(boff, cstart, cb, nb, b, e0, e1, alone)) return;
  const int range = 1 << shift;
  const uint32_t base = b << shift;
  for (int i = threadIdx.x; i < range / 4; i += kCountThreads) reinterpret_cast<uint4*>(lc)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  // four entries per load between the chunk's 16-byte boundaries
  const int64_t v0 = min((e0 + 3) & ~(int64_t)3, e1), v1 = max(e1 & ~(int64_t)3, v0);
  if (e0 + threadIdx.x < v0) atomicAdd(&lc[bu[e0 + threadIdx.x] - base], 1u);
  if (v1 + threadIdx.x < e1) atomicAdd(&lc[bu[v1 + threadIdx.x] - base], 1u);
#pragma unroll 4
  for (int64_t e = v0 + 4 * threadIdx.x; e < v1; e += 4 * kCountThreads) {
    const uint4 u = *reinterpret_cast<const uint4*>(bu + e);
    atomicAdd(&lc[u.x - base], 1u);
    atomicAdd(&lc[u.y - base], 1u);
    atomicAdd(&lc[u.z - base], 1u);
    atomicAdd(&lc[u.w - base], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < range && (int64_t)base + i < n; i += kCountThreads) {
    if (alone) cnt[base + i] = lc[i];
    else if (lc[i]) atomicAdd(&cnt[base + i], lc[i]);
  }
}

// inv_sets of the chunk's nodes: positions from inv_off, plus a base per node
// taken from fill where the bucket has several chunks.
__global__ __launch_bounds__(kThreads) void bucket_index_kernel(const uint32_t* bu, const uint32_t* bs,
                                                                const int64_t* boff, const uint32_t* cstart,
                                                                const uint32_t* cb, int nb, int shift, int64_t n,
                                                                const int64_t* inv_off, uint32_t* fill,
                                                                uint32_t* inv_sets) {
  __shared__ uint32_t lc[1 << kBucketShiftMax];  // the chunk's entries per node, then their next position
  uint32_t b;
  int64_t e0, e1;
  bool alone;
  if (!chunk_of(boff, cstart, cb, nb, b, e0, e1, alone)) return;
  const int range = 1 << shift;
  const uint32_t base = b << shift;
  for (int i = threadIdx.x; i < range; i += kThreads) lc[i] = 0u;
  __syncthreads();
  if (!alone) {
    for (int64_t e = e0 + threadIdx.x; e < e1; e += kThreads) atomicAdd(&lc[bu[e] - base], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < range && (int64_t)base + i < n; i += kThreads)
      if (lc[i]) lc[i] = atomicAdd(&fill[base + i], lc[i]);
    __syncthreads();
  }
  for (int64_t e = e0 + threadIdx.x; e < e1; e += kThreads) {
    const uint32_t u = bu[e];
    inv_sets[inv_off[u] + atomicAdd(&lc[u - base], 1u)] = bs[e];
  }
}

// Key of node u: 0 if selected, else count<<32 | (0xFFFFFFFF - u), so the
// maximum key is the largest count with the lowest id; unselected keys > 0.
// Few blocks, 4 nodes per thread and load: one atomicMax per block.
__global__ __launch_bounds__(kThreads) void argmax_kernel(const uint32_t* cnt, const uint8_t* selected, int64_t n,
                                                          unsigned long long* best) {
  unsigned long long key = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n4 = n >> 2;
  const uint4* c4 = reinterpret_cast<const uint4*>(cnt);
  const uint32_t* s4 = reinterpret_cast<const uint32_t*>(selected);
  for (int64_t i = tid; i < n4; i += stride) {
    const uint4 c = c4[i];
    const uint32_t sel = s4[i];
    const uint32_t cv[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const unsigned long long u = (unsigned long long)(4 * i + w);
      const unsigned long long k = ((unsigned long long)cv[w] << 32) | (0xFFFFFFFFull - u);
      if (!((sel >> (8 * w)) & 0xFFu)) key = k > key ? k : key;
    }
  }
  for (int64_t u = 4 * n4 + tid; u < n; u += stride) {
    if (selected[u]) continue;
    const unsigned long long k = ((unsigned long long)cnt[u] << 32) | (0xFFFFFFFFull - (unsigned long long)u);
    key = k > key ? k : key;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long y = __shfl_xor(key, o, 64);
    key = y > key ? y : key;
  }
  __shared__ unsigned long long red[kThreads / 64];
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  if (lane == 0) red[wv] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 0; w < kThreads / 64; ++w) key = red[w] > key ? red[w] : key;
    if (key) atomicMax(best, key);
  }
}

__device__ __forceinline__ int64_t node_of_key(unsigned long long key) {
  return (int64_t)(0xFFFFFFFFull - (key & 0xFFFFFFFFull));
}

// The chosen node v covers the sets listed in inv_sets[inv_off[v] ..]: mark
// those not covered yet and take them out of the counts of their members
// (v's own count is left alone: v is never chosen again).
template <class V>
__global__ __launch_bounds__(kThreads) void cover_kernel(const unsigned long long* best, const int64_t* inv_off,
                                                         const uint32_t* inv_sets, V sets, uint8_t* covered,
                                                         uint8_t* selected, uint32_t* cnt) {
  __shared__ TileShared<> t;
  if (*best == 0ull) return;  // no unselected node (cannot happen for k <= n)
  const int64_t v = node_of_key(*best);
  if (blockIdx.x == 0 && threadIdx.x == 0) selected[v] = 1u;
  const int64_t lo = inv_off[v], hi = inv_off[v + 1];
  for (int64_t i0 = lo + (int64_t)blockIdx.x * kTileSets; i0 < hi; i0 += (int64_t)gridDim.x * kTileSets) {
    const int ni = (int)min((int64_t)kTileSets, hi - i0);
    // newly covered sets of this tile and their sizes
    uint32_t len = 0;
    int64_t start = 0;
    if (threadIdx.x < ni) {
      const uint32_t sid = inv_sets[i0 + threadIdx.x];
      if (!covered[sid]) {
        covered[sid] = 1u;
        start = sets.start(sid);
        len = sets.len(sid);
      }
    }
    tile_prefix(len, start, t.start, t.pre, t.wtot);
    tile_apply<false>(sets.nodes, t, v, cnt);
  }
}

__global__ void select_kernel(const unsigned long long* best, uint8_t* selected) {
  if (threadIdx.x == 0 && *best != 0ull) selected[node_of_key(*best)] = 1u;
}

// Sets (pool layout) not covered yet that contain the chosen node v: mark
// them and take them out of the counts of their members.
__global__ __launch_bounds__(kThreads) void scan_cover_kernel(const unsigned long long* best, PoolSets sets,
                                                              uint64_t nsets, uint8_t* covered, uint32_t* cnt) {
  __shared__ TileShared<> t;
  __shared__ uint32_t s_hit[kTileSets];
  if (*best == 0ull) return;
  const int64_t v = node_of_key(*best);
  for (uint64_t s0 = (uint64_t)blockIdx.x * kTileSets; s0 < nsets; s0 += (uint64_t)gridDim.x * kTileSets) {
    const int ns = (int)min((uint64_t)kTileSets, nsets - s0);
    uint32_t len = 0;
    int64_t start = 0;
    if (threadIdx.x < ns && !covered[s0 + threadIdx.x]) {
      start = sets.start(s0 + threadIdx.x);
      len = sets.len(s0 + threadIdx.x);
    }
    if (threadIdx.x < kTileSets) s_hit[threadIdx.x] = 0u;
    tile_prefix(len, start, t.start, t.pre, t.wtot);
    // membership of v
    const int64_t tot = t.pre[kTileSets];
    for (int64_t e = threadIdx.x; e < tot; e += kThreads) {
      const int j = tile_set_of(t.pre, kTileSets, e);
      if (sets.nodes[t.start[j] + (e - t.pre[j])] == v) s_hit[j] = 1u;
    }
    __syncthreads();
    bool hit = false;
    if (threadIdx.x < ns) {
      hit = s_hit[threadIdx.x] != 0u;
      if (hit) covered[s0 + threadIdx.x] = 1u;
    }
    tile_prefix(hit ? len : 0u, start, t.start, t.pre, t.wtot);
    tile_apply<false>(sets.nodes, t, v, cnt);
  }
}

// ---- the greedy over candidates ----
//
// A choice's key is its count, ties to the lowest node.  Counts only fall, so a
// node whose initial key is below T is never chosen while some candidate
// (initial key at least T) still has T or more.  The greedy of k > 1 therefore
// takes the nodes of the largest keys as candidates (kCandPerStep per step, at
// least kCandMin, at most kCandMax) and
// keeps of every set only its candidates, as a stream of 16-bit candidate
// numbers whose top bit marks the first entry of a set.  One kernel over the
// stream takes one or several greedy steps: every block decides them itself from
// the counts, then takes the sets of the chosen candidates in its part of the
// stream out of the stream and of the counts.  No inverted index is built, no
// set offsets or covered marks are kept, and the argmax reads the candidates
// instead of n nodes.
// Several steps at once: each launch also counts, over the sets it leaves, how
// many contain each combination of kCandTop candidates of large counts (the tops).
// While the best candidate is one of those, the counts of the others after its
// choice follow from the combinations, and the best of them is the next choice as
// long as its key is above that of every candidate outside the tops (their counts
// only fall).
// A launch whose best candidate's key has fallen below T leaves key 1, which no choice
// has, and the caller runs the greedy over all nodes.  Seeds and gains are those
// of that greedy: a choice's key is the largest over all nodes at its step.
// Against the inverted index with an argmax over n nodes and a cover pass per
// step (10 to 16 us a step), TIM+ runs took: k = 50 on the 1M-node graph under IC
// 5.41 -> 4.67 ms with one step per launch (7 to 9 us), k = 50 on 15K nodes under
// LT 1.78 -> 1.48 ms, k = 25 on 123K nodes with per-edge probabilities 4.58 ->
// 3.79 ms.  With several steps per launch (13 to 16 launches instead of 50 for
// k = 50, 4 to 6 instead of 10 for k = 10) k = 50 on the 1M-node graph went 4.20 ->
// 3.76 ms, k = 50 on 15K nodes under LT 1.56 -> 1.14, k = 25 on 123K nodes 3.42 ->
// 3.16, k = 20 on 300K stored sets 1.09 -> 1.02, k = 10 on 3K nodes 0.93 -> 0.88.
// Half the candidates per step (128) leave the triggering model's greedy of
// k = 10 on 200K nodes undecided (6.1 -> 6.6 ms) and gain nothing elsewhere.
constexpr int kCandMin = 2048, kCandMax = 8192, kCandPerStep = 256;
constexpr int kCandMaxSteps = 256;   // beyond, the candidates a greedy needs outgrow kCandMax
constexpr uint32_t kCandDead = 0x7FFFu;      // number of an entry taken out
constexpr uint32_t kCandFirst = 0x8000u;     // first entry of its set
constexpr uint32_t kCandTaken = 0xFFFFFFFFu; // count of a chosen candidate
constexpr int kCandBins = 2048;
constexpr uint32_t kCandBinsUsed = 128u + 25u * 64u;  // those above belong to no 32-bit count
constexpr uint32_t kCandTies = 32;   // counts whose nodes are also counted per block: T may lie between equal counts
constexpr int kCandSegs = 256;       // parts of the stream, one per block of a step
constexpr int kCandStepThreads = 1024;
constexpr int kCandBuildThreads = 1024;
constexpr int kCandTileMax = kCandBuildThreads;  // sets per tile of the build, one per thread
constexpr int kCandWindow = 4096;    // entries per window of the build
constexpr int kCandTop = 8;          // tops whose combinations are counted
constexpr int kCandCombos = 1 << kCandTop;
constexpr int kCandRows = 8;         // counters per combination: blocks add to that of their number mod 8
constexpr int kCandTileVecs = 4;     // vectors of eight entries per thread in a tile of the stream
constexpr uint32_t kCandChosen = 0x100u;  // class bit of this launch's choices (below it: one bit per top)
constexpr uint32_t kCandOpen = 0x200u;    // with them: the set goes on after the tile
constexpr uint32_t kCandStarts = 1u << 24;

struct CandHead {  // counters of one greedy
  unsigned long long t;  // T, as a key
  uint32_t n;      // candidates
  uint32_t cursor; // stream entries reserved
  uint32_t failed; // a step found no candidate at or above T
  uint32_t picked[2];  // choices before launches j mod 2
  uint32_t tops[2][kCandTop];  // number + 1 of the tops counted by launch j - 1 (0: none), for launches j mod 2
  alignas(16) uint32_t combos[3][kCandRows][kCandCombos];  // sets left with each combination by launches j mod 3
};

struct CandArrays {
  CandHead* head;
  uint32_t* bins;       // kCandBins
  uint32_t* dec;        // 3 x kCandMax: what steps j-1, j, j+1 mod 3 take out of the counts
  uint32_t* base;       // 2 x kCandMax: counts before step j-1's part is taken out, for steps j mod 2
  uint32_t* node;       // kCandMax: node of a candidate
  uint32_t* seg_start;  // kCandSegs
  uint32_t* seg_len;    // kCandSegs
  uint16_t* map;        // n: candidate number + 1, or 0
  uint16_t* stream;
  int segs;
};

// Bins of counts: exact below 128, then 64 per power of two (the more alike the
// counts are, the finer the bins have to be to part the largest from the rest).
__device__ __forceinline__ uint32_t cand_bin(uint32_t c) {
  if (c < 128u) return c;
  const uint32_t e = 31u - (uint32_t)__clz((int)c);
  return 128u + (e - 7u) * 64u + ((c >> (e - 6u)) & 63u);
}
__device__ __forceinline__ uint32_t cand_bin_low(uint32_t b) {
  if (b < 128u) return b;
  const uint32_t e = 7u + (b - 128u) / 64u;
  return (64u + ((b - 128u) & 63u)) << (e - 6u);
}

// Nodes per block of cand_bins_kernel and cand_pick_kernel, which have the same grid.
__device__ __forceinline__ int64_t cand_span(int64_t n) {
  return ((n + gridDim.x - 1) / gridDim.x + kThreads - 1) / kThreads * kThreads;
}

// Clears the counters, bins and dec, and marks every candidate number of
// base as taken until cand_pick_kernel gives it to a node.
__global__ void cand_init_kernel(CandArrays c, unsigned long long* best, int k) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
  for (int x = i; x < (int)(sizeof(CandHead) / 4); x += stride) reinterpret_cast<uint32_t*>(c.head)[x] = 0u;
  for (int x = i; x < k; x += stride) best[x] = 0ull;
  for (int x = i; x < kCandBins; x += stride) c.bins[x] = 0u;
  for (int x = i; x < 3 * kCandMax; x += stride) c.dec[x] = 0u;
  for (int x = i; x < 2 * kCandMax; x += stride) c.base[x] = kCandTaken;
}

// ties[b * kCandTies + c]: nodes of block b with count c.
__global__ __launch_bounds__(kThreads) void cand_bins_kernel(const uint32_t* cnt, int64_t n, uint32_t* bins,
                                                             uint32_t* ties) {
  __shared__ uint32_t s_bin[kCandBins];
  for (int i = threadIdx.x; i < kCandBins; i += kThreads) s_bin[i] = 0u;
  __syncthreads();
  uint32_t low[4] = {0u, 0u, 0u, 0u};  // most nodes have counts below 4: not through one LDS word
  const int64_t lo = (int64_t)blockIdx.x * cand_span(n), hi = min(lo + cand_span(n), n);
  for (int64_t u = lo + threadIdx.x; u < hi; u += kThreads) {
    const uint32_t c = cnt[u];
    if (c >= 4u) atomicAdd(&s_bin[cand_bin(c)], 1u);
#pragma unroll
    for (uint32_t w = 0; w < 4u; ++w) low[w] += c == w ? 1u : 0u;
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    uint32_t x = low[w];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if (threadIdx.x % 64 == 0 && x) atomicAdd(&s_bin[w], x);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kCandBins; i += kThreads)
    if (s_bin[i]) atomicAdd(&bins[i], s_bin[i]);
  if (threadIdx.x < kCandTies) ties[(size_t)blockIdx.x * kCandTies + threadIdx.x] = s_bin[threadIdx.x];
}

// T: the low end of the lowest bin with at most `most` nodes in it and above.
// Of the next lower bin, if all its nodes have one small count, the blocks from
// the first on join as long as their nodes of that count fit, so that equal
// counts do not end the greedy early: T is then the key of the last node of the
// last such block.  (0 where all n nodes are candidates.)  Then the candidates'
// numbers.  Neighbouring nodes get numbers 64 apart, in different rows of lanes
// of a step, which takes its next tops from the best of each row: nodes of the
// largest keys that are numbered one after the other would leave it one choice
// per launch (graphs whose hubs come first, equal counts).
__global__ __launch_bounds__(kThreads) void cand_pick_kernel(const uint32_t* cnt, int64_t n, uint32_t most,
                                                             const uint32_t* ties, CandArrays c) {
  __shared__ unsigned long long red[kThreads / 64];
  __shared__ uint32_t s_cut, s_above;
  constexpr int per = kCandBins / kThreads;
  static_assert(per == 8, "two loads of four bins per thread");
  const int64_t span = cand_span(n);
  unsigned long long total;
  uint32_t t = 0;
  int64_t joined = 0;  // nodes below this one of count t - 1 are candidates too
  if (n > (int64_t)most) {
    // thread t holds bins from the top: kCandBins - 1 - per * t downwards
    const uint32_t top = (uint32_t)(kCandBins - 1 - per * (int)threadIdx.x);
    const uint4* b4 = reinterpret_cast<const uint4*>(c.bins) + (top + 1u - (uint32_t)per) / 4u;
    const uint4 b0 = b4[0], b1 = b4[1];
    const uint32_t b[per] = {b1.w, b1.z, b1.y, b1.x, b0.w, b0.z, b0.y, b0.x};
    if (threadIdx.x == 0) {
      s_cut = kCandBinsUsed;  // the top bin alone is too large
      s_above = 0u;
    }
    unsigned long long above = block_excl_scan((unsigned long long)(b[0] + b[1] + b[2] + b[3] + b[4] + b[5] + b[6] + b[7]),
                                               red, &total);
    uint32_t cut_here = kCandBinsUsed, above_here = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
      above += b[i];
      if (above <= most && top - (uint32_t)i < kCandBinsUsed) {
        cut_here = top - (uint32_t)i;
        above_here = (uint32_t)above;
      }
    }
    if (cut_here < kCandBinsUsed) atomicMin(&s_cut, cut_here);
    __syncthreads();
    const uint32_t cut = s_cut;
    if (cut_here == cut && cut < kCandBinsUsed) s_above = above_here;
    t = cut < kCandBinsUsed ? cand_bin_low(cut) : 0xFFFFFFFFu;
    if (cut <= kCandTies) {  // (cut > 0: all bins together hold n nodes)
      const bool block = threadIdx.x < gridDim.x;
      const unsigned long long mine = block ? ties[(size_t)threadIdx.x * kCandTies + cut - 1u] : 0ull;
      const unsigned long long upto = block_excl_scan(mine, red, &total) + mine;
      joined = min(span * (int64_t)__syncthreads_count(block && s_above + upto <= most), n);
    }
    __syncthreads();
  }
  if (blockIdx.x == 0 && threadIdx.x == 0)
    c.head->t = t == 0xFFFFFFFFu ? ~0ull : ((unsigned long long)t << 32) - (unsigned long long)joined;
  // the block's nodes in two passes, so that it reserves its candidates' numbers with one atomic
  const int64_t lo = (int64_t)blockIdx.x * span, hi = min(lo + span, n);
  const uint32_t least = lo < joined ? t - 1u : t;  // joined is a block's first node, or n
  unsigned long long mine = 0;
#pragma unroll 4
  for (int64_t u = lo + threadIdx.x; u < hi; u += kThreads) mine += cnt[u] >= least ? 1ull : 0ull;
  uint32_t id = (uint32_t)block_excl_scan(mine, red, &total);
  if (threadIdx.x == 0) s_cut = total ? atomicAdd(&c.head->n, (uint32_t)total) : 0u;
  __syncthreads();
  id += s_cut;
  const uint32_t rows = most / 64u;
#pragma unroll 4
  for (int64_t u = lo + threadIdx.x; u < hi; u += kThreads) {
    const uint32_t x = cnt[u];
    const bool in = x >= least;
    const uint32_t num = id % rows * 64u + id / rows;
    if (in) {
      c.node[num] = (uint32_t)u;
      c.base[num] = x;
    }
    c.map[u] = in ? (uint16_t)(num + 1u) : (uint16_t)0u;
    id += in ? 1u : 0u;
  }
}

// The stream: block b takes the tiles b, b + gridDim.x, ... of `ts` sets and
// writes the candidates of their sets one set after the other into its part.
// What bounds it: two dependent reads per entry (the node, its candidate
// number); an entry finds its set by counting the set starts up to it in an
// LDS bit array, as many bits as a window has entries.
template <class V>
__global__ __launch_bounds__(kCandBuildThreads) void cand_build_kernel(V sets, uint64_t nsets, int ts, CandArrays c) {
  constexpr int NW = kCandBuildThreads / 64;
  constexpr int NC = kCandWindow / 64;  // 64-entry chunks of a window, one per lane of a wavefront
  constexpr int PW = NC / NW;           // chunks per wavefront
  static_assert(NC == 64, "a wavefront scans the chunks of a window");
  __shared__ unsigned long long red[NW];
  __shared__ unsigned long long s_marks[NC];
  __shared__ int64_t s_delta[kCandTileMax];
  __shared__ uint32_t s_first[kCandTileMax], s_rank[NC], s_cnt[NC], s_base;
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const uint64_t ntiles = (nsets + (uint64_t)ts - 1) / (uint64_t)ts;
  // room for every entry of the block's sets
  unsigned long long mine = 0, room;
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint64_t s = tile * (uint64_t)ts + (uint64_t)tid;
    if (tid < ts && s < nsets) mine += sets.len(s);
  }
  (void)block_excl_scan<kCandBuildThreads>(mine, red, &room);
  if (tid == 0) s_base = atomicAdd(&c.head->cursor, (uint32_t)((room + 63ull) & ~63ull));
  __syncthreads();
  const uint32_t base = s_base;
  uint32_t at = 0;  // entries written
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint64_t s = tile * (uint64_t)ts + (uint64_t)tid;
    unsigned long long len = 0;
    int64_t start = 0;
    if (tid < ts && s < nsets) {
      len = sets.len(s);
      start = sets.start(s);
    }
    // entries (low 40 bits) and non-empty sets (above) before this one
    unsigned long long all;
    const unsigned long long ex = block_excl_scan<kCandBuildThreads>(len | (len ? 1ull << 40 : 0ull), red, &all);
    const uint64_t tot = all & ((1ull << 40) - 1ull), e0 = ex & ((1ull << 40) - 1ull);
    const uint32_t rank = (uint32_t)(ex >> 40);
    if (len) {
      s_delta[rank] = start - (int64_t)e0;
      s_first[rank] = 0xFFFFFFFFu;
    }
    uint32_t seen = 0;  // sets that started before the window
    for (uint64_t w0 = 0; w0 < tot; w0 += kCandWindow) {
      if (tid < NC) s_marks[tid] = 0ull;
      __syncthreads();
      if (len && e0 >= w0 && e0 - w0 < kCandWindow) atomicOr(&s_marks[(e0 - w0) / 64], 1ull << ((e0 - w0) % 64));
      __syncthreads();
      if (wv == 0) {
        uint32_t x = (uint32_t)__popcll(s_marks[lane]), inc = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t y = __shfl_up(inc, o, 64);
          if (lane >= o) inc += y;
        }
        s_rank[lane] = seen + inc - x;
        if (lane == 63) s_base = seen + inc;
      }
      __syncthreads();
      seen = s_base;
      uint32_t id[PW], rk[PW];  // candidate number + 1 (0: none), set of the entry
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const int ch = i * NW + wv;
        const uint64_t e = w0 + (uint64_t)(ch * 64 + lane);
        id[i] = rk[i] = 0u;
        if (e < tot) {
          rk[i] = s_rank[ch] + (uint32_t)__popcll(s_marks[ch] & (~0ull >> (63 - lane))) - 1u;
          id[i] = c.map[sets.nodes[s_delta[rk[i]] + (int64_t)e]];
        }
        const uint64_t m = __ballot(id[i] != 0u);
        if (lane == 0) s_cnt[ch] = (uint32_t)__popcll(m);
      }
      __syncthreads();
      const uint32_t x = s_cnt[lane];
      uint32_t inc = x;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
      }
      const uint32_t found = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
      const uint32_t chunk_at = at + inc - x;  // lane ch: where chunk ch's candidates go
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const uint64_t m = __ballot(id[i] != 0u);
        const uint64_t below = m & ((1ull << lane) - 1ull);
        const uint32_t pos =
            (uint32_t)__builtin_amdgcn_readlane((int)chunk_at, i * NW + wv) + (uint32_t)__popcll(below);
        // of a set's candidates in this chunk only the first bids
        const uint32_t prev = __shfl(rk[i], below ? 63 - __clzll((long long)below) : lane, 64);
        if (id[i] && (!below || prev != rk[i])) atomicMin(&s_first[rk[i]], pos);
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const uint64_t m = __ballot(id[i] != 0u);
        const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)chunk_at, i * NW + wv) +
                             (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (id[i])
          c.stream[(size_t)base + pos] = (uint16_t)((id[i] - 1u) | (s_first[rk[i]] == pos ? kCandFirst : 0u));
      }
      at += found;
    }
    __syncthreads();
  }
  const uint32_t end = (at + 63u) & ~63u;  // within the room, itself a multiple of 64
  if (at + (uint32_t)tid < end) c.stream[(size_t)base + at + (uint32_t)tid] = (uint16_t)(kCandFirst | kCandDead);
  if (tid == 0) {
    c.seg_start[blockIdx.x] = base;
    c.seg_len[blockIdx.x] = end;
  }
}

// x of the lane that DPP control CTRL names.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}

template <int CTRL>
__device__ __forceinline__ unsigned long long dpp64(unsigned long long x) {
  return ((unsigned long long)dpp32<CTRL>((uint32_t)(x >> 32)) << 32) | dpp32<CTRL>((uint32_t)x);
}

constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141;  // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppRowShr = 0x110, kDppRowRor = 0x120;                    // + 1..15

// Sum over eight neighbouring lanes, in all of them (every lane of the wavefront active).
__device__ __forceinline__ uint32_t sum8(uint32_t x) {
  x += dpp32<kDppXor1>(x);
  x += dpp32<kDppXor2>(x);
  return x + dpp32<kDppHalfMirror>(x);
}

// The lanes are consecutive pieces of the stream: with `starts` sets start in the
// piece, head are the classes before the first of them and tail those from the
// last on; without, head are its classes.  to_end: classes of the set open at the
// lane's end, from its start or lane 0 on; on: classes from the lane's first entry
// up to the next set's start or the end of lane 63.
__device__ __forceinline__ void scan_classes(uint32_t head, uint32_t tail, bool starts, int lane, uint32_t* to_end,
                                             uint32_t* on) {
  const uint64_t all = __ballot(starts), upto = all & (~0ull >> (63 - lane)), from = all & (~0ull << lane);
  const int back = upto ? lane - (63 - __clzll((long long)upto)) : lane;
  const int ahead = from ? __ffsll((unsigned long long)from) - 1 - lane : 63 - lane;
  uint32_t p = starts ? tail : head, q = head;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(p, d, 64), z = __shfl_down(q, d, 64);
    if (d <= back) p |= y;
    if (d <= ahead) q |= z;
  }
  *to_end = p;
  *on = q;
}

__device__ __forceinline__ unsigned long long max64(unsigned long long x, unsigned long long y) { return x > y ? x : y; }

// The maximum over each row of 16 lanes, in every lane.
__device__ __forceinline__ unsigned long long row_max64(unsigned long long x) {
  x = max64(x, dpp64<kDppRowRor + 8>(x));
  x = max64(x, dpp64<kDppRowRor + 4>(x));
  x = max64(x, dpp64<kDppRowRor + 2>(x));
  return max64(x, dpp64<kDppRowRor + 1>(x));
}

__device__ __forceinline__ unsigned long long lane64(unsigned long long x, int lane) {
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
  return ((unsigned long long)hi << 32) | lo;
}

// A barrier that orders LDS only, so that loads from global memory stay in flight over it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Launch j.  Counts before it are base[j mod 2] less what launch j-1 took out,
// dec[(j-1) mod 3]; nothing written here is read by another block of the launch.
// What bounds it is a chain of latencies, not the stream's bytes: the launch, the
// loads (the part's vectors are loaded with the counts), the decision, the scans,
// the counts' atomics: 10 to 17 us with a decision of 0.9 to 2.4, where one
// choice per launch took 7 to 8.  Tops in descending order of their keys come from
// ranks that eight lanes each count while wavefront 0 decides; reducing them and
// the tops' counts lane by lane instead took 3 to 16 us per launch.
// The sets' classes come from scans over the stream, which cost the same for any
// mix of sets.  A walk from every match to both ends of its set took 20 to 190 us
// in the first launches, where most sets match (LT with in-weights, k = 10 on the
// 1M-node graph: 188 against 40 us).
__global__ __launch_bounds__(kCandStepThreads) void cand_step_kernel(CandArrays c, int most, int j, int k,
                                                                      unsigned long long* best) {
  constexpr int NW = kCandStepThreads / 64, ROWS = kCandStepThreads / 16, KEYS = ROWS + kCandTop;
  constexpr int ORDER = 2 * kCandTop;  // the next tops are the first of these not chosen
  static_assert(ROWS == 64 && kCandTop == 8 && KEYS % 8 == 0 && kCandStepThreads >= 64 + 8 * KEYS,
                "a wavefront decides over the rows, eight lanes rank each key");
  constexpr int VECS = kCandTileVecs, TILE = VECS * kCandStepThreads;  // vectors per thread and tile
  static_assert(VECS * NW == 64, "a wavefront scans the chunks of a tile");
  __shared__ __align__(16) uint32_t s_dec[kCandMax];
  __shared__ __align__(16) uint16_t s_cls[kCandMax];
  __shared__ uint32_t s_chunk[64];  // of a tile's chunks of 64 vectors: head | tail << 12 | kCandStarts
  __shared__ unsigned long long s_key[KEYS];  // best outside the tops per row of lanes, then the tops
  __shared__ uint32_t s_num[KEYS];            // their numbers
  __shared__ __align__(16) uint32_t s_within[kCandCombos];  // sets whose combination is within this one
  __shared__ uint32_t s_combos[kCandCombos];
  __shared__ uint32_t s_chosen[kCandTop], s_order[ORDER];
  __shared__ int s_nchosen;
  __shared__ uint32_t s_any;
  __shared__ int s_open[2];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  CandHead* head = c.head;
  const unsigned long long t = head->t;
  const uint32_t picked = head->picked[j & 1];
  const bool failed = head->failed != 0u;
  const int nvec = (int)(c.seg_len[blockIdx.x] / 8u);
  uint16_t* part = c.stream + c.seg_start[blockIdx.x];
  uint4* vec = reinterpret_cast<uint4*>(part);
  const uint4* base = reinterpret_cast<const uint4*>(c.base + (size_t)(j & 1) * kCandMax);
  uint4* base_next = reinterpret_cast<uint4*>(c.base + (size_t)((j + 1) & 1) * kCandMax);
  const uint4* dec_prev = reinterpret_cast<const uint4*>(c.dec + (size_t)((j + 2) % 3) * kCandMax);
  uint32_t* dec_now = c.dec + (size_t)(j % 3) * kCandMax;
  uint4* dec_next = reinterpret_cast<uint4*>(c.dec + (size_t)((j + 1) % 3) * kCandMax);
  const uint4* node = reinterpret_cast<const uint4*>(c.node);
  uint32_t old[kCandTop];
#pragma unroll
  for (int i = 0; i < kCandTop; ++i) old[i] = head->tops[j & 1][i];
  constexpr int R = kCandMax / (4 * kCandStepThreads);  // fours of candidates per thread
  uint4 now[R], taken[R], id[R], x[VECS], row_of[kCandRows];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * kCandStepThreads + tid;
    now[r] = make_uint4(kCandTaken, kCandTaken, kCandTaken, kCandTaken);
    taken[r] = id[r] = make_uint4(0u, 0u, 0u, 0u);
    if (4 * i < most) {
      now[r] = base[i];
      taken[r] = dec_prev[i];
      id[r] = node[i];
    }
  }
  if (wv == 0) {
#pragma unroll
    for (int i = 0; i < kCandRows; ++i)
      row_of[i] = reinterpret_cast<const uint4*>(head->combos[(j + 2) % 3][i])[lane];
  }
  if (picked >= (uint32_t)k || failed) {  // the same in every block
    if (blockIdx.x == 0 && tid == 0) head->picked[(j + 1) & 1] = picked;
    return;
  }
#pragma unroll
  for (int v = 0; v < VECS; ++v) {
    x[v] = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (v * kCandStepThreads + tid < nvec) x[v] = vec[v * kCandStepThreads + tid];
  }
  if (tid < kCandCombos) s_combos[tid] = 0u;
  if (tid < kCandTop) s_key[ROWS + tid] = 0ull;
  if (tid < ORDER) s_order[tid] = 0u;
  if (tid == 0) {
    s_any = 0u;
    s_open[0] = -1;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * kCandStepThreads + tid;
    if (4 * i < most) {
      reinterpret_cast<uint4*>(s_dec)[i] = make_uint4(0u, 0u, 0u, 0u);
      reinterpret_cast<uint2*>(s_cls)[i] = make_uint2(0u, 0u);
    }
  }
  uint32_t mine = 0;  // which of this thread's candidates are tops
#pragma unroll
  for (int i = 0; i < kCandTop; ++i) {
    const uint32_t f = old[i] - 1u;
    if (old[i] && (f / 4u) % (uint32_t)kCandStepThreads == (uint32_t)tid)
      mine |= 1u << (f / (4u * kCandStepThreads) * 4u + f % 4u);
  }
  lds_barrier();
  // key of a candidate: count << 32 | ~node, so the largest count, ties to the lowest node
  unsigned long long key = 0;
  uint32_t num = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    uint32_t* cv[4] = {&now[r].x, &now[r].y, &now[r].z, &now[r].w};
    const uint32_t dv[4] = {taken[r].x, taken[r].y, taken[r].z, taken[r].w};
    const uint32_t uv[4] = {id[r].x, id[r].y, id[r].z, id[r].w};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (*cv[w] == kCandTaken) continue;
      *cv[w] -= dv[w];
      const unsigned long long q = ((unsigned long long)*cv[w] << 32) | (0xFFFFFFFFull - uv[w]);
      const uint32_t me = (uint32_t)(4 * (r * kCandStepThreads + tid) + w);
      if (mine >> (4 * r + w) & 1u) {
#pragma unroll
        for (int i = 0; i < kCandTop; ++i)
          if (old[i] == me + 1u) {
            s_key[ROWS + i] = q;
            s_num[ROWS + i] = me;
          }
      } else if (q > key) {
        key = q;
        num = me;
      }
    }
  }
  {
    const unsigned long long row = row_max64(key);
    // keys differ between candidates: one lane of the row holds its best
    if (key == row && (row || tid % 16 == 0)) {
      s_key[tid / 16] = row;
      s_num[tid / 16] = num;
    }
  }
  if (wv == 0) {
    // sets by combination (lane l: 4l .. 4l + 3), then summed over the combinations within each
    uint32_t h[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < kCandRows; ++i) {
      h[0] += row_of[i].x;
      h[1] += row_of[i].y;
      h[2] += row_of[i].z;
      h[3] += row_of[i].w;
    }
    h[1] += h[0];
    h[3] += h[2];
    h[2] += h[0];
    h[3] += h[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t y = dpp32<kDppRowShr + 1>(h[i]);
      h[i] += lane & 1 ? y : 0u;
      y = dpp32<kDppRowShr + 2>(h[i]);
      h[i] += lane & 2 ? y : 0u;
      y = dpp32<kDppRowShr + 4>(h[i]);
      h[i] += lane & 4 ? y : 0u;
      y = dpp32<kDppRowShr + 8>(h[i]);
      h[i] += lane & 8 ? y : 0u;
      y = __shfl_xor(h[i], 16, 64);
      h[i] += lane & 16 ? y : 0u;
      y = __shfl_xor(h[i], 32, 64);
      h[i] += lane & 32 ? y : 0u;
    }
    reinterpret_cast<uint4*>(s_within)[lane] = make_uint4(h[0], h[1], h[2], h[3]);
  }
  lds_barrier();
  if (wv == 0) {
    const unsigned long long rows = row_max64(s_key[lane]);
    const unsigned long long bound =
        max64(max64(lane64(rows, 0), lane64(rows, 16)), max64(lane64(rows, 32), lane64(rows, 48)));
    unsigned long long in = lane < kCandTop ? s_key[ROWS + lane] : 0ull;  // lane i: top i
    unsigned long long top = lane64(row_max64(in), 0);
    int n = 0;
    if (bound >= top) {
      if (bound != 0ull && bound >= t) {
        if (s_key[lane] == bound) s_chosen[0] = s_num[lane];
        if (lane == 0 && blockIdx.x == 0) best[picked] = bound;
        n = 1;
      }
    } else {
      const uint32_t low = (uint32_t)in;
      uint32_t left = kCandCombos - 1;      // the tops not chosen
      bool is_left = in != 0ull;
      while (top > bound && top >= t && picked + (uint32_t)n < (uint32_t)k) {
        const uint64_t who = __ballot(in == top && is_left);
        const int i = __ffsll((unsigned long long)who) - 1;
        if (lane == i) {
          s_chosen[n] = s_num[ROWS + i];
          is_left = false;
        }
        if (lane == 0 && blockIdx.x == 0) best[picked + (uint32_t)n] = top;
        ++n;
        left &= ~(1u << i);
        // a top's sets left: those with none chosen, less those without this top too
        const uint32_t cnt = s_within[left] - s_within[left & ~(1u << (lane % kCandTop))];
        in = is_left ? ((unsigned long long)cnt << 32) | low : 0ull;
        top = lane64(row_max64(in), 0);
      }
    }
    if (lane == 0) s_nchosen = n;
  } else if (tid < 64 + 8 * KEYS) {
    // the order of the largest keys
    const int q = (tid - 64) / 8;
    const unsigned long long me = s_key[q];
    uint32_t larger = 0;
#pragma unroll
    for (int e = 0; e < KEYS / 8; ++e) larger += s_key[e * 8 + tid % 8] > me ? 1u : 0u;
    larger = sum8(larger);
    if (me != 0ull && larger < (uint32_t)ORDER && tid % 8 == 0) s_order[larger] = s_num[q] + 1u;
  }
  lds_barrier();
  const int n = s_nchosen;
  if (tid < 64) {
    const uint32_t o = tid < ORDER ? s_order[tid] : 0u;
    bool next = o != 0u;
    for (int q = 0; q < n; ++q) next = next && s_chosen[q] != o - 1u;
    const uint64_t all = __ballot(next);
    const int at = (int)__popcll(all & ((1ull << lane) - 1ull));
    if (next && at < kCandTop) s_cls[o - 1u] = (uint16_t)(1u << at);
    if (blockIdx.x == 0) {
      if (next && at < kCandTop) head->tops[(j + 1) & 1][at] = o;
      if (tid < kCandTop && tid >= (int)__popcll(all)) head->tops[(j + 1) & 1][tid] = 0u;
    }
  } else if (tid - 64 < n) {
    s_cls[s_chosen[tid - 64]] = (uint16_t)kCandChosen;
  }
  if (blockIdx.x == 0) {
    if (tid == 0) {
      if (n == 0) {
        best[picked] = 1ull;
        head->failed = 1u;
      }
      head->picked[(j + 1) & 1] = picked + (uint32_t)n;
    }
    for (int i = tid; i < kCandRows * kCandCombos; i += kCandStepThreads) head->combos[(j + 1) % 3][0][i] = 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = r * kCandStepThreads + tid;
      if (4 * i < most) {
        uint4 b = now[r];
        for (int q = 0; q < n; ++q) {
          const uint32_t v = s_chosen[q];
          if (v == 4u * (uint32_t)i) b.x = kCandTaken;
          if (v == 4u * (uint32_t)i + 1u) b.y = kCandTaken;
          if (v == 4u * (uint32_t)i + 2u) b.z = kCandTaken;
          if (v == 4u * (uint32_t)i + 3u) b.w = kCandTaken;
        }
        base_next[i] = b;
        dec_next[i] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
  }
  if (n == 0 || picked + (uint32_t)n >= (uint32_t)k) return;  // the last choice changes no later step
  lds_barrier();
  // of the set open at the tile's start, where there are several tiles: its classes and first entry
  uint32_t open = 0;
  int open_at = 0, turn = 0;
  for (int t0 = 0; t0 < nvec; t0 += TILE) {
    const bool ends = t0 + TILE >= nvec;
    uint32_t p[VECS], q[VECS], hits = 0;  // hits: which of the wavefront's chunks have classes
    uint4 y[VECS];
    if (!ends) {  // the next tile
#pragma unroll
      for (int v = 0; v < VECS; ++v) {
        const int i = t0 + TILE + v * kCandStepThreads + tid;
        y[v] = i < nvec ? vec[i] : make_uint4(~0u, ~0u, ~0u, ~0u);
      }
    }
#pragma unroll
    for (int v = 0; v < VECS; ++v) {
      const uint32_t word[4] = {x[v].x, x[v].y, x[v].z, x[v].w};
      uint32_t some = 0;
      p[v] = q[v] = 0u;
      if (t0 + v * kCandStepThreads + wv * 64 < nvec) {
#pragma unroll
        for (int w = 0; w < 8; ++w) {
          const uint32_t e = (word[w >> 1] >> (16 * (w & 1))) & kCandDead;
          if (e != kCandDead) some |= s_cls[e];
        }
      }
      const bool starts = ((word[0] | word[1] | word[2] | word[3]) & 0x80008000u) != 0u;
      uint32_t sum = __ballot(starts) ? kCandStarts : 0u;
      if (__ballot(some != 0u)) {
        hits |= 1u << v;
        uint32_t head = 0, acc = 0;
        bool first = true;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
          const uint32_t e = (word[w >> 1] >> (16 * (w & 1))) & 0xFFFFu;
          if (e & kCandFirst) {
            if (first) head = acc;
            first = false;
            acc = 0;
          }
          if ((e & kCandDead) != kCandDead) acc |= s_cls[e & kCandDead];
        }
        if (first) head = acc;
        scan_classes(head, acc, starts, lane, &p[v], &q[v]);
        sum |= (uint32_t)__builtin_amdgcn_readlane((int)q[v], 0) |
               (uint32_t)__builtin_amdgcn_readlane((int)p[v], 63) << 12;
      }
      if (lane == 0) s_chunk[v * NW + wv] = sum;
    }
    lds_barrier();
    const uint32_t sum = s_chunk[lane];
    uint32_t cp, cq;
    scan_classes(sum & 0xFFFu, (sum >> 12) & 0xFFFu, (sum & kCandStarts) != 0u, lane, &cp, &cq);
    const uint64_t cstarts = __ballot((sum & kCandStarts) != 0u);
    // the set from before the tile reaches into it, the last one perhaps out of it
    const bool in_first = !(cstarts & (~0ull >> (63 - lane)));  // no start up to this chunk's end
    const bool to_last = !(cstarts & (~0ull << lane));          // no start from this chunk on
    if (in_first) cp |= open;
    if (to_last && !ends) cq |= kCandOpen;
#pragma unroll
    for (int v = 0; v < VECS; ++v) {
      const int ch = v * NW + wv;
      const uint32_t in = ch ? (uint32_t)__builtin_amdgcn_readlane((int)cp, ch ? ch - 1 : 0) : open;
      const uint32_t out = ch < 63 ? (uint32_t)__builtin_amdgcn_readlane((int)cq, ch < 63 ? ch + 1 : 63)
                                   : (ends ? 0u : kCandOpen);
      const bool hit = (hits >> v & 1u) != 0u;
      if (!hit && !(in & kCandChosen) && !(out & ~kCandOpen)) continue;
      const uint32_t word[4] = {x[v].x, x[v].y, x[v].z, x[v].w};
      const bool starts = ((word[0] | word[1] | word[2] | word[3]) & 0x80008000u) != 0u;
      const uint64_t all = __ballot(starts);
      uint32_t before = __shfl_up(p[v], 1, 64), after = __shfl_down(q[v], 1, 64);  // of the sets open at the lane's ends
      if (lane == 0) before = 0u;
      if (lane == 63) after = 0u;
      if (!(all & ((1ull << lane) - 1ull))) before |= in;
      if (lane == 63 || !(all & (~0ull << (lane + 1)))) after |= out;
      uint32_t kill = 0, acc = 0, seg = 0;
      bool last = true;
#pragma unroll
      for (int w = 7; w >= 0; --w) {
        const uint32_t e = (word[w >> 1] >> (16 * (w & 1))) & 0xFFFFu;
        if ((e & kCandDead) != kCandDead) {
          acc |= s_cls[e & kCandDead];
          seg |= 1u << w;
        }
        if (e & kCandFirst) {
          if (last) acc |= after;
          last = false;
          if (!(acc & kCandOpen)) {
            if (acc & kCandChosen) kill |= seg;
            else if (acc) atomicAdd(&s_combos[acc], 1u);
          }
          acc = seg = 0;
        }
      }
      acc |= before;
      if (last) acc |= after;
      if ((acc & kCandChosen) && !(acc & kCandOpen)) kill |= seg;
      s_any = 1u;
      if (__ballot(kill != 0u)) {
        uint32_t dead[4] = {x[v].x, x[v].y, x[v].z, x[v].w};
#pragma unroll
        for (int w = 0; w < 8; ++w) {
          if (kill >> w & 1u) {
            atomicAdd(&s_dec[(word[w >> 1] >> (16 * (w & 1))) & kCandDead], 1u);
            dead[w >> 1] |= kCandDead << (16 * (w & 1));
          }
        }
        if (kill) vec[t0 + v * kCandStepThreads + tid] = make_uint4(dead[0], dead[1], dead[2], dead[3]);
      }
    }
    if (ends && t0 == 0) break;
    // several tiles: the set that was open before this one, where it ends here, and the one open after it
    const uint32_t total = open | (uint32_t)__builtin_amdgcn_readlane((int)cq, 0);
    if (t0 && total && !(total & kCandOpen)) {
      if (total & kCandChosen) {
        __syncthreads();  // the stores of earlier tiles are done
        for (int i = open_at + tid; i < t0 * 8; i += kCandStepThreads) {
          const uint32_t e = part[i];
          if ((e & kCandDead) != kCandDead) {
            atomicAdd(&s_dec[e & kCandDead], 1u);
            part[i] = (uint16_t)(e | kCandDead);
          }
        }
      } else if (tid == 0) {
        atomicAdd(&s_combos[total], 1u);
      }
      s_any = 1u;
    }
    if (ends) break;
    bool found = false;
#pragma unroll
    for (int v = VECS - 1; v >= 0; --v) {
      const uint32_t word[4] = {x[v].x, x[v].y, x[v].z, x[v].w};
      int w_last = -1;
#pragma unroll
      for (int w = 0; w < 8; ++w)
        if ((word[w >> 1] >> (16 * (w & 1))) & kCandFirst) w_last = w;
      const uint64_t all = __ballot(w_last >= 0);
      if (all && !found && lane == 63 - __clzll((long long)all))
        atomicMax(&s_open[turn], (t0 + v * kCandStepThreads + tid) * 8 + w_last);
      found = found || all;
    }
    if (tid == 0) s_open[turn ^ 1] = -1;
    lds_barrier();
    open = (uint32_t)__builtin_amdgcn_readlane((int)cp, 63);
    if (s_open[turn] >= 0) open_at = s_open[turn];
    turn ^= 1;
#pragma unroll
    for (int v = 0; v < VECS; ++v) x[v] = y[v];
  }
  __syncthreads();
  if (!s_any) return;
  for (int i = tid; i < most; i += kCandStepThreads)
    if (s_dec[i]) atomicAdd(&dec_now[i], s_dec[i]);
  if (tid < kCandCombos && s_combos[tid])
    atomicAdd(&head->combos[j % 3][blockIdx.x % kCandRows][tid], s_combos[tid]);
}

unsigned grid_for(uint64_t items, unsigned cap) {
  uint64_t g = (items + kThreads - 1) / kThreads;
  if (g < 1) g = 1;
  return (unsigned)(g > cap ? cap : g);
}

}  // namespace

size_t scan_temp_bytes(uint64_t len) { return ((len + kTile - 1) / kTile + 1) * sizeof(unsigned long long); }

void launch_scan_u32_to_i64(const uint32_t* in, int64_t* out, uint64_t len, void* temp, hipStream_t s) {
  const uint64_t ntiles = (len + kTile - 1) / kTile;
  unsigned long long* ts = static_cast<unsigned long long*>(temp);
  if (ntiles) hipLaunchKernelGGL(scan_tile_sums, dim3((unsigned)ntiles), dim3(kThreads), 0, s, in, len, ts);
  hipLaunchKernelGGL(scan_tile_offsets, dim3(1), dim3(kThreads), 0, s, ts, ntiles, out, len);
  if (ntiles) hipLaunchKernelGGL(scan_apply, dim3((unsigned)ntiles), dim3(kThreads), 0, s, in, len, ts, out);
}

void launch_compact(const int32_t* pool, const uint64_t* set_start, const uint32_t* set_len, const int64_t* out_off,
                    int32_t* out_nodes, uint64_t nsets, hipStream_t s) {
  if (!nsets) return;
  hipLaunchKernelGGL(compact_kernel, dim3(grid_for(nsets, 8192)), dim3(kThreads), 0, s, pool, set_start, set_len,
                     out_off, out_nodes, nsets);
}

void launch_check_ids(const int32_t* nodes, uint64_t total, int64_t n, unsigned int* flag, hipStream_t s) {
  hipLaunchKernelGGL(zero_u32, dim3(1), dim3(64), 0, s, flag, (uint64_t)1);
  if (total)
    hipLaunchKernelGGL(check_ids_kernel, dim3(grid_for(total, 4096)), dim3(kThreads), 0, s, nodes, total, n, flag);
}

void launch_set_sizes(const int64_t* set_off, uint32_t* sizes, uint64_t nsets, hipStream_t s) {
  if (!nsets) return;
  hipLaunchKernelGGL(set_sizes_kernel, dim3(grid_for(nsets, 8192)), dim3(kThreads), 0, s, set_off, sizes, nsets);
}

namespace {

CsrSets csr_of(const GreedyArgs& a) { return CsrSets{a.set_off, a.nodes}; }
PoolSets pool_of(const GreedyArgs& a) { return PoolSets{a.set_start, a.set_len, a.nodes}; }

unsigned tile_grid(uint64_t items, uint64_t per_tile) {
  return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((items + per_tile - 1) / per_tile, 8192));
}

}  // namespace

// ---- the counting sort's workspace ----
namespace {

int bucket_shift(int64_t n) {
  int shift = kBucketShiftMin;
  while (shift <= kBucketShiftMax && ((n + (1ll << shift) - 1) >> shift) > kBucketMax) ++shift;
  return shift;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct BucketLayout {
  int shift = 0, nb = 0;
  uint64_t max_chunks = 0;
  size_t bcnt = 0, bcnt_s = 0, bfill = 0, boff = 0, cstart = 0, cb = 0, temp = 0, bu = 0, bs = 0, bytes = 0;
};

// Offsets of the workspace's arrays; bytes == 0 where the collection does not
// fit the counting sort (node ids beyond its ranges, 2^32 entries or more).
BucketLayout bucket_layout(int64_t n, uint64_t total, bool index) {
  BucketLayout L;
  L.shift = bucket_shift(n);
  if (L.shift > kBucketShiftMax || total >= 0xFFFFFFFFull || n < 1) return L;
  L.nb = (int)((n + (1ll << L.shift) - 1) >> L.shift);
  L.max_chunks = (uint64_t)L.nb + total / kBucketChunk + 1;
  size_t at = 0;
  L.bcnt = at;
  at += align256((size_t)L.nb * 4);
  L.bcnt_s = at;
  at += align256((size_t)L.nb * 4 * kLinePad);
  L.bfill = at;
  at += align256((size_t)L.nb * 4 * kLinePad);
  L.boff = at;
  at += align256((size_t)(L.nb + 1) * 8);
  L.cstart = at;
  at += align256((size_t)(L.nb + 1) * 4);
  L.cb = at;
  at += align256((size_t)L.max_chunks * 4);
  L.temp = at;
  at += align256(scan_temp_bytes((uint64_t)L.nb));
  L.bu = at;
  at += align256((size_t)total * 4);
  L.bs = at;
  if (index) at += align256((size_t)total * 4);
  L.bytes = at;
  return L;
}

template <class T>
T* at_offset(void* base, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(base) + off);
}

// Sorts the entries into buckets and counts them (cnt zeroed first); with
// `index`, leaves the set ids beside them for bucket_index_kernel.
template <class V>
void bucket_counts(const GreedyArgs& a, V sets, const BucketLayout& L, bool index, hipStream_t s) {
  uint32_t* bcnt = at_offset<uint32_t>(a.bkt, L.bcnt);
  uint32_t* bcnt_s = at_offset<uint32_t>(a.bkt, L.bcnt_s);
  int64_t* boff = at_offset<int64_t>(a.bkt, L.boff);
  uint32_t* cstart = at_offset<uint32_t>(a.bkt, L.cstart);
  uint32_t* cb = at_offset<uint32_t>(a.bkt, L.cb);
  uint32_t* bu = at_offset<uint32_t>(a.bkt, L.bu);
  uint32_t* bs = index ? at_offset<uint32_t>(a.bkt, L.bs) : nullptr;
  // the padded counts and cursors are adjacent: one clear; the scan reads the counts unpadded
  const uint64_t zlen = (uint64_t)(L.bfill - L.bcnt_s) / 4 + (uint64_t)L.nb * kLinePad;
  hipLaunchKernelGGL(zero_u32, dim3(grid_for(zlen, 64)), dim3(kThreads), 0, s, bcnt_s, zlen);
  // tiles of as many sets as leave each block one, at most one per thread
  const int ts = (int)std::min<uint64_t>(kSortThreads, std::max<uint64_t>(64, a.nsets / kSortBlocks + 1));
  const unsigned grid = (unsigned)std::min<uint64_t>(kSortBlocks, (a.nsets + (uint64_t)ts - 1) / (uint64_t)ts);
  hipLaunchKernelGGL((bucket_sort_kernel<V, kSortCount>), dim3(grid), dim3(kSortThreads), 0, s, sets, a.nsets, ts,
                     L.shift, L.nb, nullptr, bcnt_s, nullptr, nullptr);
  hipLaunchKernelGGL(unpad_u32, dim3(grid_for((uint64_t)L.nb, 64)), dim3(kThreads), 0, s, bcnt_s, bcnt, L.nb);
  launch_scan_u32_to_i64(bcnt, boff, (uint64_t)L.nb, at_offset<void>(a.bkt, L.temp), s);
  hipLaunchKernelGGL(bucket_chunks_kernel, dim3(1), dim3(kThreads), 0, s, boff, L.nb, cstart, cb);
  uint32_t* bfill = at_offset<uint32_t>(a.bkt, L.bfill);
  if (index)
    hipLaunchKernelGGL((bucket_sort_kernel<V, kSortMoveIds>), dim3(grid), dim3(kSortThreads), 0, s, sets, a.nsets, ts,
                       L.shift, L.nb, boff, bfill, bu, bs);
  else
    hipLaunchKernelGGL((bucket_sort_kernel<V, kSortMove>), dim3(grid), dim3(kSortThreads), 0, s, sets, a.nsets, ts,
                       L.shift, L.nb, boff, bfill, bu, bs);
  hipLaunchKernelGGL(bucket_count_kernel, dim3((unsigned)L.max_chunks), dim3(kCountThreads), 0, s, bu, boff, cstart, cb,
                     L.nb, L.shift, a.n, a.cnt);
}


// ---- the candidate greedy's workspace ----
struct CandLayout {
  size_t head = 0, bins = 0, dec = 0, base = 0, node = 0, seg = 0, map = 0, stream = 0, bytes = 0;
};

CandLayout cand_layout(int64_t n, uint64_t total) {
  CandLayout L;
  size_t at = 0;
  L.head = at;
  at += align256(sizeof(CandHead));
  L.bins = at;
  at += (size_t)kCandBins * 4;
  L.dec = at;
  at += (size_t)kCandMax * 4 * 3;
  L.base = at;
  at += (size_t)kCandMax * 4 * 2;
  L.node = at;
  at += (size_t)kCandMax * 4;
  L.seg = at;
  at += (size_t)kCandSegs * 4 * 2;
  L.map = at;
  at += align256((size_t)n * 2);
  L.stream = at;
  at += align256(((size_t)total + 64 * (size_t)kCandSegs) * 2);
  L.bytes = at;
  return L;
}

CandArrays cand_arrays(const GreedyArgs& a) {
  const CandLayout L = cand_layout(a.n, a.total);
  CandArrays c;
  c.head = at_offset<CandHead>(a.bkt, L.head);
  c.bins = at_offset<uint32_t>(a.bkt, L.bins);
  c.dec = at_offset<uint32_t>(a.bkt, L.dec);
  c.base = at_offset<uint32_t>(a.bkt, L.base);
  c.node = at_offset<uint32_t>(a.bkt, L.node);
  c.seg_start = at_offset<uint32_t>(a.bkt, L.seg);
  c.seg_len = c.seg_start + kCandSegs;
  c.map = at_offset<uint16_t>(a.bkt, L.map);
  c.stream = at_offset<uint16_t>(a.bkt, L.stream);
  // at least 1024 entries per part: smaller collections are bound by their steps' latency, not by the parts' work
  c.segs = (int)std::max<uint64_t>(1, std::min<uint64_t>(kCandSegs, a.total / 1024));
  return c;
}

// The candidate greedy runs where it has its workspace and its positions fit
// 32 bits, for 2 to kCandMaxSteps steps (a.k; 0 where the steps are launched
// one by one), unless it has failed on this collection (a.all_nodes).
bool use_candidates(const GreedyArgs& a) {
  return a.bkt && a.k > 1 && a.k <= kCandMaxSteps && !a.all_nodes && a.nsets && a.total &&
         a.total + 64ull * kCandSegs < 0xFFFFFFFFull && bucket_layout(a.n, a.total, true).bytes;
}

int cand_most(const GreedyArgs& a) { return std::min(kCandMax, std::max(kCandMin, kCandPerStep * a.k)); }

template <class V>
void cand_prepare(const GreedyArgs& a, V sets, hipStream_t s) {
  const CandArrays c = cand_arrays(a);
  hipLaunchKernelGGL(cand_init_kernel, dim3(16), dim3(kThreads), 0, s, c, a.best, a.k);
  const unsigned grid = grid_for((uint64_t)a.n, 256);
  const int most = cand_most(a);
  // the nodes of small counts per block lie where the stream is built after that (it has 64 entries per part to spare)
  static_assert((size_t)kThreads * kCandTies * 4 <= 64 * (size_t)kCandSegs * 2, "a grid of kThreads blocks fits");
  uint32_t* ties = reinterpret_cast<uint32_t*>(c.stream);
  if (a.n > most) hipLaunchKernelGGL(cand_bins_kernel, dim3(grid), dim3(kThreads), 0, s, a.cnt, a.n, c.bins, ties);
  hipLaunchKernelGGL(cand_pick_kernel, dim3(grid), dim3(kThreads), 0, s, a.cnt, a.n, (uint32_t)most, ties, c);
  // tiles of about two windows' entries, at least one per block
  const uint64_t mean = a.total / a.nsets + 1;
  const uint64_t ts = std::min<uint64_t>(2 * kCandWindow / mean, a.nsets / (uint64_t)c.segs + 1);
  hipLaunchKernelGGL(cand_build_kernel<V>, dim3((unsigned)c.segs), dim3(kCandBuildThreads), 0, s, sets, a.nsets,
                     (int)std::min<uint64_t>(kCandTileMax, std::max<uint64_t>(16, ts)), c);
}

}  // namespace

size_t bucket_workspace_bytes(int64_t n, uint64_t total, bool index) {
  const size_t b = bucket_layout(n, total, index).bytes;
  // the candidate arrays take the sort's place once the counts are done
  return b && index ? std::max(b, cand_layout(n, total).bytes) : b;
}

void launch_counts(const GreedyArgs& a, hipStream_t s) {
  const uint64_t n = (uint64_t)a.n;
  hipLaunchKernelGGL(zero_u32, dim3(grid_for(n, 4096)), dim3(kThreads), 0, s, a.cnt, n);
  if (!a.nsets) return;
  if (a.bkt && a.total > kDirectCounts) {
    const BucketLayout L = bucket_layout(a.n, a.total, false);
    if (L.bytes) {
      if (a.set_off) bucket_counts(a, csr_of(a), L, false, s);
      else bucket_counts(a, pool_of(a), L, false, s);
      return;
    }
  }
  if (a.set_off) {
    if (a.total)
      hipLaunchKernelGGL(hist_flat_kernel, dim3(tile_grid(a.total, kTileEntries)), dim3(kThreads), 0, s, a.set_off,
                         a.nodes, a.total, a.cnt);
  } else {
    hipLaunchKernelGGL(hist_sets_kernel<PoolSets>, dim3(tile_grid(a.nsets, kHistTileSets)), dim3(kThreads), 0, s,
                       pool_of(a), a.nsets, a.cnt);
  }
}

void launch_index(const GreedyArgs& a, hipStream_t s) {
  const uint64_t n = (uint64_t)a.n;
  if (use_candidates(a)) {
    launch_counts(a, s);
    if (a.set_off) cand_prepare(a, csr_of(a), s);
    else cand_prepare(a, pool_of(a), s);
    return;
  }
  if (a.bkt && a.nsets && a.total) {
    const BucketLayout L = bucket_layout(a.n, a.total, true);
    if (L.bytes) {
      hipLaunchKernelGGL(zero_u32, dim3(grid_for(n, 4096)), dim3(kThreads), 0, s, a.cnt, n);
      if (a.set_off) bucket_counts(a, csr_of(a), L, true, s);
      else bucket_counts(a, pool_of(a), L, true, s);
      hipLaunchKernelGGL(zero_u32, dim3(grid_for(n, 4096)), dim3(kThreads), 0, s, a.fill, n);
      launch_scan_u32_to_i64(a.cnt, a.inv_off, n, a.scan_temp, s);
      hipLaunchKernelGGL(bucket_index_kernel, dim3((unsigned)L.max_chunks), dim3(kThreads), 0, s,
                         at_offset<uint32_t>(a.bkt, L.bu), at_offset<uint32_t>(a.bkt, L.bs),
                         at_offset<int64_t>(a.bkt, L.boff), at_offset<uint32_t>(a.bkt, L.cstart),
                         at_offset<uint32_t>(a.bkt, L.cb), L.nb, L.shift, a.n, a.inv_off, a.fill, a.inv_sets);
      return;
    }
  }
  launch_counts(a, s);
  hipLaunchKernelGGL(zero_u32, dim3(grid_for(n, 4096)), dim3(kThreads), 0, s, a.fill, n);
  launch_scan_u32_to_i64(a.cnt, a.inv_off, n, a.scan_temp, s);
  if (!a.nsets) return;
  const unsigned grid = tile_grid(a.nsets, kTileSets);
  if (a.set_off)
    hipLaunchKernelGGL(scatter_kernel<CsrSets>, dim3(grid), dim3(kThreads), 0, s, csr_of(a), a.nsets, a.inv_off,
                       a.fill, a.inv_sets);
  else
    hipLaunchKernelGGL(scatter_kernel<PoolSets>, dim3(grid), dim3(kThreads), 0, s, pool_of(a), a.nsets, a.inv_off,
                       a.fill, a.inv_sets);
}

void launch_zero_counts(uint32_t* cnt, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(zero_u32, dim3(grid_for((uint64_t)n, 4096)), dim3(kThreads), 0, s, cnt, (uint64_t)n);
}

void launch_greedy_init(const GreedyArgs& a, uint64_t covered_len, int k, hipStream_t s) {
  const uint64_t n = (uint64_t)a.n;
  if (covered_len)
    hipLaunchKernelGGL(zero_u8, dim3(grid_for(covered_len, 4096)), dim3(kThreads), 0, s, a.covered, covered_len);
  hipLaunchKernelGGL(zero_u8, dim3(grid_for(n, 4096)), dim3(kThreads), 0, s, a.selected, n);
  hipLaunchKernelGGL(zero_u64, dim3(1), dim3(kThreads), 0, s, a.best, (uint64_t)k);
}

namespace {
void launch_argmax(const GreedyArgs& a, int j, hipStream_t s) {
  const uint64_t n4 = ((uint64_t)a.n + 3) / 4;
  hipLaunchKernelGGL(argmax_kernel, dim3(grid_for(n4, 256)), dim3(kThreads), 0, s, a.cnt, a.selected, a.n,
                     a.best + j);
}
}  // namespace

void launch_argmax_step(const GreedyArgs& a, int j, hipStream_t s) {
  launch_argmax(a, j, s);
  hipLaunchKernelGGL(select_kernel, dim3(1), dim3(64), 0, s, a.best + j, a.selected);
}

void launch_cover_step(const GreedyArgs& a, int j, hipStream_t s) {
  if (!a.nsets) {
    // nothing to cover, but the choice must still leave the candidates
    hipLaunchKernelGGL(select_kernel, dim3(1), dim3(64), 0, s, a.best + j, a.selected);
    return;
  }
  // the chosen node's list holds at most nsets sets: no more blocks than its tiles
  const dim3 grid((unsigned)std::min<uint64_t>(1024, (a.nsets + kTileSets - 1) / kTileSets));
  if (a.set_off)
    hipLaunchKernelGGL(cover_kernel<CsrSets>, grid, dim3(kThreads), 0, s, a.best + j, a.inv_off, a.inv_sets,
                       csr_of(a), a.covered, a.selected, a.cnt);
  else
    hipLaunchKernelGGL(cover_kernel<PoolSets>, grid, dim3(kThreads), 0, s, a.best + j, a.inv_off, a.inv_sets,
                       pool_of(a), a.covered, a.selected, a.cnt);
}

void launch_pool_hist(const int32_t* pool, const uint64_t* set_start, const uint32_t* set_len, uint64_t nsets,
                      uint32_t* cnt, hipStream_t s) {
  if (!nsets) return;
  hipLaunchKernelGGL(hist_sets_kernel<PoolSets>, dim3(tile_grid(nsets, kHistTileSets)), dim3(kThreads), 0, s,
                     PoolSets{set_start, set_len, pool}, nsets, cnt);
}

void launch_pool_cover(const unsigned long long* best, const int32_t* pool, const uint64_t* set_start,
                       const uint32_t* set_len, uint64_t nsets, uint8_t* covered, uint32_t* cnt, hipStream_t s) {
  if (!nsets) return;
  hipLaunchKernelGGL(scan_cover_kernel, dim3(tile_grid(nsets, kTileSets)), dim3(kThreads), 0, s, best,
                     PoolSets{set_start, set_len, pool}, nsets, covered, cnt);
}

// ---- a greedy that allocates nothing ----
//
// For callers that cannot allocate device memory (under HIP graph capture, in
// serving loops), the greedy's work arrays can live in one fixed device array
// instead of context buffers.  Each GPU holds its own copy at its own
// address, found once per device with hipGetSymbolAddress; in host code the
// array's name is not a device address, so only that address is ever used.
namespace {
constexpr size_t kStaticCnt = 0;                                             // uint32 [kStaticMaxN]
constexpr size_t kStaticFill = kStaticCnt + 4 * kStaticMaxN;                 // uint32 [kStaticMaxN]
constexpr size_t kStaticInvOff = kStaticFill + 4 * kStaticMaxN;              // int64 [kStaticMaxN + 1]
constexpr size_t kStaticInvSets = kStaticInvOff + 8 * (kStaticMaxN + 64);   // uint32 [kStaticMaxEntries]
constexpr size_t kStaticCovered = kStaticInvSets + 4 * kStaticMaxEntries;    // uint8 [kStaticMaxSets]
constexpr size_t kStaticSelected = kStaticCovered + kStaticMaxSets;          // uint8 [kStaticMaxN]
constexpr size_t kStaticBest = kStaticSelected + kStaticMaxN;                // uint64 [kStaticMaxK]
constexpr size_t kStaticMisc = kStaticBest + 8 * kStaticMaxK;                // id-check flag, an empty CSR offset
constexpr size_t kStaticScan = kStaticMisc + 256;                            // scan tile sums
constexpr size_t kStaticBytes = kStaticScan + ((kStaticMaxN + 1 + kTile - 1) / kTile + 1) * 8 + 256;
static_assert(kStaticInvSets % 256 == 0 && kStaticBest % 8 == 0, "alignment");

__device__ __align__(256) unsigned char scratch[kStaticBytes];

std::mutex g_static_mu;
void* g_static_ptr[kStaticMaxDevices] = {};

__global__ void set_u64_kernel(unsigned long long* p, unsigned long long v) {
  if (threadIdx.x == 0) *p = v;
}
}  // namespace

size_t static_scratch_bytes() { return kStaticBytes; }

hipError_t static_scratch_init(int device) {
  if (device < 0 || device >= kStaticMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_static_mu);
  if (g_static_ptr[device]) return hipSuccess;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_static_ptr[device] = ptr;
  return hipSuccess;
}

StaticGreedy static_greedy_layout(int device) {
  StaticGreedy st;
  memset(&st, 0, sizeof(st));
  void* base = nullptr;
  if (device >= 0 && device < kStaticMaxDevices) {
    std::lock_guard<std::mutex> lk(g_static_mu);
    base = g_static_ptr[device];
  }
  if (!base) return st;
  unsigned char* b = static_cast<unsigned char*>(base);
  st.cnt = reinterpret_cast<uint32_t*>(b + kStaticCnt);
  st.fill = reinterpret_cast<uint32_t*>(b + kStaticFill);
  st.inv_off = reinterpret_cast<int64_t*>(b + kStaticInvOff);
  st.inv_sets = reinterpret_cast<uint32_t*>(b + kStaticInvSets);
  st.covered = b + kStaticCovered;
  st.selected = b + kStaticSelected;
  st.best = reinterpret_cast<unsigned long long*>(b + kStaticBest);
  st.flag = reinterpret_cast<unsigned int*>(b + kStaticMisc);
  st.zero_off = reinterpret_cast<int64_t*>(b + kStaticMisc + 8);
  st.scan_temp = b + kStaticScan;
  return st;
}

void launch_set_u64(unsigned long long* p, unsigned long long v, hipStream_t s) {
  hipLaunchKernelGGL(set_u64_kernel, dim3(1), dim3(64), 0, s, p, v);
}

void launch_greedy(const GreedyArgs& a, int k, hipStream_t s) {
  if (use_candidates(a)) {
    const CandArrays c = cand_arrays(a);
    for (int j = a.launched; j < a.launched + a.launches; ++j)
      hipLaunchKernelGGL(cand_step_kernel, dim3((unsigned)c.segs), dim3(kCandStepThreads), 0, s, c, cand_most(a), j, k,
                         a.best);
    return;
  }
  launch_greedy_init(a, a.nsets, k, s);
  for (int j = 0; j < k; ++j) {
    launch_argmax(a, j, s);
    // the last choice changes no later step: its cover pass is skipped
    if (j + 1 < k) launch_cover_step(a, j, s);
  }
}

}  // namespace tim
