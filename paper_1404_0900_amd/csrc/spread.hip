// Spread evaluation by forward Monte-Carlo runs: E[I(S)] in the live-edge view
// of Section 2.2, estimated as the paper's experiments do it (Section 7) by
// the mean spread over independent runs.  Run r is the live-edge world of
// phase 65 and set id r: IC edge e is live iff its coin word (kind 1, group
// e >> 2, word e & 3) is at most its threshold, and in LT node v's live
// in-edge is the one its pick draw (kind 2, index v) selects, and under the
// general triggering model v's live in-edges are the set its draw of kind 3
// selects - the same rules the RR-set samplers use (pick.hpp).  A run's spread is the number of nodes
// reachable from S along live edges, found by a forward BFS over the graph's
// out-edge lists (built once from the in-CSR and kept with the graph).
#include <algorithm>

#include "engine.hpp"
#include "pick.hpp"
#include "rng.hpp"

namespace tim {
namespace {

constexpr int kThreads = 256;
constexpr int kWave = 64;
constexpr uint32_t kPhaseEval = 65;
constexpr int kSpreadMaxWords = 37 * 1024;  // largest LDS bitmap of visited nodes: 148 KB of the CU's 160

__global__ void out_count_kernel(const int32_t* src, int64_t m, uint32_t* cnt) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += stride) atomicAdd(&cnt[src[e]], 1u);
}

// In-edge e (into v, the largest node with in_off[v] <= e) joins the out-list
// of its source as (v, e); the order inside an out-list is not defined.
__global__ void out_scatter_kernel(const int64_t* in_off, const int32_t* src, int64_t n, int64_t m,
                                   const int64_t* out_off, uint32_t* fill, int32_t* out_dst, uint32_t* out_eid) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += stride) {
    int64_t lo = 0, hi = n - 1;
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) >> 1;
      if (in_off[mid] <= e) lo = mid;
      else hi = mid - 1;
    }
    const int32_t u = src[e];
    const int64_t pos = out_off[u] + (int64_t)atomicAdd(&fill[u], 1u);
    out_dst[pos] = (int32_t)lo;
    out_eid[pos] = (uint32_t)e;
  }
}

__device__ __forceinline__ unsigned long long wave_incl_scan64(unsigned long long x, int lane) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const unsigned long long y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  return x;
}

// IC threshold of in-edge e of v: its own where the graph has thresholds, else
// floor(2^32 / indeg(v)) - 1 (x at most that is the coin test of pick.hpp).
__device__ __forceinline__ uint32_t ic_threshold(const GraphView& g, int32_t v, uint32_t e) {
  return g.thr ? g.thr[e] : (uint32_t)((1ull << 32) / (uint64_t)(g.off32[v + 1] - g.off32[v]) - 1ull);
}

__global__ void out_thr_kernel(GraphView g, const int32_t* out_dst, const uint32_t* out_eid, uint32_t* out_thr) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < g.m; x += stride)
    out_thr[x] = ic_threshold(g, out_dst[x], out_eid[x]);
}

// Is in-edge e of v live in the run's world?  (t: its IC threshold.)  LT asks
// whether v's draw picks e, without searching v's list: with cumulative
// thresholds e is the first edge at or above the draw iff it is at or above it
// and the edge before it in v's list, if any, is below.
template <int MODEL>
__device__ __forceinline__ bool out_edge_live(const GraphView& g, const Key& key, const SetStream& st, int32_t v,
                                              uint32_t e, uint32_t t) {
  if (MODEL == 0) {
    const uint4 c = draw(key, st, kKindCoin, (uint64_t)(e >> 2));
    const uint32_t lo = (e & 1u) ? c.y : c.x, hi = (e & 1u) ? c.w : c.z;
    return ((e & 2u) ? hi : lo) <= t;
  } else if (MODEL == 2) {
    // general triggering: e is live iff it belongs to the set v draws
    const int64_t iv = g.off[v];
    const int64_t j = trig_pick(g, key, st, v);
    bool live = false;
    if (j >= 0)
      for (int64_t i = g.tset[j]; i < g.tset[j + 1]; ++i) live = live || iv + (int64_t)g.tmem[i] == (int64_t)e;
    return live;
  } else {
    const uint32_t iv = g.off32[v];
    if (!g.lthr) {
      const uint32_t d = g.off32[v + 1] - iv;
      return iv + (uint32_t)scale64(draw(key, st, kKindPick, (uint64_t)v), (uint64_t)d) == e;
    }
    const uint32_t x = draw(key, st, kKindPick, (uint64_t)v).x;
    return x <= g.lthr[e] && (e == iv || x > g.lthr[e - 1u]);
  }
}

// One block of T threads per slot; the block takes runs from a counter until
// they run out.  A run's visited nodes are a bitmap of WORDS words in LDS
// where n fits (the chip's runs then touch memory only for the out-lists and
// their queues), else stamps in device memory (WORDS = 0).
//
// What bounds it: one Philox block per out-edge of a reached node whose head is
// not visited yet (about 480 issue cycles per 64 edges).  The T queued nodes of
// a batch share their out-edges evenly whatever their degrees: in windows of
// 16 T edges, the first edge of every node sets a mark in an LDS bit array, and
// a lane finds its edge's node by counting the marks up to it (a 64-bit word per
// wavefront and 64 edges, plus the marks before it) instead of a binary search
// over the nodes.  Each lane loads kSpreadLoads edges before it decides them.
// The kernel before this one (256 threads, stamps, binary search, in-degree
// gathered per edge) took 139 ms for 1000 runs of 50 seeds on a 1M-node /
// 10M-edge graph under IC and 25.3 ms for 4000 runs of 10 seeds on 50K nodes
// under LT; this one takes 31.7 and 6.6 ms.  One, two or eight loads per lane
// instead of four change that by 1 to 8%.
constexpr int kSpreadLoads = 4;

// A bitmap of more than 8192 words leaves a CU one or two blocks, and a run of a
// few nodes, a chain of latencies, keeps a block as long as it takes whatever the
// block's size: 20000 LT runs of one seed (3.8 nodes each) on 1M nodes took 0.36
// ms with four blocks of stamps per CU and 0.64 ms with one bitmap.  Runs on such
// graphs therefore start with stamps (pass 1), and one that visits more than
// kSpreadFewNodes nodes besides its seeds, or is about to take more than
// kSpreadFewEdges out-edges at once, goes to a list for the bitmap (pass 2): the
// runs above take 0.37 ms, 50000 runs of one seed on 400K nodes 0.66 (0.66 with
// stamps, 0.83 with the bitmap), 1000 runs of 50 hubs on 1M nodes 31.4 (139 and
// 31.3), 1000 runs of 50 random seeds (200 nodes) 0.53 (2.8 and 0.49).  With 256
// nodes or 4096 edges the last become 0.57, with 256 edges 5000 runs of 53 nodes
// take 0.33 instead of 0.15.
constexpr uint32_t kSpreadFewNodes = 64, kSpreadFewEdges = 1024;

// PASS: 0: all runs here; 1: large runs go to the list; 2: the runs are those of the list.
template <int MODEL, int WORDS, int T, int PASS>
__global__ __launch_bounds__(T) void spread_kernel(SpreadArgs a) {
  constexpr int NW = T / kWave;
  constexpr uint32_t W = 16u * T;    // edges per window
  constexpr int NC = W / kWave;      // 64-edge chunks per window
  constexpr int CPL = NC / kWave;    // chunks per lane of the wavefront that counts marks
  __shared__ uint32_t s_bits[WORDS ? WORDS : 1];
  __shared__ uint32_t s_delta[T];                   // by rank among the batch's nodes with out-edges: list start - first edge number
  __shared__ unsigned long long s_marks[NC];        // window: bit set where a node's edges start
  __shared__ uint32_t s_rank[NC];                   // marks before each chunk, over the whole batch
  __shared__ unsigned long long s_wtot[NW];
  __shared__ unsigned long long s_idx;
  __shared__ uint32_t s_tail, s_epoch, s_seen;
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const GraphView g = a.g;
  const Key key = make_key(a.seed);
  const int slot = blockIdx.x;
  uint32_t* stamp = WORDS ? nullptr : a.stamp + (size_t)slot * (size_t)a.stride;
  int32_t* queue = a.queue + (size_t)slot * (size_t)a.stride;
  const int nwords = WORDS ? (int)((g.n + 31) >> 5) : 0;  // at most WORDS (launch_spread)
  const uint64_t upto = ~0ull >> (63 - lane);             // lanes up to this one
  const unsigned long long todo = PASS == 2 ? min(a.ctr[2], (unsigned long long)a.list_cap) : a.runs;
  unsigned long long total = 0;
  uint32_t ep = 0;

  auto seen = [&](int32_t u) -> bool {
    if (WORDS) return (s_bits[(uint32_t)u >> 5] >> ((uint32_t)u & 31u)) & 1u;
    return stamp[u] == ep;
  };
  auto visit = [&](int32_t u) -> bool {  // true the first time
    if (WORDS) {
      const uint32_t b = 1u << ((uint32_t)u & 31u);
      return (atomicOr(&s_bits[(uint32_t)u >> 5], b) & b) == 0u;
    }
    return atomicExch(&stamp[u], ep) != ep;
  };

  for (;;) {
    if (tid == 0) {
      s_idx = atomicAdd(&a.ctr[PASS == 2 ? 3 : 0], 1ull);
      if (!WORDS) s_epoch = a.epoch[slot] + 1u;
      s_tail = 0u;
    }
    if (WORDS)
      for (int i = tid; i < nwords; i += T) s_bits[i] = 0u;
    __syncthreads();
    unsigned long long idx = s_idx;
    if (idx >= todo) break;
    if (PASS == 2) idx = a.list[idx];
    if (!WORDS) {
      ep = s_epoch;
      if (ep == 0u) {  // stamp counter wrapped: start the slot afresh
        for (uint64_t i = tid; i < a.stride; i += T) stamp[i] = 0u;
        ep = 1u;
      }
      __syncthreads();
      if (tid == 0) a.epoch[slot] = ep;
    }
    // the run's id in scalar registers: the first rounds of its Philox blocks are then partly scalar
    const unsigned long long run = a.first + idx;
    SetStream st = make_set_stream(kPhaseEval, run);
    st.s_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)st.s_lo);
    st.s_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)st.s_hi);
    for (int i = tid; i < a.nseeds; i += T) {
      const int32_t u = a.seeds[i];
      if (visit(u)) queue[atomicAdd(&s_tail, 1u)] = u;
    }
    __syncthreads();
    uint32_t head = 0;
    bool few = PASS == 1, listed = false;  // few: a run that turns out large goes to the list
    for (;;) {
      const uint32_t tail = s_tail;
      if (head >= tail) break;
      const int nb = (int)min(tail - head, (uint32_t)T);
      uint32_t ea = 0;
      unsigned long long d = 0;
      if (tid < nb) {
        const int32_t u = queue[head + tid];
        const int64_t x0 = a.out_off[u];
        ea = (uint32_t)x0;
        d = (unsigned long long)(a.out_off[u + 1] - x0);
      }
      // edges (low 40 bits) and nodes with edges (above) before this one
      const unsigned long long own = d | (d ? 1ull << 40 : 0ull);
      const unsigned long long incl = wave_incl_scan64(own, lane);
      if (lane == kWave - 1) s_wtot[wv] = incl;
      if (tid == 0) s_seen = 0u;
      __syncthreads();
      unsigned long long before = incl - own, all = 0;
      for (int w = 0; w < NW; ++w) {
        if (w < wv) before += s_wtot[w];
        all += s_wtot[w];
      }
      const uint32_t items = (uint32_t)(all & ((1ull << 40) - 1ull));  // at most m < 2^32
      if (PASS == 1 && few && (tail > (uint32_t)a.nseeds + kSpreadFewNodes || items > kSpreadFewEdges)) {
        __syncthreads();
        if (tid == 0) s_idx = atomicAdd(&a.ctr[2], 1ull);
        __syncthreads();
        const unsigned long long at = s_idx;
        if (at < (unsigned long long)a.list_cap) {
          if (tid == 0) a.list[at] = idx;
          listed = true;
          break;
        }
        few = false;  // no room: it is finished here
      }
      const uint32_t first_edge = (uint32_t)(before & ((1ull << 40) - 1ull));
      if (d) s_delta[(uint32_t)(before >> 40)] = ea - first_edge;
      head += (uint32_t)nb;
      for (uint32_t w0 = 0; w0 < items;) {
        for (int i = tid; i < NC; i += T) s_marks[i] = 0ull;
        __syncthreads();
        if (d && first_edge >= w0 && first_edge - w0 < W)
          atomicOr(&s_marks[(first_edge - w0) / kWave], 1ull << ((first_edge - w0) % kWave));
        __syncthreads();
        if (wv == 0) {
          uint32_t c[CPL], sum = 0;
#pragma unroll
          for (int i = 0; i < CPL; ++i) {
            c[i] = sum;
            sum += (uint32_t)__popcll(s_marks[lane * CPL + i]);
          }
          uint32_t inc = sum;
#pragma unroll
          for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o, kWave);
            if (lane >= o) inc += y;
          }
          const uint32_t base = s_seen + inc - sum;
#pragma unroll
          for (int i = 0; i < CPL; ++i) s_rank[lane * CPL + i] = base + c[i];
          if (lane == kWave - 1) s_seen = base + sum;
        }
        __syncthreads();
        const uint32_t left = items - w0;
        const int nc = left >= W ? NC : (int)((left + kWave - 1) / kWave);
        for (int c0 = wv; c0 < nc; c0 += NW * kSpreadLoads) {
          int32_t v[kSpreadLoads];
          uint32_t e[kSpreadLoads], t[kSpreadLoads];
          bool ok[kSpreadLoads];
#pragma unroll
          for (int r = 0; r < kSpreadLoads; ++r) {
            const int c = c0 + r * NW;
            const uint32_t item = (uint32_t)c * kWave + (uint32_t)lane;
            ok[r] = c < nc && item < left;
            v[r] = 0;
            e[r] = t[r] = 0u;
            if (ok[r]) {
              const uint32_t rank = s_rank[c] + (uint32_t)__popcll(s_marks[c] & upto) - 1u;
              const uint32_t x = s_delta[rank] + (w0 + item);
              v[r] = a.out_dst[x];
              e[r] = a.out_eid[x];
              if (MODEL == 0) t[r] = a.out_thr ? a.out_thr[x] : ic_threshold(g, v[r], e[r]);
            }
          }
#pragma unroll
          for (int r = 0; r < kSpreadLoads; ++r) {
            bool add = false;
            if (ok[r] && !seen(v[r]) && out_edge_live<MODEL>(g, key, st, v[r], e[r], t[r])) add = visit(v[r]);
            const uint64_t am = __ballot(add);
            if (am) {
              uint32_t base = 0;
              if (lane == 0) base = atomicAdd(&s_tail, (uint32_t)__popcll(am));
              base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
              if (add) queue[base + (uint32_t)__popcll(am & (upto >> 1))] = v[r];
            }
          }
        }
        if (left <= W) break;
        w0 += W;
        __syncthreads();
      }
      __syncthreads();
    }
    if (tid == 0 && !listed) {
      const uint32_t cnt = s_tail;
      if (a.counts) a.counts[idx] = cnt;
      total += cnt;
    }
    __syncthreads();
  }
  if (tid == 0 && total) atomicAdd(&a.ctr[1], total);
}

}  // namespace

void launch_out_csr_count(const int32_t* src, int64_t m, uint32_t* cnt, hipStream_t s) {
  hipLaunchKernelGGL(out_count_kernel, dim3(2048), dim3(kThreads), 0, s, src, m, cnt);
}

void launch_out_csr_scatter(const int64_t* in_off, const int32_t* src, int64_t n, int64_t m, const int64_t* out_off,
                            uint32_t* fill, int32_t* out_dst, uint32_t* out_eid, hipStream_t s) {
  hipLaunchKernelGGL(out_scatter_kernel, dim3(2048), dim3(kThreads), 0, s, in_off, src, n, m, out_off, fill, out_dst,
                     out_eid);
}

namespace {

// Blocks of the variant that fit a CU by its LDS and 2048 threads, over the
// whole chip, but no more than there are slots or runs.
template <int MODEL, int WORDS, int T, int PASS>
uint64_t spread_blocks() {
  const void* k = reinterpret_cast<const void*>(spread_kernel<MODEL, WORDS, T, PASS>);
  int per_cu = 0, dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1 ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, T, 0) != hipSuccess || per_cu < 1) {
    (void)hipGetLastError();
    per_cu = cus = 1 << 10;  // the slots then bound the grid
  }
  return (uint64_t)per_cu * (uint64_t)cus;
}

template <int MODEL, int WORDS, int T, int PASS = 0>
void launch_spread_as(const SpreadArgs& a, hipStream_t s) {
  const uint64_t grid = std::min<uint64_t>({spread_blocks<MODEL, WORDS, T, PASS>(), (uint64_t)a.slots, a.runs});
  hipLaunchKernelGGL((spread_kernel<MODEL, WORDS, T, PASS>), dim3((unsigned)std::max<uint64_t>(grid, 1)), dim3(T), 0, s, a);
}

// The smallest LDS bitmap that holds n nodes: the less LDS a block takes, the
// more runs a CU holds at once, which hides the latency of their first and last
// BFS levels.  Up to 2^18 nodes three 512-thread blocks share a CU (by their
// registers; 4000 runs on 50K nodes under LT take 6.6 ms, 7.4 ms with seven
// 256-thread blocks); larger bitmaps leave room for one or two blocks, so those
// have 1024 threads, up to the 1.2M nodes whose bitmap takes most of a CU's
// 160 KB.  Larger graphs keep stamps in device memory.
// The two passes above, where there are more runs than the bitmap's blocks hold at once.
template <int MODEL, int WORDS, int T>
void launch_spread_large(const SpreadArgs& a, hipStream_t s) {
  if (!a.list || std::min<uint64_t>(a.runs, (uint64_t)a.slots) <= spread_blocks<MODEL, WORDS, T, 0>()) {
    launch_spread_as<MODEL, WORDS, T>(a, s);
    return;
  }
  launch_spread_as<MODEL, 0, 512, 1>(a, s);
  launch_spread_as<MODEL, WORDS, T, 2>(a, s);
}

template <int MODEL>
void launch_spread_model(const SpreadArgs& a, hipStream_t s) {
  const int64_t words = (a.g.n + 31) >> 5;
  if (words <= 2048) launch_spread_as<MODEL, 2048, 512>(a, s);
  else if (words <= 8192) launch_spread_as<MODEL, 8192, 512>(a, s);
  else if (words <= 16384) launch_spread_large<MODEL, 16384, 1024>(a, s);
  else if (words <= kSpreadMaxWords) launch_spread_large<MODEL, kSpreadMaxWords, 1024>(a, s);
  else launch_spread_as<MODEL, 0, 512>(a, s);
}

}  // namespace

void launch_spread(int model, const SpreadArgs& a, hipStream_t s) {
  if (model == 0) {
    if (a.build_thr)
      hipLaunchKernelGGL(out_thr_kernel, dim3(2048), dim3(kThreads), 0, s, a.g, a.out_dst, a.out_eid, a.out_thr);
    launch_spread_model<0>(a, s);
  } else if (model == 2) {
    launch_spread_model<2>(a, s);
  } else {
    launch_spread_model<1>(a, s);
  }
}

}  // namespace tim
