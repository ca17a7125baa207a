// The live-edge rules of the two models, shared by the RR-set samplers
// (reverse) and the spread evaluator (forward), so that both see the same
// world for the same (seed, phase, set): IC edges by their coin words and
// thresholds (Section 2.1), LT by the one in-edge each node picks (Section 4.2;
// Section 7.1).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "engine.hpp"
#include "rng.hpp"

namespace tim {

// Edge e of an in-list of length d decided by word x: live iff x <= t(e).
template <bool WC>
__device__ __forceinline__ bool edge_live(uint32_t x, uint32_t t, int64_t d) {
  if (WC) {
    // t = floor(2^32/d) - 1, and x <= t  <=>  (x + 1) * d <= 2^32
    return (uint64_t)((uint64_t)x + 1ull) * (uint64_t)d <= (1ull << 32);
  } else {
    return x <= t;
  }
}

// Position of the first of the d >= 1 non-decreasing thresholds t that is at
// least x, or d if none is.  The thresholds are cumulative weights, so the
// position is near x * d / 2^32: windows of four thresholds are read where the
// slope 2^32 / d predicts it, from the ends of the window before (for random
// weights the error falls to about its square root each time), then at the
// middle of what is left.  A binary search takes log2(d) dependent loads, and
// the lanes of a wavefront wait for the largest d among them: LT with in-weights
// on the 1M-node graph, 733 -> 608 us per stored-set launch.  The loads may read up to three words past the
// list (GraphView::lthr is padded).
__device__ __forceinline__ uint32_t lt_lower_bound(const uint32_t* t, uint32_t d, uint32_t x) {
  uint32_t lo = 0, hi = d;  // t[lo - 1] < x <= t[hi]
  uint32_t guess = __umulhi(x, d);
  for (int it = 0; lo < hi; ++it) {
    if (it > 3) guess = lo + (hi - lo) / 2;
    uint32_t w = guess > lo ? guess - 1u : lo;
    if (w + 4u > hi) w = hi > lo + 4u ? hi - 4u : lo;
    const uint32_t left = hi - w;  // thresholds of the window that count (4 or fewer)
    uint32_t v[4];
    __builtin_memcpy(v, t + w, 16);
    uint32_t c = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4u; ++i) c += i < left && v[i] < x ? 1u : 0u;
    if (c > 0u) lo = w + c;
    if (c < 4u && c < left) hi = w + c;
    guess = c ? w + 4u + __umulhi(x - v[3], d) : w - min(w, 1u + __umulhi(v[0] - x, d));
  }
  return lo;
}

// The in-edge an LT walk takes at v (in-degree d >= 1, first in-edge ea), or
// -1 if it stops there.  With 1/indeg weights: in-edge floor(X64 * d / 2^64).
// With cumulative thresholds t (Section 7.1's normalized random weights): the
// first in-edge j with word0 <= t_j; the walk stops if word0 exceeds t_{d-1}
// (weights summing below 1).
__device__ __forceinline__ int64_t lt_pick_edge(const GraphView& g, const Key& key, const SetStream& st, int32_t v,
                                                int64_t ea, int64_t d) {
  const uint4 x = draw(key, st, kKindPick, (uint64_t)v);
  if (!g.lthr) return ea + (int64_t)scale64(x, (uint64_t)d);
  const uint32_t j = lt_lower_bound(g.lthr + ea, (uint32_t)d, x.x);
  return j < (uint32_t)d ? ea + (int64_t)j : -1;
}

// General triggering model (Section 4.2): the outcome node v draws from its
// explicit distribution (an index into g.tthr / g.tset), or -1 for the empty
// triggering set.  The outcomes of v are [toff[v], toff[v+1]) with
// non-decreasing cumulative thresholds; with x = word 0 of v's draw of kind
// 3, the first outcome with x <= its threshold, found by binary search.
__device__ __forceinline__ int64_t trig_pick(const GraphView& g, const Key& key, const SetStream& st, int32_t v) {
  int64_t lo = g.toff[v];
  const int64_t end = g.toff[v + 1];
  if (lo == end) return -1;
  const uint32_t x = draw(key, st, kKindTrigger, (uint64_t)v).x;
  if (x > g.tthr[end - 1]) return -1;
  int64_t hi = end - 1;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (x <= g.tthr[mid]) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

}  // namespace tim
