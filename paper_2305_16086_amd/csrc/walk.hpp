// One step of a random walk, as every TGT+ walk kernel takes it.
//
// A step of 64 unrelated walks is three gathers (row bounds, neighbour id, state) of 64
// lines each.  Most miss the L1s, so a walk runs at the latency of the L2s, and three
// times slower where it misses those as well: per-source walks read the neighbour ids
// of a graph of up to 65,536 nodes from a 16-bit copy (7.7 G steps on R-MAT scale 15: 93
// -> 80 ms).  A record of id, degree and row start per slot saves a gather but misses
// the L2s more often (100 ms).
#pragma once
#include "philox.hpp"
#include "sc_internal.hpp"

namespace sc {

// Id: type of the neighbour ids read.
template <typename Id>
struct WalkGraph {
  const int32_t* __restrict__ rowptr;
  const Id* __restrict__ col;

  __device__ int step(int node, uint32_t word) const {
    const int b = rowptr[node], e = rowptr[node + 1];
    return static_cast<int>(
        col[b + static_cast<int>(pick_neighbour(word, static_cast<uint32_t>(e - b)))]);
  }
};

// Sums of value(node) over the nodes that walk pair r of half-edge (i, j), CSR slot k,
// visits in `len` steps from i (sum0) and from j (sum1).  Four steps per Philox draw,
// the word of each a compile-time index (a run-time index would put the draw in
// scratch memory); the two walks advance in lockstep so that their loads overlap.
template <typename Graph, typename Value>
__device__ inline void walk_pair(const Graph& g, int i, int64_t k, long long r, int len,
                                 unsigned k0, unsigned k1, Value value, double* sum0, double* sum1) {
  int p0 = i, p1 = static_cast<int>(g.col[k]);
  const uint32_t j = static_cast<uint32_t>(p1);
  double s0 = 0.0, s1 = 0.0;
  for (int t4 = 0; t4 < len; t4 += 4) {
    const uint32_t h = static_cast<uint32_t>(t4 >> 2);
    const U32x4 w0 = philox4x32_10(static_cast<uint32_t>(i), j, static_cast<uint32_t>(r), h, k0, k1);
    const U32x4 w1 =
        philox4x32_10(static_cast<uint32_t>(i), j, static_cast<uint32_t>(r), (1u << 31) | h, k0, k1);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (t4 + u >= len) break;
      p0 = g.step(p0, w0.w[u]);
      p1 = g.step(p1, w1.w[u]);
      s0 += value(p0);
      s1 += value(p1);
    }
  }
  *sum0 = s0;
  *sum1 = s1;
}

}  // namespace sc
