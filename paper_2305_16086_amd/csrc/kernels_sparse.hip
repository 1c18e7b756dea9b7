// Per-source TGT+ (Algorithm 4) with a frontier-sparse traversal and the
// adaptive switch step of Eq. 14 (Section 4.2.1).
//
// One workgroup owns one source i at a time and keeps its column in a private
// slot of device memory, as 64-bit fixed point (unit 2^-63):
//
//   Q_l[y] = r_l[y] / d_y,   r_l[y] = p_l(i, y) (the walk distribution from i),
//
// so that by reversibility (Eq. 4) q[y] = p_l(y, i) = d_i * Q_l[y] * 2^-63.
// One step is a push over the support S_l: r_{l+1}[y] = sum over u in N(y) of
// Q_l[u], added with 64-bit integer atomics (exact and order-free, so the
// result does not depend on the schedule), then Q_{l+1}[y] = r_{l+1}[y] / d_y
// rounded to nearest.  The support list S_{l+1} collects the nodes whose
// accumulator was zero before their first addition.
//
// At every l the workgroup evaluates Algorithm 3 on q = p_l(., i) (top-gamma
// threshold by radix select, rho-hat over the candidate edges, extremes over
// N(i), N(j) and V), the walk counts of Eq. 13, and Eq. 14's two sides; the
// first l where the frontier volume exceeds the walk work becomes tilde_tau_i.
// Sources that outgrow a workgroup go on in kernels that step them together (k_heavy_*).
// The walks of a wave of sources then run flat over the whole GPU (chunks of 64 walk pairs,
// fixed-order sums), reading q from the sources' slots.
#include "sc_internal.hpp"
#include "walk.hpp"

#include <cfloat>
#include <climits>

namespace sc {

namespace {

constexpr double kInvUnit = 1.0 / 9223372036854775808.0;   // 2^-63
constexpr int kWalkGrid = 2048;   // a multiple of 8
constexpr int kUnit = 128;        // chunks a workgroup of k_src_walks_lds takes at a time
constexpr int kUnitThreads = 1024, kUnitGrid = 256;
constexpr int kLdsNodes = 13600;  // 12 bytes of LDS each
constexpr int kShortRow = 128;    // N(j) up to this is scanned by 16 lanes, up to kLongRow by a
constexpr int kLongRow = 2048;    // wave, and a longer one by the whole workgroup
constexpr int kHubEdges = 1024;   // a longer list is pushed by the whole workgroup
constexpr int kLongList = 1024;
constexpr int kCandList = 64;     // rho candidates whose pairs are looked up one by one

// Lanes of one wave share LDS without a barrier: their LDS operations are in
// order, the fence keeps the compiler from moving them.
__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

struct MaxU64 {
  __device__ uint64_t operator()(uint64_t a, uint64_t b) const { return a > b ? a : b; }
};
struct MinU64 {
  __device__ uint64_t operator()(uint64_t a, uint64_t b) const { return a < b ? a : b; }
};
struct AddU64 {
  __device__ uint64_t operator()(uint64_t a, uint64_t b) const { return a + b; }
};
struct AddD {
  __device__ double operator()(double a, double b) const { return a + b; }
};

template <typename V, typename Op>
__device__ inline V wave_reduce(V v, Op op) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = op(v, __shfl_xor(v, off, 64));
  return v;
}

template <int kT, typename V, typename Op>
__device__ inline V block_reduce(V v, V* s, Op op) {
  v = wave_reduce(v, op);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
  __syncthreads();
  V r = s[0];
#pragma unroll
  for (int w = 1; w < kT / 64; ++w) r = op(r, s[w]);
  __syncthreads();
  return r;
}

constexpr int kEdgeIlp = 4;   // neighbour slots (or entries) of one lane in flight

// (x + d / 2) / d, exactly, for 0 < d < 2^31: the quotient by a double reciprocal (off by
// up to 2^12), once more for the remainder, and a last step either way.  The compiler's
// division of 64-bit words takes several times as long.
__device__ inline uint64_t div_round(uint64_t x, uint32_t d) {
  x += d / 2;
  const double inv = 1.0 / static_cast<double>(d);
  uint64_t q = static_cast<uint64_t>(static_cast<double>(x) * inv);
  int64_t r = static_cast<int64_t>(x - q * d);
  const int64_t c = static_cast<int64_t>(static_cast<double>(r) * inv);
  q += static_cast<uint64_t>(c);
  r -= c * static_cast<int64_t>(d);
  if (r < 0) {
    --q;
    r += d;
  }
  if (r >= static_cast<int64_t>(d)) ++q;
  return q;
}

// What the phases of a source's workgroup share.
template <int kT>
struct SrcLds {
  int off[kT], beg[kT];
  uint64_t val[kT];
  uint64_t r64[5][kT / 64];
  double rd[kT / 64];
  unsigned hist[256];
  int cnt;               // entries of the next support
  int lng[kLongList];    // list entries or halves left to more lanes
  int nlong;
  uint64_t key[64];      // the last keys of the selection
  int cand[kCandList];
  int ncand;
  uint64_t prefix;       // digits chosen so far; the threshold at the end
  int rank, left;
};

// Visit every (value, neighbour) pair of the entries [0, cnt) of a node list that
// pass `keep` (of `parts` workgroups, workgroup `part` takes its tiles).  Each wave
// takes 64 entries at a time, scans their degrees and spreads the neighbour slots over
// its lanes without a workgroup barrier; an entry with more than kHubEdges neighbours
// is left to the whole workgroup.
// act(value[], y[], live[]) gets kEdgeIlp pairs of the lane at once, so that
// their memory operations are in flight together.  Called by the whole
// workgroup; barriers inside.
template <int kT, typename Keep, typename Act>
__device__ inline void visit_edges(SrcLds<kT>& s, const int32_t* __restrict__ list, int cnt,
                                   int part, int parts, const int32_t* __restrict__ rowptr,
                                   const int32_t* __restrict__ col, Keep keep, Act act) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) s.nlong = 0;
  __syncthreads();
  int* so = s.off + wave * 64;
  int* sb = s.beg + wave * 64;
  uint64_t* sv = s.val + wave * 64;
  for (int base = part * kT + wave * 64; base < cnt; base += parts * kT) {
    const int e = base + lane;
    int du = 0, beg = 0;
    uint64_t val = 0;
    if (e < cnt) {
      const int u = list[e];
      if (keep(u, &val)) {
        beg = rowptr[u];
        du = rowptr[u + 1] - beg;
        if (du > kHubEdges) {
          const int slot = atomicAdd(&s.nlong, 1);
          if (slot < kLongList) {
            s.lng[slot] = u;
            du = 0;
          }
        }
      }
    }
    int x = du;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    const int total = __shfl(x, 63, 64);
    so[lane] = x - du;
    sb[lane] = beg - (x - du);
    sv[lane] = val;
    wave_fence();
    for (int x0 = lane; x0 < total; x0 += 64 * kEdgeIlp) {
      uint64_t v[kEdgeIlp];
      int y[kEdgeIlp];
      bool live[kEdgeIlp];
#pragma unroll
      for (int q = 0; q < kEdgeIlp; ++q) {
        const int xx = x0 + 64 * q;
        live[q] = xx < total;
        int lo = 0;   // last entry with so[] <= xx (entries without slots share offsets)
#pragma unroll
        for (int h = 32; h >= 1; h >>= 1)
          if (so[lo + h] <= xx) lo += h;
        v[q] = sv[lo];
        y[q] = live[q] ? col[sb[lo] + xx] : 0;
      }
      act(v, y, live);
    }
    wave_fence();
  }
  __syncthreads();
  const int nlong = min(s.nlong, kLongList);
  for (int t = 0; t < nlong; ++t) {
    const int u = s.lng[t];
    const int b = rowptr[u], total = rowptr[u + 1] - b;
    uint64_t val = 0;
    keep(u, &val);
    for (int x0 = tid; x0 < total; x0 += kT * kEdgeIlp) {
      uint64_t v[kEdgeIlp];
      int y[kEdgeIlp];
      bool live[kEdgeIlp];
#pragma unroll
      for (int q = 0; q < kEdgeIlp; ++q) {
        const int xx = x0 + kT * q;
        live[q] = xx < total;
        v[q] = val;
        y[q] = live[q] ? col[b + xx] : 0;
      }
      act(v, y, live);
    }
  }
  __syncthreads();
}

// x in the sorted neighbour list col[b, e)
__device__ inline bool adjacent(const int32_t* __restrict__ col, int b, int e, int x) {
  while (b < e) {
    const int mid = (b + e) >> 1;
    const int v = col[mid];
    if (v == x) return true;
    if (v < x) b = mid + 1;
    else e = mid;
  }
  return false;
}

// Threshold T = the gamma-th largest q (Algorithm 3 line 2); 0 when the
// support has fewer than gamma nodes (the candidate list then holds zeros).
// Digits of up to 8 bits from the highest set one down: a histogram of the
// keys that share the digits chosen so far, until at most 64 keys are left,
// which one wave ranks against each other.
// kKeys: the keys are kept in the column at l + 1 (all zero before), *keyed tells so.
template <int kT, bool kKeys>
__device__ inline uint64_t threshold(SrcLds<kT>& s, const SrcArgs& a, uint64_t* Q, int oc, int on,
                                     const int32_t* Sc, int cnt, uint64_t qmx, uint64_t qmn,
                                     bool* keyed_out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.n;
  bool keyed = false;
  uint64_t T = 0;
  if (a.gamma > 0 && cnt < a.gamma && cnt == n) T = qmn;   // every node is a candidate
  if (a.gamma > 0 && cnt >= a.gamma) {
    int pos = 64 - __clzll(static_cast<long long>(qmx | 1ull));   // bits below pos undecided
    uint64_t prefix = 0;
    if (tid == 0) {
      s.rank = a.gamma;
      s.left = cnt;
    }
    __syncthreads();
    int left = cnt;
    while (left > 64 && pos > 0) {
      const int width = pos < 8 ? pos : 8;
      const int shift = pos - width;
      for (int d = tid; d < 256; d += kT) s.hist[d] = 0;
      __syncthreads();
      if (!keyed) {
        for (int e0 = tid; e0 < cnt; e0 += kT * kEdgeIlp) {
          uint64_t v[kEdgeIlp];
          int y[kEdgeIlp];
#pragma unroll
          for (int q = 0; q < kEdgeIlp; ++q) y[q] = Sc[min(e0 + q * kT, cnt - 1)];
#pragma unroll
          for (int q = 0; q < kEdgeIlp; ++q) v[q] = Q[oc + y[q]];
#pragma unroll
          for (int q = 0; q < kEdgeIlp; ++q)
            if (e0 + q * kT < cnt) {
              if (kKeys) Q[on + e0 + q * kT] = v[q];   // the column at l + 1 is all zero here
              if (pos == 64 || (v[q] >> pos) == (prefix >> pos))
                atomicAdd(&s.hist[(v[q] >> shift) & ((1u << width) - 1u)], 1u);
            }
        }
        keyed = kKeys;
      } else {
        for (int e = tid; e < cnt; e += kT) {
          const uint64_t v = Q[on + e];
          if ((v >> pos) == (prefix >> pos))
            atomicAdd(&s.hist[(v >> shift) & ((1u << width) - 1u)], 1u);
        }
      }
      __syncthreads();
      if (wave == 0) {   // lane's buckets 255 - 4 lane .. 252 - 4 lane, from the top
        unsigned c[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          c[q] = s.hist[255 - 4 * lane - q];
          sum += c[q];
        }
        unsigned x = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const unsigned y = __shfl_up(x, off, 64);
          if (lane >= off) x += y;
        }
        const unsigned k = static_cast<unsigned>(s.rank);
        unsigned above = x - sum;
        if (above < k && k <= x) {   // one lane
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (above < k && k <= above + c[q]) {
              s.prefix = prefix | (static_cast<uint64_t>(255 - 4 * lane - q) << shift);
              s.rank = static_cast<int>(k - above);
              s.left = static_cast<int>(c[q]);
            }
            above += c[q];
          }
        }
      }
      __syncthreads();
      prefix = s.prefix;
      left = s.left;
      pos = shift;
    }
    if (pos == 0) {
      T = prefix;   // every bit is decided
    } else {
      if (tid == 0) s.ncand = 0;
      __syncthreads();
      for (int e = tid; e < cnt; e += kT) {
        const uint64_t v = keyed ? Q[on + e] : Q[oc + Sc[e]];
        if (pos == 64 || (v >> pos) == (prefix >> pos)) s.key[atomicAdd(&s.ncand, 1)] = v;
      }
      __syncthreads();
      if (wave == 0) {
        const uint64_t v = lane < left ? s.key[lane] : 0;
        int gt = 0, eq = 0;
        for (int q = 0; q < left; ++q) {
          const uint64_t x = s.key[q];
          gt += x > v ? 1 : 0;
          eq += x == v ? 1 : 0;
        }
        if (lane < left && gt < s.rank && s.rank <= gt + eq) s.prefix = v;   // equal values
      }
      __syncthreads();
      T = s.prefix;
    }
  }
  *keyed_out = keyed;
  return T;
}

// rho-hat (Eq. 16 bound, Algorithm 3 lines 3-5, safe reading): the best
// candidate-pair edge against q[c_1] + q[c_gamma].  Few candidates (ties may
// add more): every pair of them is looked up in the shorter of its two sorted
// lists; else every edge of a candidate is visited.
template <int kT>
__device__ inline double rho_hat(SrcLds<kT>& s, const SrcArgs& a, const uint64_t* Q, int oc, int on,
                                 const int32_t* Sc, int cnt, uint64_t T, double maxV, bool keyed) {
  const int tid = threadIdx.x;
  const uint64_t thr = T > 0 ? T : 1;
  unsigned long long best = 0;
  if (tid == 0) s.ncand = 0;
  __syncthreads();
  for (int e = tid; e < cnt; e += kT) {
    const int y = Sc[e];
    const uint64_t v = keyed ? Q[on + e] : Q[oc + y];
    if (v >= thr) {
      const int slot = atomicAdd(&s.ncand, 1);
      if (slot < kCandList) s.cand[slot] = y;
    }
  }
  __syncthreads();
  const int nc = s.ncand;
  if (nc <= kCandList) {
    for (int pq = tid; pq < nc * nc; pq += kT) {
      const int p = pq / nc, q = pq % nc;
      if (p >= q) continue;
      int c1 = s.cand[p], c2 = s.cand[q];
      int b1 = a.rowptr[c1], e1 = a.rowptr[c1 + 1];
      const int b2 = a.rowptr[c2], e2 = a.rowptr[c2 + 1];
      const unsigned long long pair = Q[oc + c1] + Q[oc + c2];
      if (e2 - b2 < e1 - b1) {
        b1 = b2;
        e1 = e2;
        c2 = c1;
      }
      if (pair > best && adjacent(a.col, b1, e1, c2)) best = pair;
    }
  } else {
    visit_edges<kT>(
        s, Sc, cnt, 0, 1, a.rowptr, a.col,
        [&](int u, uint64_t* val) {
          *val = Q[oc + u];
          return *val >= thr;
        },
        [&](const uint64_t(&v)[kEdgeIlp], const int(&y)[kEdgeIlp], const bool(&live)[kEdgeIlp]) {
#pragma unroll
          for (int q = 0; q < kEdgeIlp; ++q) {
            const uint64_t qy = live[q] ? Q[oc + y[q]] : 0;
            if (qy >= thr) best = v[q] + qy > best ? v[q] + qy : best;
          }
        });
  }
  best = block_reduce<kT>(static_cast<uint64_t>(best), s.r64[0], MaxU64{});
  return fmax(static_cast<double>(best), maxV + static_cast<double>(T));
}

// Per half (i, j) of row [rb, re): extremes over N(j), chi (Eq. 17 / Eq. 15), n_r (Eq.
// 13).  Returns the thread's share of Eq. 14's right side; of `parts` workgroups, this
// one takes the halves of part_wg.
template <int kT>
__device__ inline double scan_halves(SrcLds<kT>& s, const SrcArgs& a, const uint64_t* Q, int oc,
                                     const int32_t* Sc, int cnt, int rb, int re, int ell,
                                     int part_wg, int parts, double maxV, double minV, double maxNi,
                                     double minNi, double rhoQ) {
  constexpr int kTW = kT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double part = 0.0;
  auto count_walks = [&](int k, int len, double jmx, double jmn) {
    double chiQ;
    if (a.gamma > 0) {
      const double lb_i = minNi + (len - 1) * minV;
      const double ub_i = maxNi * 0.5 + maxV * 0.5 + (len - 1) * rhoQ * 0.5;
      const double lb_j = jmn + (len - 1) * minV;
      const double ub_j = jmx * 0.5 + maxV * 0.5 + (len - 1) * rhoQ * 0.5;
      chiQ = ub_i + ub_j - lb_i - lb_j;
    } else {
      chiQ = 2.0 * len * (maxV - minV);
    }
    // q = d_i Q 2^-63 and Eq. 13 divides chi^2 by d_i^2: d_i cancels
    const double chi = chiQ * kInvUnit;
    double r = ceil(a.coef * chi * chi);
    if (!(r >= 1.0)) r = 1.0;
    const long long nr = r > static_cast<double>(a.nr_cap) ? a.nr_cap : static_cast<long long>(r);
    a.nr_slot[k] = nr;
    part += a.rule == 0 ? static_cast<double>(nr) : 2.0 * len * static_cast<double>(nr);
  };
  // a short support against a long N(j): visit the support and test adjacency
  // to j instead
  auto by_support = [&](int dj) { return static_cast<int64_t>(cnt) * 16 < dj; };
  // extremes over N(j) seen by lane `ln` of `st` lanes, and the support nodes
  // found in it (by_support only); q is zero off the support
  auto scan_row = [&](int jb, int je, int j, int ln, int st, uint64_t* mx, uint64_t* mn,
                      int* hits) {
    *mx = 0;
    *mn = ~0ull;
    *hits = 0;
    if (by_support(je - jb)) {
      for (int e = ln; e < cnt; e += st) {
        const int y = Sc[e];
        const int yb = a.rowptr[y], ye = a.rowptr[y + 1];
        const bool in_j = ye - yb < je - jb ? adjacent(a.col, yb, ye, j)
                                            : adjacent(a.col, jb, je, y);
        if (in_j) {
          const uint64_t v = Q[oc + y];
          *mx = v > *mx ? v : *mx;
          *mn = v < *mn ? v : *mn;
          ++*hits;
        }
      }
      return;
    }
    for (int q = jb + ln; q < je; q += st * kEdgeIlp) {
      int y[kEdgeIlp];
      uint64_t v[kEdgeIlp];
#pragma unroll
      for (int x = 0; x < kEdgeIlp; ++x) y[x] = a.col[min(q + x * st, je - 1)];   // repeats the last
#pragma unroll
      for (int x = 0; x < kEdgeIlp; ++x) v[x] = Q[oc + y[x]];
#pragma unroll
      for (int x = 0; x < kEdgeIlp; ++x) {
        *mx = v[x] > *mx ? v[x] : *mx;
        *mn = v[x] < *mn ? v[x] : *mn;
      }
    }
  };
  auto row_min = [&](uint64_t mn, int hits, int dj) {
    // by support: the minimum is 0 unless the support fills N(j)
    return by_support(dj) && hits < dj ? 0.0 : static_cast<double>(mn);
  };
  if (tid == 0) s.nlong = 0;
  __syncthreads();
  const int sub = tid & 15;
  for (int k = rb + (part_wg * kT + tid) / 16; k < re; k += parts * kT / 16) {
    // 16 lanes per half; longer lists go to the list below while it has room
    const int len = a.tau_slot[k] - ell;
    if (len <= 0) {
      if (sub == 0) a.nr_slot[k] = 0;
    } else if (a.gamma <= 0) {
      if (sub == 0) count_walks(k, len, 0.0, 0.0);
    } else {
      const int j = a.col[k];
      const int jb = a.rowptr[j], je = a.rowptr[j + 1];
      bool later = false;
      if (je - jb > kShortRow) {
        int slot = 0;
        if (sub == 0) slot = atomicAdd(&s.nlong, 1);
        slot = __shfl(slot, lane & 48, 64);
        later = slot < kLongList;
        if (later && sub == 0) s.lng[slot] = k;
      }
      if (!later) {
        uint64_t mx, mn;
        int hits;
        scan_row(jb, je, j, sub, 16, &mx, &mn, &hits);
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) {
          mx = MaxU64{}(mx, __shfl_xor(mx, off, 64));
          mn = MinU64{}(mn, __shfl_xor(mn, off, 64));
          hits += __shfl_xor(hits, off, 64);
        }
        if (sub == 0) count_walks(k, len, static_cast<double>(mx), row_min(mn, hits, je - jb));
      }
    }
  }
  __syncthreads();
  const int nlong = s.nlong < kLongList ? s.nlong : kLongList;
  for (int t = wave; t < nlong; t += kTW) {   // a wave per list
    const int k = s.lng[t];
    const int j = a.col[k];
    const int jb = a.rowptr[j], je = a.rowptr[j + 1];
    if (je - jb > kLongRow && !by_support(je - jb)) continue;
    uint64_t mx, mn;
    int hits;
    scan_row(jb, je, j, lane, 64, &mx, &mn, &hits);
    mx = wave_reduce(mx, MaxU64{});
    mn = wave_reduce(mn, MinU64{});
    hits = wave_reduce(hits, [](int x, int y) { return x + y; });
    if (lane == 0)
      count_walks(k, a.tau_slot[k] - ell, static_cast<double>(mx), row_min(mn, hits, je - jb));
  }
  for (int t = 0; t < nlong; ++t) {   // hubs' lists, all threads at once
    const int k = s.lng[t];
    const int j = a.col[k];
    const int jb = a.rowptr[j], je = a.rowptr[j + 1];
    if (je - jb <= kLongRow || by_support(je - jb)) continue;
    uint64_t mx, mn;
    int hits;
    scan_row(jb, je, j, tid, kT, &mx, &mn, &hits);
    mx = block_reduce<kT>(mx, s.r64[0], MaxU64{});
    mn = block_reduce<kT>(mn, s.r64[1], MinU64{});
    if (tid == 0)
      count_walks(k, a.tau_slot[k] - ell, static_cast<double>(mx), static_cast<double>(mn));
  }
  return part;
}

// The outcome of the source in list entry li at its switch step: positions, walk counts
// and totals for the walks.
template <int kT>
__device__ inline void finish_source(SrcLds<kT>& s, const SrcArgs& a, int64_t li, int i, int w, int ell,
                                     int cnt, int parity, uint64_t pushed) {
  const int tid = threadIdx.x;
  const int rb = a.rowptr[i], re = a.rowptr[i + 1];
  unsigned long long wk = 0, ws = 0;
  const int64_t pbase = (a.hoff ? a.hoff[li] : static_cast<int64_t>(rb)) - a.pos_base;
  __syncthreads();   // walk counts written by other threads of the workgroup
  for (int k = rb + tid; k < re; k += kT) {
    const int len = a.tau_slot[k] - ell;
    const long long nr = len > 0 ? a.nr_slot[k] : 0;
    if (len <= 0) a.nr_slot[k] = 0;
    const int64_t p = pbase + (k - rb);
    a.pos_slot[p] = k;
    a.pos_w[p] = w;
    a.nr_pos[p] = nr;
    wk += static_cast<unsigned long long>(nr);
    ws += static_cast<unsigned long long>(nr) * 2ull * static_cast<unsigned long long>(len > 0 ? len : 0);
  }
  wk = block_reduce<kT>(static_cast<uint64_t>(wk), s.r64[0], AddU64{});
  ws = block_reduce<kT>(static_cast<uint64_t>(ws), s.r64[1], AddU64{});
  if (tid == 0) {
    a.tilde_row[i] = ell;
    a.slot_ctl[2 * w] = cnt;
    a.slot_ctl[2 * w + 1] = parity;
    atomicAdd(&a.totals[0], wk);
    atomicAdd(&a.totals[1], ws);
    atomicAdd(&a.totals[2], static_cast<unsigned long long>(pushed));
    atomicMin(&a.totals[3], static_cast<unsigned long long>(ell));
    atomicMax(&a.totals[4], static_cast<unsigned long long>(ell));
  }
}

// One source per workgroup of kT threads.  A step is a chain of dependent
// accesses (list, degree, neighbour, column word) with a barrier between its
// phases, so it is bound by how many of them one workgroup has in flight: the
// waves spread edges by themselves with four slots per lane, the Eq. 13 scans
// give 16 lanes to a short list, and the selection of the gamma-th largest entry
// ranks the last 64 keys in one wave.
template <int kT, bool kLds>
__global__ __launch_bounds__(kT) void k_src_head(SrcArgs a) {
  extern __shared__ uint64_t s_col[];   // kLds: [2 n], both columns
  __shared__ SrcLds<kT> s;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int w = blockIdx.x;
  const int n = a.n;
  {
    // the final column of the slot's previous source, read by that wave's walks
    // (earlier in stream order), is zeroed here instead of by a launch of its own
    const int cnt_old = a.slot_ctl[2 * w];
    if (cnt_old > 0) {
      const size_t c = 2 * static_cast<size_t>(w) + static_cast<size_t>(a.slot_ctl[2 * w + 1]);
      uint64_t* Qo = a.Q + c * static_cast<size_t>(n);
      const int32_t* So = a.S + c * static_cast<size_t>(n);
      for (int e = tid; e < cnt_old; e += kT) Qo[So[e]] = 0;
    }
    __syncthreads();
  }
  const int64_t li = a.list_base + w;
  if (li >= a.nsrc) {
    if (tid == 0) {
      a.slot_ctl[2 * w] = 0;
      a.slot_ctl[2 * w + 1] = 0;
    }
    return;
  }
  const int i = a.srcs ? a.srcs[li] : static_cast<int>(li);
  const int rb = a.rowptr[i], re = a.rowptr[i + 1];
  const int di = re - rb;
  const int taup = a.tau_row[i];
  // the columns at l and l + 1: Q[oc + y], Q[on + y]
  uint64_t* const Q = kLds ? s_col : a.Q + static_cast<size_t>(2 * w) * n;
  int oc = 0, on = n;
  if constexpr (kLds) {
    for (int x = tid; x < 2 * n; x += kT) s_col[x] = 0;
    __syncthreads();
  }
  int32_t* Sc = a.S + static_cast<size_t>(2 * w) * n;
  int32_t* Sn = Sc + n;
  int parity = 0;
  // r_0 = e_i, and what the loop below keeps of the support at each l: its
  // volume (Eq. 14 left side), extremes over it and over N(i)
  const uint64_t q0 = ((1ull << 63) + static_cast<uint64_t>(di) / 2) / static_cast<uint64_t>(di);
  if (tid == 0) {
    Q[oc + i] = q0;
    Sc[0] = i;
  }
  int cnt = 1;
  int ell = 0;
  uint64_t pushed = 0;
  uint64_t vol = static_cast<uint64_t>(di), qmx = q0, qmn = q0, qmx_i = 0, qmn_i = 0;
  __syncthreads();

  for (;;) {
    const double maxV = static_cast<double>(qmx);
    const double minV = cnt == n ? static_cast<double>(qmn) : 0.0;   // zeros outside S
    bool keyed = false;   // Qn holds the selection's keys

    // ---- (1)-(4) walk counts at this l (skipped where no half needs walks)
    // a forced switch step (tests, and a fixed tilde_tau option) skips Eq. 14 and
    // evaluates the walk counts only where it stops.  Eq. 14 itself is not
    // evaluated at l = 0: its left side is then d_i while each of the d_i halves
    // needs at least one walk pair, so it cannot switch there.
    const bool forced = a.force_tilde >= 0;
    const int stop_forced = forced ? (a.force_tilde < taup ? a.force_tilde : taup) : -1;
    const bool need = ell < taup && (forced ? ell == stop_forced : ell > 0);
    double rhs = 0.0;
    double rhoQ = 0.0;
    const double maxNi = static_cast<double>(qmx_i), minNi = static_cast<double>(qmn_i);
    if (need) {
      const uint64_t T = threshold<kT, true>(s, a, Q, oc, on, Sc, cnt, qmx, qmn, &keyed);
      if (a.gamma > 0) rhoQ = rho_hat<kT>(s, a, Q, oc, on, Sc, cnt, T, maxV, keyed);
      const double part = scan_halves<kT>(s, a, Q, oc, Sc, cnt, rb, re, ell, 0, 1, maxV, minV, maxNi,
                                          minNi, rhoQ);
      rhs = block_reduce<kT>(part, s.rd, AddD{});
    }
    // ---- (4) Eq. 14: switch when the next push costs more than the walks
    const bool done = forced ? ell >= stop_forced
                             : (ell >= taup || (need && static_cast<double>(vol) > rhs));
    if (done) {
      // clear the select keys (or hand the column to the walks), record the outcome
      if constexpr (kLds) {
        uint64_t* Qg = a.Q + (2 * static_cast<size_t>(w) + static_cast<size_t>(parity)) * n;
        for (int e = tid; e < cnt; e += kT) Qg[Sc[e]] = Q[oc + Sc[e]];
      } else if (keyed) {
        for (int e = tid; e < cnt; e += kT) Q[on + e] = 0;
      }
      finish_source<kT>(s, a, li, i, w, ell, cnt, parity, pushed);
      return;
    }

    // ---- (5) push l -> l + 1: r_{l+1}[y] = sum over u in N(y) of Q_l[u]
    if (keyed)
      for (int e = tid; e < cnt; e += kT) Q[on + e] = 0;
    if (!kLds && a.heavy && !forced && vol > a.heavy_vol) {
      // left to the heavy kernels, which begin with this push
      if (tid == 0) {
        SrcHeavy h;
        h.li = li;
        h.row = i;
        h.slot = w;
        h.ell = ell;
        h.cnt = cnt;
        h.parity = parity;
        h.pushed = pushed;
        h.vol = vol;
        h.qmx = qmx;
        h.qmn = qmn;
        h.rhs = DBL_MAX;
        a.heavy[atomicAdd(&a.heavy_ctl[0], 1)] = h;
        atomicAdd(&a.heavy_ctl[1], 1);
      }
      return;
    }
    if (tid == 0) s.cnt = 0;
    __syncthreads();
    visit_edges<kT>(
        s, Sc, cnt, 0, 1, a.rowptr, a.col,
        [&](int u, uint64_t* val) {
          *val = Q[oc + u];
          return *val != 0;
        },
        [&](const uint64_t(&v)[kEdgeIlp], const int(&y)[kEdgeIlp], const bool(&live)[kEdgeIlp]) {
          unsigned long long old[kEdgeIlp];
#pragma unroll
          for (int q = 0; q < kEdgeIlp; ++q) {
            old[q] = 1;
            if (live[q])   // only this workgroup touches the slot
              old[q] = __hip_atomic_fetch_add(reinterpret_cast<unsigned long long*>(&Q[on + y[q]]),
                                              static_cast<unsigned long long>(v[q]),
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
#pragma unroll
          for (int q = 0; q < kEdgeIlp; ++q)
            if (old[q] == 0) Sn[atomicAdd(&s.cnt, 1)] = y[q];
        });
    pushed += vol;
    const int cntn = s.cnt;
    // ---- (6) Q_{l+1}[y] = r_{l+1}[y] / d_y (rounded to nearest), the support's
    // volume and extremes; (7) clear Q_l
    uint64_t r_vol = 0, r_mx = 0, r_mn = ~0ull;
    for (int e0 = tid; e0 < cntn; e0 += kT * kEdgeIlp) {
      int y[kEdgeIlp], d[kEdgeIlp];
      uint64_t v[kEdgeIlp];
#pragma unroll
      for (int q = 0; q < kEdgeIlp; ++q) y[q] = Sn[min(e0 + q * kT, cntn - 1)];
#pragma unroll
      for (int q = 0; q < kEdgeIlp; ++q) {
        d[q] = a.rowptr[y[q] + 1] - a.rowptr[y[q]];
        v[q] = Q[on + y[q]];
      }
#pragma unroll
      for (int q = 0; q < kEdgeIlp; ++q)
        if (e0 + q * kT < cntn) {
          v[q] = div_round(v[q], static_cast<uint32_t>(d[q]));
          Q[on + y[q]] = v[q];
          r_vol += static_cast<uint64_t>(d[q]);
          r_mx = v[q] > r_mx ? v[q] : r_mx;
          r_mn = v[q] < r_mn ? v[q] : r_mn;
        }
    }
    for (int e0 = tid; e0 < cnt; e0 += kT * kEdgeIlp) {
      int y[kEdgeIlp];
#pragma unroll
      for (int q = 0; q < kEdgeIlp; ++q) y[q] = Sc[min(e0 + q * kT, cnt - 1)];
#pragma unroll
      for (int q = 0; q < kEdgeIlp; ++q) Q[oc + y[q]] = 0;
    }
    __syncthreads();
    // ---- (8) step l + 1 of Eq. 9: g(i, j) += (p(i,i) - p(j,i)) / d_i = (Q[i] - Q[j]) 2^-63,
    // and the extremes over N(i)
    const double qi = static_cast<double>(Q[on + i]);
    uint64_t r_imx = 0, r_imn = ~0ull;
    for (int k = rb + tid; k < re; k += kT) {
      const uint64_t v = Q[on + a.col[k]];
      r_imx = v > r_imx ? v : r_imx;
      r_imn = v < r_imn ? v : r_imn;
      if (ell + 1 <= a.tau_slot[k])
        a.gacc[k] += (qi - static_cast<double>(v)) * kInvUnit;
    }
    r_vol = wave_reduce(r_vol, AddU64{});
    r_mx = wave_reduce(r_mx, MaxU64{});
    r_mn = wave_reduce(r_mn, MinU64{});
    r_imx = wave_reduce(r_imx, MaxU64{});
    r_imn = wave_reduce(r_imn, MinU64{});
    if (lane == 0) {
      s.r64[0][wave] = r_vol;
      s.r64[1][wave] = r_mx;
      s.r64[2][wave] = r_mn;
      s.r64[3][wave] = r_imx;
      s.r64[4][wave] = r_imn;
    }
    __syncthreads();
    vol = 0;
    qmx = qmx_i = 0;
    qmn = qmn_i = ~0ull;
    for (int x = 0; x < kT / 64; ++x) {
      vol += s.r64[0][x];
      qmx = MaxU64{}(qmx, s.r64[1][x]);
      qmn = MinU64{}(qmn, s.r64[2][x]);
      qmx_i = MaxU64{}(qmx_i, s.r64[3][x]);
      qmn_i = MinU64{}(qmn_i, s.r64[4][x]);
    }
    __syncthreads();
    const int to = oc;
    oc = on;
    on = to;
    int32_t* ts = Sc;
    Sc = Sn;
    Sn = ts;
    cnt = cntn;
    parity ^= 1;
    ++ell;
  }
}

// ---------------------------------------------------------------- heavy sources
// Sources whose pushes outgrow one workgroup: the slowest of a launch would be alone on its
// CU (0.57 G pushed edges a second) while the others idle.
// k_src_head leaves such a source in `heavy`, and the host runs rounds of four launches,
// one step of all of them, each over `gridDim.x` workgroups per source (blockIdx.y):
// k_heavy_push (Eq. 14's decision of the last round first; who is done is finished
// there), k_heavy_divide, k_heavy_bound (one workgroup per source) and k_heavy_count.
// All sums are of whole numbers, so the results are those of k_src_head (512 sources of
// R-MAT scale 15: 32 -> 7.7 ms).
constexpr int kHeavyThreads = 512;

struct HeavyView {
  uint64_t* Q;   // [2 n]
  int oc, on;
  int32_t *Sc, *Sn;
};
__device__ inline HeavyView heavy_view(const SrcArgs& a, const SrcHeavy& h) {
  const size_t base = static_cast<size_t>(2 * h.slot) * a.n;
  const size_t at = static_cast<size_t>(h.parity) * a.n, next = static_cast<size_t>(1 - h.parity) * a.n;
  return {a.Q + base, static_cast<int>(at), static_cast<int>(next), a.S + base + at, a.S + base + next};
}

// A workgroup's share of the next support's volume and extremes.
template <int kT>
__device__ inline void add_support(uint64_t* s0, uint64_t* s1, uint64_t* s2, SrcHeavy* hp, uint64_t vol,
                                   uint64_t mx, uint64_t mn) {
  vol = block_reduce<kT>(vol, s0, AddU64{});
  mx = block_reduce<kT>(mx, s1, MaxU64{});
  mn = block_reduce<kT>(mn, s2, MinU64{});
  if (threadIdx.x == 0 && vol > 0) {
    atomicAdd(&hp->vol_n, static_cast<unsigned long long>(vol));
    atomicMax(&hp->mx_n, static_cast<unsigned long long>(mx));
    atomicMin(&hp->mn_n, static_cast<unsigned long long>(mn));
  }
}

// A push of a good part of all edges is made as a pull: the sum over each row's
// neighbours needs no atomics, which the memory takes at 17 G/s against some 200 G
// gathers (all heads of the sample above with an eighth of the edges 8.8 ms, a half 9.0,
// a 32nd 8.8; with pushes alone 28).
__device__ inline bool pulls(const SrcArgs& a, uint64_t vol) {
  return vol * 8 > static_cast<uint64_t>(a.rowptr[a.n]);
}

// The rows of part blockIdx.x, in tiles of kPullTile: 16 lanes per row, longer ones by a
// wave or the workgroup.  Rows reached are divided at once, and a tile's are appended
// to the support together.
constexpr int kPullTile = 1024;
template <int kT>
__device__ inline void pull_rows(SrcLds<kT>& s, const SrcArgs& a, SrcHeavy* hp, const HeavyView& v) {
  __shared__ int s_new[kPullTile];
  __shared__ int s_count, s_at;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = tid & 15;
  const uint64_t* Qc = v.Q + v.oc;
  uint64_t vol = 0, mx = 0, mn = ~0ull;
  // the sum over col[b, e) seen by lane `ln` of `st`
  auto row_sum = [&](int b, int e, int ln, int st) {
    uint64_t r = 0;
    for (int k = b + ln; k < e; k += st * kEdgeIlp) {
      int y[kEdgeIlp];
      uint64_t q[kEdgeIlp];
#pragma unroll
      for (int x = 0; x < kEdgeIlp; ++x) y[x] = a.col[min(k + x * st, e - 1)];
#pragma unroll
      for (int x = 0; x < kEdgeIlp; ++x) q[x] = Qc[y[x]];
#pragma unroll
      for (int x = 0; x < kEdgeIlp; ++x) r += k + x * st < e ? q[x] : 0;
    }
    return r;
  };
  auto reached = [&](int y, uint64_t r, int d) {
    const uint64_t q = div_round(r, static_cast<uint32_t>(d));
    v.Q[v.on + y] = q;
    s_new[atomicAdd(&s_count, 1)] = y;
    vol += static_cast<uint64_t>(d);
    mx = MaxU64{}(mx, q);
    mn = MinU64{}(mn, q);
  };
  // tile t has the rows t, t + tiles, ...: of similar total length also where ids go by
  // degree
  const int tiles = (a.n + kPullTile - 1) / kPullTile;
  for (int t0 = static_cast<int>(blockIdx.x); t0 < tiles; t0 += static_cast<int>(gridDim.x)) {
    if (tid == 0) {
      s_count = 0;
      s.nlong = 0;
    }
    __syncthreads();
    for (int r0 = tid / 16; r0 < kPullTile; r0 += kT / 16) {
      const int64_t y64 = t0 + static_cast<int64_t>(r0) * tiles;
      if (y64 >= a.n) break;
      const int y = static_cast<int>(y64);
      const int b = a.rowptr[y], e = a.rowptr[y + 1];
      if (e - b > kShortRow) {   // at most kPullTile = kLongList of them
        if (sub == 0) s.lng[atomicAdd(&s.nlong, 1)] = y;
        continue;
      }
      uint64_t r = row_sum(b, e, sub, 16);
#pragma unroll
      for (int off = 8; off >= 1; off >>= 1) r += __shfl_xor(r, off, 64);
      if (sub == 0 && r != 0) reached(y, r, e - b);
    }
    __syncthreads();
    const int nlong = s.nlong;
    for (int t = wave; t < nlong; t += kT / 64) {
      const int y = s.lng[t];
      const int b = a.rowptr[y], e = a.rowptr[y + 1];
      if (e - b > kLongRow) continue;
      const uint64_t r = wave_reduce(row_sum(b, e, lane, 64), AddU64{});
      if (lane == 0 && r != 0) reached(y, r, e - b);
    }
    for (int t = 0; t < nlong; ++t) {
      const int y = s.lng[t];
      const int b = a.rowptr[y], e = a.rowptr[y + 1];
      if (e - b <= kLongRow) continue;
      const uint64_t r = block_reduce<kT>(row_sum(b, e, tid, kT), s.r64[0], AddU64{});
      if (tid == 0 && r != 0) reached(y, r, e - b);
    }
    __syncthreads();
    const int count = s_count;
    if (tid == 0) s_at = count > 0 ? atomicAdd(&hp->cntn, count) : 0;
    __syncthreads();
    for (int x = tid; x < count; x += kT) v.Sn[s_at + x] = s_new[x];
    __syncthreads();
  }
  add_support<kT>(s.r64[0], s.r64[1], s.r64[2], hp, vol, mx, mn);
}

__global__ __launch_bounds__(kHeavyThreads) void k_heavy_push(SrcArgs a) {
  constexpr int kT = kHeavyThreads;
  __shared__ SrcLds<kT> s;
  SrcHeavy* hp = a.heavy + blockIdx.y;
  if (hp->done) return;
  const SrcHeavy h = *hp;
  const int tid = threadIdx.x, lane = tid & 63;
  if (h.ell >= a.tau_row[h.row] || static_cast<double>(h.vol) > h.rhs) {
    if (blockIdx.x == 0) {   // the others see `done` or the same decision
      finish_source<kT>(s, a, h.li, h.row, h.slot, h.ell, h.cnt, h.parity, h.pushed);
      if (tid == 0) {
        hp->done = 1;
        atomicSub(&a.heavy_ctl[1], 1);
      }
    }
    return;
  }
  const HeavyView v = heavy_view(a, h);
  uint64_t* Q = v.Q;
  if (pulls(a, h.vol)) {
    pull_rows<kT>(s, a, hp, v);
    return;
  }
  visit_edges<kT>(
      s, v.Sc, h.cnt, static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x), a.rowptr, a.col,
      [&](int u, uint64_t* val) {
        *val = Q[v.oc + u];
        return *val != 0;
      },
      [&](const uint64_t(&q)[kEdgeIlp], const int(&y)[kEdgeIlp], const bool(&live)[kEdgeIlp]) {
        unsigned long long old[kEdgeIlp];
#pragma unroll
        for (int x = 0; x < kEdgeIlp; ++x) {
          old[x] = 1;
          if (live[x])
            old[x] = atomicAdd(reinterpret_cast<unsigned long long*>(&Q[v.on + y[x]]),
                               static_cast<unsigned long long>(q[x]));
        }
        // one addition to the support's length per wave
        int mine = 0;
#pragma unroll
        for (int x = 0; x < kEdgeIlp; ++x) mine += old[x] == 0 ? 1 : 0;
        int before = 0, total = 0;
#pragma unroll
        for (int bit = 0; bit < 3; ++bit) {   // mine <= 4
          const uint64_t b = __ballot((mine >> bit) & 1);
          before += __popcll(b & ((1ull << lane) - 1)) << bit;
          total += __popcll(b) << bit;
        }
        if (total == 0) return;
        int at = 0;
        const uint64_t here = __ballot(1);
        const int first = __ffsll(static_cast<unsigned long long>(here)) - 1;
        if (lane == first) at = atomicAdd(&hp->cntn, total);
        at = __shfl(at, first, 64) + before;
#pragma unroll
        for (int x = 0; x < kEdgeIlp; ++x)
          if (old[x] == 0) v.Sn[at++] = y[x];
      });
}

// Q_{l+1} = r_{l+1} / d_y, its volume and extremes; Q_l is cleared.
__global__ __launch_bounds__(kHeavyThreads) void k_heavy_divide(SrcArgs a) {
  constexpr int kT = kHeavyThreads;
  __shared__ uint64_t s_r[3][kT / 64];
  SrcHeavy* hp = a.heavy + blockIdx.y;
  if (hp->done) return;
  const HeavyView v = heavy_view(a, *hp);
  const int cnt = hp->cnt, cntn = hp->cntn;
  const int t0 = static_cast<int>(blockIdx.x) * kT + threadIdx.x;
  const int stride = static_cast<int>(gridDim.x) * kT;
  uint64_t vol = 0, mx = 0, mn = ~0ull;
  if (pulls(a, hp->vol)) {   // divided already
    for (int e = t0; e < cnt; e += stride) v.Q[v.oc + v.Sc[e]] = 0;
    return;
  }
  for (int e = t0; e < cntn; e += stride) {
    const int y = v.Sn[e];
    const int d = a.rowptr[y + 1] - a.rowptr[y];
    const uint64_t q = div_round(v.Q[v.on + y], static_cast<uint32_t>(d));
    v.Q[v.on + y] = q;
    vol += static_cast<uint64_t>(d);
    mx = MaxU64{}(mx, q);
    mn = MinU64{}(mn, q);
  }
  for (int e = t0; e < cnt; e += stride) v.Q[v.oc + v.Sc[e]] = 0;
  add_support<kT>(s_r[0], s_r[1], s_r[2], hp, vol, mx, mn);
}

// Step l + 1 becomes the current one: its term of Eq. 9, the extremes over N(i) and,
// unless the source ends here, rho-hat.
__global__ __launch_bounds__(1024) void k_heavy_bound(SrcArgs a) {
  constexpr int kT = 1024;
  __shared__ SrcLds<kT> s;
  SrcHeavy* hp = a.heavy + blockIdx.x;
  if (hp->done) return;
  SrcHeavy h = *hp;
  const int tid = threadIdx.x;
  __syncthreads();
  h.pushed += h.vol;
  h.cnt = h.cntn;
  h.parity ^= 1;
  ++h.ell;
  h.vol = h.vol_n;
  h.qmx = h.mx_n;
  h.qmn = h.mn_n;
  h.cntn = 0;
  h.vol_n = h.mx_n = 0;
  h.mn_n = ~0ull;
  h.rhs = 0.0;
  h.rho = 0.0;
  const HeavyView v = heavy_view(a, h);
  const double qi = static_cast<double>(v.Q[v.oc + h.row]);
  uint64_t mx = 0, mn = ~0ull;
  for (int k = a.rowptr[h.row] + tid; k < a.rowptr[h.row + 1]; k += kT) {
    const uint64_t q = v.Q[v.oc + a.col[k]];
    mx = MaxU64{}(mx, q);
    mn = MinU64{}(mn, q);
    if (h.ell <= a.tau_slot[k]) a.gacc[k] += (qi - static_cast<double>(q)) * kInvUnit;
  }
  h.qmx_i = block_reduce<kT>(mx, s.r64[0], MaxU64{});
  h.qmn_i = block_reduce<kT>(mn, s.r64[1], MinU64{});
  if (h.ell < a.tau_row[h.row] && a.gamma > 0) {
    bool keyed;
    const uint64_t T =
        threshold<kT, false>(s, a, v.Q, v.oc, v.on, v.Sc, h.cnt, h.qmx, h.qmn, &keyed);
    h.rho = rho_hat<kT>(s, a, v.Q, v.oc, v.on, v.Sc, h.cnt, T, static_cast<double>(h.qmx), false);
  }
  if (tid == 0) *hp = h;
}

// Walk counts at the new step and Eq. 14's right side.
__global__ __launch_bounds__(kHeavyThreads) void k_heavy_count(SrcArgs a) {
  constexpr int kT = kHeavyThreads;
  __shared__ SrcLds<kT> s;
  SrcHeavy* hp = a.heavy + blockIdx.y;
  if (hp->done) return;
  const SrcHeavy h = *hp;
  if (h.ell >= a.tau_row[h.row]) return;
  const HeavyView v = heavy_view(a, h);
  const double part = block_reduce<kT>(
      scan_halves<kT>(s, a, v.Q, v.oc, v.Sc, h.cnt, a.rowptr[h.row], a.rowptr[h.row + 1], h.ell,
                      static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x),
                      static_cast<double>(h.qmx), h.cnt == a.n ? static_cast<double>(h.qmn) : 0.0,
                      static_cast<double>(h.qmx_i), static_cast<double>(h.qmn_i), h.rho),
      s.rd, AddD{});
  if (threadIdx.x == 0 && part != 0.0) atomicAdd(&hp->rhs, part);
}

// ---------------------------------------------------------------- walks of a wave
// chunk_off[p] = exclusive prefix of ceil(nr_pos[p] / 64); ctl = {chunks, fits}
// One workgroup:
// 1024 threads of eight positions take a wave of a small graph in one or two rounds
// (n = 3,000, k = 5: 11.6 us a wave with 256).
__global__ __launch_bounds__(1024) void k_src_scan(int64_t P, const int64_t* __restrict__ nr_pos,
                                                   int64_t* __restrict__ chunk_off,
                                                   int64_t capacity, int64_t* __restrict__ ctl) {
  constexpr int kPer = 8, kScan = 1024;
  __shared__ int64_t s_w[kScan / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t carry = 0;
  for (int64_t base = 0; base < P; base += kScan * kPer) {
    int64_t v[kPer];
    int64_t ts = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int64_t p = base + tid * kPer + q;
      const int64_t r = p < P ? nr_pos[p] : 0;
      v[q] = r > 0 ? (r + 63) / 64 : 0;
      ts += v[q];
    }
    int64_t x = ts;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) s_w[wave] = x;
    __syncthreads();
    int64_t pre = 0, all = 0;
#pragma unroll
    for (int q = 0; q < kScan / 64; ++q) {
      pre += q < wave ? s_w[q] : 0;
      all += s_w[q];
    }
    int64_t run = carry + pre + x - ts;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int64_t p = base + tid * kPer + q;
      if (p < P) chunk_off[p] = run;
      run += v[q];
    }
    carry += all;
    __syncthreads();
  }
  if (tid == 0) {
    chunk_off[P] = carry;
    ctl[0] = carry;
    ctl[1] = carry <= capacity ? 1 : 0;
    ctl[2] = 0;   // units drawn by k_src_walks_lds
  }
}

// Largest p in [lo, hi) with off[p] <= c (off is not decreasing and off[lo] <= c):
// 64 probes a round, so two to four rounds of one load each.
template <typename V>
__device__ inline long long find_position(const V* __restrict__ off, long long lo, long long hi,
                                          long long c, int lane) {
  while (hi - lo > 1) {
    const long long step = (hi - lo + 63) / 64;
    const long long q = lo + lane * step;
    const uint64_t below = __ballot(q < hi && off[q] <= c);
    lo += (63 - __clzll(static_cast<long long>(below))) * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// Chunks are taken in turn by all waves of the grid, those of one XCD together, so that
// at any time its L2 holds the columns of the one or two sources it walks on.
template <typename Id>
__global__ __launch_bounds__(256) void k_src_walks(SrcWalkArgs a, const Id* __restrict__ ids) {
  const WalkGraph<Id> g{a.rowptr, ids};
  const int lane = threadIdx.x & 63;
  const long long nwaves = static_cast<long long>(gridDim.x) * 4;
  // workgroup w runs on XCD w % 8: the waves of one XCD are numbered one after another
  const long long wv = static_cast<long long>((blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8) * 4 +
                       (threadIdx.x >> 6);
  const size_t n = static_cast<size_t>(a.n);
  auto slot_q = [&](int w) {
    return a.Q + (2 * static_cast<size_t>(w) + static_cast<size_t>(a.slot_ctl[2 * w + 1])) * n;
  };
  if (a.cend < 0 && a.ctl[1] == 0) {
    // the chunks do not fit the partial-sum buffer: one wave per half-edge
    for (long long p = wv; p < a.P; p += nwaves) {
      const long long nr = a.nr_pos[p];
      if (nr <= 0) continue;
      const int k = a.pos_slot[p];
      const int i = a.slot_row[k];
      const int len = a.tau_slot[k] - a.tilde_row[i];
      const uint64_t* Qs = slot_q(a.pos_w[p]);
      double acc = 0.0;
      for (long long r = lane; r < nr; r += 64) {
        double s0, s1;
        walk_pair(g, i, k, r, len, a.k0, a.k1,
                  [&](int y) { return static_cast<double>(Qs[y]); }, &s0, &s1);
        acc += (s0 - s1) * kInvUnit;   // X of Eq. 11
      }
      acc = wave_reduce(acc, AddD{});
      if (lane == 0) a.gacc[k] += acc / static_cast<double>(nr);
    }
    return;
  }
  // chunks [cb, ce): a batch given by the host, or all of them
  const long long cb = a.cend < 0 ? 0 : a.cbeg;
  const long long ce = a.cend < 0 ? a.ctl[0] : a.cend;
  long long p = 0;
  for (long long c = cb + wv; c < ce; c += nwaves) {
    if (c >= a.chunk_off[p + 1]) p = find_position(a.chunk_off, p, a.P, c, lane);
    const int k = a.pos_slot[p];
    const long long nr = a.nr_pos[p];
    const long long r = (c - a.chunk_off[p]) * 64 + lane;
    double x = 0.0;
    if (r < nr) {
      const int i = a.slot_row[k];
      const int len = a.tau_slot[k] - a.tilde_row[i];
      const uint64_t* Qs = slot_q(a.pos_w[p]);
      double s0, s1;
      walk_pair(g, i, k, r, len, a.k0, a.k1,
                [&](int y) { return static_cast<double>(Qs[y]); }, &s0, &s1);
      x = (s0 - s1) * kInvUnit;   // X of Eq. 11
    }
    x = wave_reduce(x, AddD{});
    if (lane == 0) a.part[c - cb] = x;
  }
}

// The same for a wave whose sources have many chunks each.  A CU's vector memory path
// takes about half a line per clock of such gathers, whatever cache they hit (R-MAT
// scale 15, 7.7 G steps: three gathers a step 78 ms, with the row bounds in LDS 57 ms), so
// a workgroup takes the whole CU and keeps the row bounds and the column of the nodes
// below `kc` in LDS: all of a small graph, the hubs where ids go by degree or age
// (31 ms, the time of one gather a step; 118 ms with a contiguous run of chunks per wave).
// Workgroups draw units of kUnit chunks and change the column where the source changes.
template <typename Id>
struct PrefixGraph {
  WalkGraph<Id> g;
  const Id* __restrict__ col;
  const int32_t* s_row;
  int kc;

  __device__ int step(int node, uint32_t word) const {
    int b, e;
    if (node < kc) {
      b = s_row[node];
      e = s_row[node + 1];
    } else {
      b = g.rowptr[node];
      e = g.rowptr[node + 1];
    }
    return static_cast<int>(
        col[b + static_cast<int>(pick_neighbour(word, static_cast<uint32_t>(e - b)))]);
  }
};

template <typename Id>
__global__ __launch_bounds__(kUnitThreads) void k_src_walks_lds(SrcWalkArgs a,
                                                                const Id* __restrict__ ids, int kc) {
  extern __shared__ uint64_t s_mem[];   // [kc] column, then [kc + 1] row bounds
  __shared__ long long s_unit;
  uint64_t* s_q = s_mem;
  int32_t* s_row = reinterpret_cast<int32_t*>(s_mem + kc);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int x = tid; x <= kc; x += kUnitThreads) s_row[x] = a.rowptr[x];
  const PrefixGraph<Id> g{{a.rowptr, ids}, ids, s_row, kc};
  const size_t n = static_cast<size_t>(a.n);
  int cur = -1;
  for (;;) {
    __syncthreads();
    if (tid == 0)
      s_unit = static_cast<long long>(
          atomicAdd(reinterpret_cast<unsigned long long*>(a.ctl + 2), 1ull));
    __syncthreads();
    long long c = a.cbeg + s_unit * kUnit;
    const long long end = min(static_cast<long long>(a.cend), c + kUnit);
    if (c >= end) return;
    while (c < end) {
      const long long p0 = find_position(a.chunk_off, 0, a.P, c, lane);
      const int w = a.pos_w[p0];   // the source's positions follow one another
      const long long pe = find_position(a.pos_w, p0, a.P, w, lane) + 1;
      const long long stop = min(end, static_cast<long long>(a.chunk_off[pe]));
      const uint64_t* Qs =
          a.Q + (2 * static_cast<size_t>(w) + static_cast<size_t>(a.slot_ctl[2 * w + 1])) * n;
      if (w != cur) {
        __syncthreads();
        for (int x = tid; x < kc; x += kUnitThreads) s_q[x] = Qs[x];
        __syncthreads();
        cur = w;
      }
      long long p = p0;
      for (long long x = c + wave; x < stop; x += kUnitThreads / 64) {
        if (x >= a.chunk_off[p + 1]) p = find_position(a.chunk_off, p, pe, x, lane);
        const int k = a.pos_slot[p];
        const long long r = (x - a.chunk_off[p]) * 64 + lane;
        double v = 0.0;
        if (r < a.nr_pos[p]) {
          const int i = a.slot_row[k];
          const int len = a.tau_slot[k] - a.tilde_row[i];
          double s0, s1;
          walk_pair(g, i, k, r, len, a.k0, a.k1,
                    [&](int y) { return static_cast<double>(y < kc ? s_q[y] : Qs[y]); }, &s0, &s1);
          v = (s0 - s1) * kInvUnit;   // X of Eq. 11
        }
        v = wave_reduce(v, AddD{});
        if (lane == 0) a.part[x - a.cbeg] = v;
      }
      c = stop;
    }
  }
}

// The half's chunks inside this batch: [lo, hi), stored from part[lo - cb].
__device__ inline bool finish_range(const SrcWalkArgs& a, long long p, long long* cb,
                                    long long* lo, long long* hi) {
  if (a.nr_pos[p] <= 0) return false;
  *cb = a.cend < 0 ? 0 : a.cbeg;
  *lo = max(a.chunk_off[p], *cb);
  *hi = a.cend < 0 ? a.chunk_off[p + 1] : min(a.chunk_off[p + 1], a.cend);
  return *lo < *hi;
}

// gacc[k] += (chunk sums of half p in chunk order) / n_r, one thread per half with
// at most finish_seg chunks in the batch.  The halves with more are then taken one
// by one by the whole workgroup, each thread summing one fixed segment of
// ceil(chunks / 256) in order, then the 256 segment sums in order (the order depends
// only on the chunk count).
__global__ __launch_bounds__(256) void k_src_finish(SrcWalkArgs a) {
  __shared__ double s_seg[256];
  __shared__ int s_long[256];
  __shared__ int s_nlong;
  if (a.cend < 0 && a.ctl[1] == 0) return;
  const int tid = threadIdx.x;
  if (tid == 0) s_nlong = 0;
  if (tid == 0 && blockIdx.x == 0) a.ctl[2] = 0;   // for the next batch
  __syncthreads();
  const long long base = static_cast<long long>(blockIdx.x) * 256;
  long long cb, lo, hi;
  if (base + tid < a.P && finish_range(a, base + tid, &cb, &lo, &hi)) {
    if (hi - lo > a.finish_seg) {
      s_long[atomicAdd(&s_nlong, 1)] = tid;
    } else {
      double s = 0.0;
      for (long long c = lo; c < hi; ++c) s += a.part[c - cb];
      a.gacc[a.pos_slot[base + tid]] += s / static_cast<double>(a.nr_pos[base + tid]);
    }
  }
  __syncthreads();
  for (int x = 0; x < s_nlong; ++x) {
    const long long p = base + s_long[x];
    finish_range(a, p, &cb, &lo, &hi);
    const long long seg = (hi - lo + 255) / 256;
    const long long c0 = lo + tid * seg;
    const long long c1 = min(hi, c0 + seg);
    double s = 0.0;
    for (long long c = c0; c < c1; ++c) s += a.part[c - cb];
    s_seg[tid] = s;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int q = 0; q < 256; ++q) t += s_seg[q];
      a.gacc[a.pos_slot[p]] += t / static_cast<double>(a.nr_pos[p]);
    }
    __syncthreads();
  }
}

// zero the slot's final column over its support list
__global__ __launch_bounds__(256) void k_src_clear(int n, int nslots_used, uint64_t* __restrict__ Q,
                                                   const int32_t* __restrict__ S,
                                                   const int32_t* __restrict__ slot_ctl) {
  const int w = blockIdx.x;
  if (w >= nslots_used) return;
  const int cnt = slot_ctl[2 * w];
  const int par = slot_ctl[2 * w + 1];
  uint64_t* Qs = Q + (2 * static_cast<size_t>(w) + par) * static_cast<size_t>(n);
  const int32_t* Ss = S + (2 * static_cast<size_t>(w) + par) * static_cast<size_t>(n);
  for (int e = threadIdx.x; e < cnt; e += 256) Qs[Ss[e]] = 0;
}

__global__ __launch_bounds__(256) void k_fill_u64(uint64_t* __restrict__ p, int64_t count,
                                                  uint64_t value) {
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; k < count;
       k += static_cast<int64_t>(gridDim.x) * 256)
    p[k] = value;
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* __restrict__ p, int64_t count,
                                                  uint32_t value) {
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; k < count;
       k += static_cast<int64_t>(gridDim.x) * 256)
    p[k] = value;
}

__global__ __launch_bounds__(256) void k_src_init(unsigned long long* __restrict__ totals,
                                                  int ntotals, int64_t* __restrict__ nr_slot,
                                                  int64_t slots, int32_t* __restrict__ slot_ctl,
                                                  int64_t nctl, int32_t* __restrict__ tilde_row,
                                                  int64_t n) {
  const int64_t k0 = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t st = static_cast<int64_t>(gridDim.x) * 256;
  for (int64_t k = k0; k < slots; k += st) nr_slot[k] = 0;
  for (int64_t k = k0; k < nctl; k += st) slot_ctl[k] = 0;
  for (int64_t k = k0; k < n; k += st) tilde_row[k] = -1;
  if (k0 < ntotals) totals[k0] = k0 == 3 || k0 == 6 ? ~0ull : 0ull;
}

__global__ __launch_bounds__(256) void k_narrow(const int32_t* __restrict__ src,
                                                uint16_t* __restrict__ dst, int64_t count) {
  const int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (k < count) dst[k] = static_cast<uint16_t>(src[k]);
}

// smallest and largest row truncation (tau_row) into mm[0] / mm[1]
__global__ __launch_bounds__(256) void k_tau_range(int n, const int32_t* __restrict__ tau_row,
                                                   unsigned long long* __restrict__ mm) {
  unsigned long long lo = ~0ull, hi = 0;
  for (int x = blockIdx.x * 256 + threadIdx.x; x < n; x += gridDim.x * 256) {
    const unsigned long long t = static_cast<unsigned long long>(tau_row[x]);
    lo = t < lo ? t : lo;
    hi = t > hi ? t : hi;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned long long a = __shfl_xor(lo, off, 64);
    const unsigned long long b = __shfl_xor(hi, off, 64);
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
  }
  if ((threadIdx.x & 63) == 0) {
    atomicMin(&mm[0], lo);
    atomicMax(&mm[1], hi);
  }
}

// vol[x] = sum over the neighbours j of x of d_j (one wave per node)
__global__ __launch_bounds__(256) void k_nbr_volume(int n, const int32_t* __restrict__ rowptr,
                                                    const int32_t* __restrict__ col,
                                                    int64_t* __restrict__ vol) {
  const int x = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (x >= n) return;
  int64_t v = 0;
  for (int k = rowptr[x] + lane; k < rowptr[x + 1]; k += 64) {
    const int j = col[k];
    v += rowptr[j + 1] - rowptr[j];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  if (lane == 0) vol[x] = v;
}

inline unsigned fill_grid(int64_t count) {
  const int64_t g = (count + 255) / 256;
  return static_cast<unsigned>(g < 4096 ? (g > 0 ? g : 1) : 4096);
}

}  // namespace

hipError_t launch_fill_u64(uint64_t* p, int64_t count, uint64_t value, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  k_fill_u64<<<fill_grid(count), 256, 0, st>>>(p, count, value);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, int64_t count, uint32_t value, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  k_fill_u32<<<fill_grid(count), 256, 0, st>>>(p, count, value);
  return hipGetLastError();
}

hipError_t launch_src_init(unsigned long long* totals, int ntotals, int64_t* nr_slot, int64_t slots,
                           int32_t* slot_ctl, int64_t nctl, int32_t* tilde_row, int64_t n,
                           hipStream_t st) {
  if (ntotals > 256) return hipErrorInvalidValue;
  k_src_init<<<fill_grid(std::max(slots, nctl)), 256, 0, st>>>(totals, ntotals, nr_slot, slots,
                                                               slot_ctl, nctl, tilde_row, n);
  return hipGetLastError();
}

hipError_t launch_narrow(const int32_t* src, uint16_t* dst, int64_t count, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  k_narrow<<<static_cast<unsigned>((count + 255) / 256), 256, 0, st>>>(src, dst, count);
  return hipGetLastError();
}

hipError_t launch_nbr_volume(const DeviceGraph& g, int64_t* vol, hipStream_t st) {
  k_nbr_volume<<<static_cast<unsigned>((g.n + 3) / 4), 256, 0, st>>>(g.n, g.rowptr, g.col, vol);
  return hipGetLastError();
}

hipError_t launch_tau_range(int n, const int32_t* tau_row, unsigned long long* mm, hipStream_t st) {
  k_tau_range<<<fill_grid(n) < 1024 ? fill_grid(n) : 1024, 256, 0, st>>>(n, tau_row, mm);
  return hipGetLastError();
}

hipError_t launch_src_head(const SrcArgs& a, int grid, hipStream_t st) {
  if (grid <= 0) return hipSuccess;
  // A source's time is that of one workgroup's chain of phases, so it gets as many
  // threads as leave every source of the launch a place on the chip at once (512 sources
  // of R-MAT scale 15: 34.1 ms with 512 threads, 31.8 with 1,024; 1,500 of n = 3,000: 308
  // us with 512, 289 with 256).  Up to kSrcLdsColumns nodes, both columns are kept in LDS.
  if (a.n <= kSrcLdsColumns) {
    k_src_head<512, true><<<grid, 512, static_cast<size_t>(a.n) * 16, st>>>(a);
  } else if (grid <= 512) {
    k_src_head<1024, false><<<grid, 1024, 0, st>>>(a);
  } else if (grid <= 1024) {
    k_src_head<512, false><<<grid, 512, 0, st>>>(a);
  } else {
    k_src_head<256, false><<<grid, 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_src_heavy(const SrcArgs& a, int count, int rounds, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  // a workgroup of a source that is done, or beyond its work, ends at once
  const dim3 grid(static_cast<unsigned>(std::max(4, std::min(64, 8192 / count))),
                  static_cast<unsigned>(count));
  for (int r = 0; r < rounds; ++r) {
    k_heavy_push<<<grid, kHeavyThreads, 0, st>>>(a);
    k_heavy_divide<<<grid, kHeavyThreads, 0, st>>>(a);
    k_heavy_bound<<<count, 1024, 0, st>>>(a);
    k_heavy_count<<<grid, kHeavyThreads, 0, st>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_src_scan(const SrcWalkArgs& a, hipStream_t st) {
  if (a.P <= 0) return hipSuccess;
  k_src_scan<<<1, 1024, 0, st>>>(a.P, a.nr_pos, a.chunk_off, a.capacity, a.ctl);
  return hipGetLastError();
}

hipError_t launch_src_walk_batch(const SrcWalkArgs& a, hipStream_t st) {
  if (a.P <= 0) return hipSuccess;
  const int kc = std::min(a.n, kLdsNodes);
  const size_t lds = static_cast<size_t>(kc) * 12 + 4;
  // Two units per workgroup, and enough chunks a source to be worth its column (512
  // sources of BA n = 20,000, us with k_src_walks / k_src_walks_lds: 45 k chunks 116 / 200,
  // 52 k 191 / 144, 140 k 515 / 294; 64 sources: 16 k 62 / 75, 86 k 483 / 236)
  if (a.cend >= 0 && a.cend - a.cbeg >= std::max<int64_t>(a.lds_chunks, a.lds_source * a.nsources)) {
    if (a.col16) k_src_walks_lds<<<kUnitGrid, kUnitThreads, lds, st>>>(a, a.col16, kc);
    else k_src_walks_lds<<<kUnitGrid, kUnitThreads, lds, st>>>(a, a.col, kc);
  } else if (a.col16) k_src_walks<<<kWalkGrid, 256, 0, st>>>(a, a.col16);
  else k_src_walks<<<kWalkGrid, 256, 0, st>>>(a, a.col);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_src_finish<<<static_cast<unsigned>((a.P + 255) / 256), 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_src_clear(const SrcWalkArgs& a, int nslots_used, hipStream_t st) {
  k_src_clear<<<nslots_used, 256, 0, st>>>(a.n, nslots_used, a.Qw, a.S, a.slot_ctl);
  return hipGetLastError();
}

__global__ void k_gather_i32(const int32_t* __restrict__ src, const int32_t* __restrict__ idx,
                             int32_t* __restrict__ dst, int64_t n) {
  const int64_t x = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (x < n) dst[x] = src[idx[x]];
}

hipError_t launch_gather_i32(const int32_t* src, const int32_t* idx, int32_t* dst, int64_t n,
                             hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_gather_i32<<<static_cast<unsigned>((n + 255) / 256), 256, 0, st>>>(src, idx, dst, n);
  return hipGetLastError();
}

hipError_t launch_src_walks(const SrcWalkArgs& a, hipStream_t st) {
  hipError_t e = launch_src_scan(a, st);
  if (e == hipSuccess) e = launch_src_walk_batch(a, st);
  return e;
}

}  // namespace sc
