// Host-side pieces shared by the translation units of libsc: error reporting,
// the graph handle, work buffers and the per-block traversal driver.
#pragma once

#include "sc_internal.hpp"

#include <algorithm>
#include <new>
#include <stdexcept>
#include <string>
#include <vector>

namespace sc {

// Records the message for sc_last_error() and returns code.
int fail(int code, const std::string& msg);

// Every device allocation of the library goes through these two calls, which
// keep the live byte count.  When the environment variable
// SC_DEVICE_BYTES_LIMIT holds a positive number, an allocation that would
// take the live bytes above it fails with hipErrorOutOfMemory (a device-memory
// budget; also how the out-of-memory paths are tested).
hipError_t tracked_malloc_bytes(void** p, size_t bytes);
hipError_t tracked_free(void* p);
size_t tracked_live_bytes();

template <typename P>
hipError_t tracked_malloc(P** p, size_t bytes) {
  void* q = nullptr;
  const hipError_t e = tracked_malloc_bytes(&q, bytes);
  *p = static_cast<P*>(q);
  return e;
}

template <typename P>
hipError_t dev_alloc(P** p, size_t count) {
  *p = nullptr;
  if (count == 0) count = 1;
  return tracked_malloc(p, count * sizeof(P));
}

template <typename P>
void dev_free(P*& p) {
  if (p) (void)tracked_free(p);
  p = nullptr;
}

// Source blocks run in groups of up to kMaxGroup, one launch per step and group (see
// k_step).  TGT+ overlaps the tails of a group with the traversal of the next on a
// second stream, the groups alternating between kPipeSets sets of states.  A group
// takes states (two per block) of up to kGroupBytes, but at least kMinGroup blocks where
// the states of all sets fit kPipeBudgetBytes (ms per call with 2, 4, 8, 16 and 32 blocks:
// BA TGT+ n = 100,000 199, 187, 175, 178, 173; TGT n = 34,401 44.7, 32.1, 28.6, 28.4, 29.9;
// G(n, m) TGT+ n = 10,000 3.86, 2.84, 2.30, 2.06, 1.98).
constexpr int kPipeSets = 2;
constexpr int kMinGroup = 8;
constexpr size_t kGroupBytes = size_t(160) << 20;
constexpr size_t kPipeBudgetBytes = size_t(2) << 30;
constexpr size_t kTailBytes = size_t(256) << 20;   // candidate-summary scratch

// Blocks per group and the layout of the state arrays for block width B.
struct PipeLayout {
  int sets = kPipeSets;   // sets of states: one where no tails run beside the next group
  int group = 1;          // blocks per group
  int tail_group = 1;     // blocks per tail launch
  int64_t ystride = 0;    // elements per block state
  int64_t bitmap_nodes = kBitmapNodes;         // see StepJob
  uint64_t buffer_bytes = kBufferBytes;
  int bufs() const { return sets * group; }
};

// f(), with host memory that runs out reported as SC_ENOMEM: no exception leaves an entry
// point.  Device work enqueued before it uses buffers that the handle keeps.
template <typename F>
int no_throw(F f) {
  try {
    return f();
  } catch (const std::bad_alloc&) {
  } catch (const std::length_error&) {   // a vector beyond its own limit
  }
  return fail(SC_ENOMEM, "host allocation failed");
}

// runs f when the scope ends (releases buffers on every return path)
template <typename F>
struct ScopeExit {
  F& f;
  ~ScopeExit() { f(); }
};

}  // namespace sc

#define HIP_TRY(expr)                                                              \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess) {                                                        \
      return ::sc::fail(e_ == hipErrorOutOfMemory ? SC_ENOMEM : SC_EHIP,           \
                        std::string(#expr) + ": " + hipGetErrorString(e_));        \
    }                                                                              \
  } while (0)

struct sc_graph {
  sc::DeviceGraph d;
  int device = 0;
  std::vector<int32_t> rowptr_h;
  std::vector<int32_t> deg_h;
  // SC_DEGREE_ORDER: the caller's node x is stored as rank_h[x]; stored node y is
  // the caller's label_h[y] (both empty when the graph keeps the caller's ids)
  std::vector<int32_t> rank_h;
  std::vector<int32_t> label_h;
  int32_t* rank_d = nullptr;            // device copy of rank_h
  double lambda_star = -1.0;
  int lambda_converged = -1;            // of the cached lambda* (see sc_stats)
  // spectrum for CalTau (Algorithm 1): spec_omega eigenpairs of D^-1/2 A D^-1/2,
  // |lambda| descending after the trivial pair; phi node-major [n][spec_omega]
  int spec_omega = 0;
  int spec_version = 0;                 // bumped on every change (keys the cached plan)
  double* spec_lam = nullptr;           // device [spec_omega]
  double* spec_phi = nullptr;           // device [n * spec_omega]
  std::vector<double> spec_lam_h;

  // work buffers, grown on demand
  void* Y = nullptr;                    // [2 parities][bufs][ystride] block states
  size_t ybytes = 0;
  size_t group_limit = 0;               // bytes of a group's states (0: kGroupBytes); less
                                        // once a call has not found the memory for more
  hipStream_t tail_stream = nullptr;    // a group's tails overlap the next traversal
  // [0] stream joins, [1 + q] traversal of the group in set q done,
  // [1 + kPipeSets + q] its tails done
  hipEvent_t pipe_ev[1 + 2 * sc::kPipeSets] = {};
  hipEvent_t call_ev[2] = {};           // start and end of a call (timing)
  void* partials = nullptr;             // [bufs][nparts][B] giant-row chunk sums
  size_t pbytes = 0;
  unsigned long long* mask = nullptr;   // [2][group][n] neighbour bits
  size_t mask_words = 0;
  uint8_t* nz = nullptr;                // [bufs][slices][n] nonzero rows of the two-hop state
  size_t nz_bytes = 0;
  unsigned* anymask = nullptr;          // [2][group][ceil(n/32)], one bit per node
  size_t anymask_words = 0;
  bool mask_clean = false;              // every mask word is zero but mask_pending's bits
  sc::BlockList mask_pending;           // blocks whose bits are set (nb == 0: none), in
  int mask_pending_buf = 0;             // this mask set
  int mask_pending_B = 0;
  double* gacc = nullptr;
  int32_t* tau_slot = nullptr;
  int32_t* tau_row = nullptr;           // [n], then (8-aligned) the capped count
  bool capped_clean = false;            // which is zero between calls
  int64_t* nr_slot = nullptr;
  int32_t* tau_host = nullptr;          // pinned [n + 2]: tau_row, then the capped count
  unsigned long long* work = nullptr;
  unsigned long long* plan_work = nullptr;   // [4][2 x 64] walk totals per candidate switch step
  sc::TailScratch tail;                      // candidate summaries and flattened walks
  size_t tail_blocks = 0;                    // blocks the tail buffers hold
  // cached switch-step plan (the cost model depends only on these inputs)
  struct PlanKey {
    double eps;
    int L, max_L;
    double lam;
    int B, tsize, gamma;
    double delta;
    int tau_policy;   // 0: lambda*-bound, else the spectrum version used by CalTau
    bool operator==(const PlanKey& o) const {
      return eps == o.eps && L == o.L && max_L == o.max_L && lam == o.lam && B == o.B &&
             tsize == o.tsize && gamma == o.gamma && delta == o.delta &&
             tau_policy == o.tau_policy;
    }
  };
  PlanKey plan_key{};
  int plan_tilde = -1;
  bool plan_valid = false;
  // per-source TGT+ (SC_PER_SOURCE): workgroup-slot columns and the wave buffers
  struct SourceBuffers {
    uint64_t* Q = nullptr;          // [2 * slots * n] 64-bit fixed-point columns
    int32_t* S = nullptr;           // [2 * slots * n] support lists
    size_t qcap = 0;
    bool clean = false;             // Q is all zero (every call that finished leaves it so)
    int32_t* slot_ctl = nullptr;
    size_t ctl_cap = 0;
    int32_t* tilde_row = nullptr;
    size_t tilde_cap = 0;
    int32_t* pos_slot = nullptr;
    size_t pos_cap = 0;
    int32_t* pos_w = nullptr;
    size_t posw_cap = 0;
    int64_t* nr_pos = nullptr;
    size_t nrp_cap = 0;
    int64_t* chunk_off = nullptr;
    size_t co_cap = 0;
    double* part = nullptr;
    size_t part_cap = 0;
    int64_t* ctl = nullptr;
    size_t ctl2_cap = 0;
    unsigned long long* totals = nullptr;
    size_t tot_cap = 0;
    sc::SrcHeavy* heavy = nullptr;
    size_t heavy_cap = 0;
    int32_t* list = nullptr;
    size_t list_cap = 0;
    int64_t* hoff = nullptr;
    size_t hoff_cap = 0;
    std::vector<int64_t> nbr_vol_h;   // per node: sum of its neighbours' degrees (wave order)
  } src;
  double* out_dev = nullptr;
  int32_t* tau_out_dev = nullptr;
  int64_t* nr_out_dev = nullptr;
  // learned closure buffers
  void* rdiag = nullptr;
  void* roff = nullptr;
  size_t rbytes = 0;
  float* feat = nullptr;       // [m][16]
  float* zpred = nullptr;      // [m]
  double* cl_s0 = nullptr;     // [m] x 4: s0, uK, lo, hi
  unsigned char* fb = nullptr; // [m]
  int* block_flag = nullptr;   // [nblocks of width 16]
  std::vector<hipEvent_t> events;

  void release();
};

namespace sc {

// CSR and task lists of one graph, built and validated on the host.
struct HostCSR {
  int32_t n = 0;
  int64_t m = 0, nslots = 0;
  std::vector<int32_t> rowptr, col, deg, slot_row, slot_half, half_slot;
  std::vector<Task> tasks, wg_tasks;
  std::vector<HeavyRow> giant;
  int32_t nparts = 0;
  std::vector<float> inv_f;
  std::vector<double> inv_d;
};

int build_host_csr(int64_t n, int64_t m, const int64_t* u, const int64_t* v, unsigned flags,
                   HostCSR& out);
int upload_csr(const HostCSR& h, DeviceGraph& d);
// New handle owning an upload of h (h.rowptr and h.deg are moved into it).
int graph_from_csr(HostCSR& h, sc_graph** out);
// TGT+ with the frontier-sparse traversal and the per-source switch step of
// Eq. 14 (SC_PER_SOURCE).
int run_per_source(sc_graph* g, double eps, int L, const sc_options& o, double* out,
                   sc_stats* st);

// Lanczos for the omega eigenpairs of largest |lambda| (stores the converged prefix in g)
int lanczos_spectrum(sc_graph* g, int omega, int max_iter, double tol, hipStream_t st, int* kept,
                     double* worst);

PipeLayout pipe_layout(const sc_graph* g, int B, size_t tsize, int sets);
// work buffers of the traversal (and the sliced lists for B = 64)
int ensure_buffers(sc_graph* g, int B, size_t tsize, int sets, hipStream_t st);
// Gives back what is sized by the group and halves the groups to come; false when they
// are single blocks already (or the device does not answer).
bool shrink_groups(sc_graph* g, int B, size_t tsize, hipStream_t st);
// f() until it does not run out of memory, each time with groups of half the size (f
// starts over and writes no output before it has what it needs).
template <typename F>
int with_smaller_groups(sc_graph* g, int B, size_t tsize, hipStream_t st, F f) {
  int rc = f();
  while (rc == SC_ENOMEM && shrink_groups(g, B, tsize, st)) rc = f();
  return rc;
}
// DeviceGraph::col16, where the ids fit and the memory is there
int ensure_narrow_ids(sc_graph* g, hipStream_t st);
// buffers of `blocks` tails; walks: also the chunk sums
int ensure_tail(sc_graph* g, int blocks, bool walks);
int ensure_pipeline(sc_graph* g);
int ensure_closure_buffers(sc_graph* g, size_t tsize);
int compute_lambda_star(sc_graph* g, hipStream_t st, double* out);
int graph_lambda_star(sc_graph* g, hipStream_t st, double* out);

template <typename T>
__global__ void k_init_low(int n, int s0, int B, int ell, const int32_t* __restrict__ rowptr,
                           const int32_t* __restrict__ col, const T* __restrict__ inv_deg,
                           T* __restrict__ Y) {
  const int c = blockIdx.x;
  const int s = s0 + c;
  if (s >= n) return;
  if (ell == 0) {
    if (threadIdx.x == 0) Y[static_cast<size_t>(s) * B + c] = T(1);
    return;
  }
  for (int k = rowptr[s] + threadIdx.x; k < rowptr[s + 1]; k += blockDim.x) {
    const int x = col[k];
    Y[static_cast<size_t>(x) * B + c] = inv_deg[x];   // p_1(x, s) = 1/d_x for x in N(s)
  }
}

template <typename T>
inline const T* inv_deg_host_sel(const DeviceGraph& g);
template <>
inline const float* inv_deg_host_sel<float>(const DeviceGraph& g) { return g.inv_deg_f; }
template <>
inline const double* inv_deg_host_sel<double>(const DeviceGraph& g) { return g.inv_deg_d; }

// Drives the launches of groups of source blocks.
template <typename T>
struct Runner {
  sc_graph* g;
  int B;
  hipStream_t st;
  bool timing;
  PipeLayout lay;
  sc_stats stats{};
  size_t ev_used = 0;
  int par = 0;            // parity of the states of the latest step
  T* rdiag = nullptr;     // optional per-slot recordings of p_l(s,s), p_l(j,s)
  T* roff = nullptr;
  int record_to = -1;     // record steps 2..record_to

  Runner(sc_graph* g_, int B_, int sets, hipStream_t st_, bool timing_)
      : g(g_), B(B_), st(st_), timing(timing_), lay(pipe_layout(g_, B_, sizeof(T), sets)) {}

  T* Y(int parity) {
    return static_cast<T*>(g->Y) + static_cast<int64_t>(parity) * lay.bufs() * lay.ystride;
  }
  T* parts() { return static_cast<T*>(g->partials); }

  // odd: the sampled launches cycle through the dense steps of a group
  static constexpr int64_t kTimeEvery = 15;

  // timing-only events: no system-scope fence (a fence writes back and
  // invalidates the caches)
  int event_pair(hipEvent_t* a, hipEvent_t* b) {
    while (g->events.size() < ev_used + 2) {
      hipEvent_t e;
      HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableSystemFence));
      g->events.push_back(e);
    }
    *a = g->events[ev_used];
    *b = g->events[ev_used + 1];
    ev_used += 2;
    return SC_OK;
  }

  // algorithmic bytes of one dense step of one block: the state read once and
  // written once, the CSR column array, the task list and the degree vector
  double step_bytes() const {
    const double n = g->d.n, S = static_cast<double>(g->rowptr_h[g->d.n]);
    return 2.0 * n * B * sizeof(T) + 4.0 * S + 16.0 * (g->d.ntasks + g->d.nwg) + sizeof(T) * n;
  }

  AccJob pending;         // accumulation of the latest step, not yet launched

  // launches the pending accumulation on its own
  int flush_acc() {
    HIP_TRY(launch_accumulate<T>(g->d, B, pending, Y(par), lay.ystride, st));
    pending = AccJob{};
    return SC_OK;
  }

  MaskJob mask_job(const BlockList& set, const BlockList& clear, int buf) {
    MaskJob mj;
    mj.set = set;
    mj.clear = clear;
    mj.buf = buf;
    mj.slots = lay.group;
    mj.awords = (g->d.n + 31) / 32;
    mj.mask = g->mask;
    mj.anymask = g->anymask;
    return mj;
  }

  // clears the neighbour bits a traversal left set
  int flush_masks() {
    if (g->mask_pending.nb > 0) {
      HIP_TRY(launch_mask_update(g->d, g->mask_pending_B,
                                 mask_job(BlockList{}, g->mask_pending, 1 - g->mask_pending_buf),
                                 st));
      g->mask_pending = BlockList{};
    }
    return SC_OK;
  }

  // Traverses the blocks from l = 2 (l = 0, 1 are closed form) to their own last
  // steps lend[i] >= 2; the accumulation of step l rides on the launch of step
  // l + 1, that of the last step stays pending (flush_acc or a fused consumer
  // launches it).  The first dense step also sets the masks of the blocks of
  // `next` (may be null) and clears these blocks' (the two-hop step, the only
  // reader, is done by then).
  // Bit i of `keep`: the state block i ends with is read by the caller; else only its
  // accumulation is (B = 64).
  int traverse(const BlockList& blocks, const int* lend, bool acc, double* gacc,
               const BlockList* next = nullptr, uint32_t keep = ~0u) {
    pending = AccJob{};
    if (blocks.nb == 0) return SC_OK;
    int L = 2;
    for (int i = 0; i < blocks.nb; ++i) L = std::max(L, lend[i]);
    bool ready = g->mask_pending.nb == blocks.nb && g->mask_pending_B == B;
    for (int i = 0; ready && i < blocks.nb; ++i) ready = g->mask_pending.b[i].s0 == blocks.b[i].s0;
    if (!ready) {
      const int rc = flush_masks();
      if (rc) return rc;
      HIP_TRY(launch_mask_update(g->d, B, mask_job(blocks, BlockList{}, 0), st));
      g->mask_pending = blocks;
      g->mask_pending_buf = 0;
      g->mask_pending_B = B;
    }
    const int mbuf = g->mask_pending_buf;
    const int64_t awords = (g->d.n + 31) / 32;
    // blocks that have a step l, and the accumulation (or recording) of step l
    auto having = [&](int ell) {
      BlockList bl;
      for (int i = 0; i < blocks.nb; ++i)
        if (lend[i] >= ell) bl.b[bl.nb++] = blocks.b[i];
      return bl;
    };
    auto job = [&](int ell) {
      AccJob j;
      j.ell = ell;
      if (acc) {
        j.list = having(ell);
        j.tau = g->tau_slot;
        j.gacc = gacc;
      } else if (rdiag && ell <= record_to) {
        j.list = having(ell);
        j.rdiag = rdiag;
        j.roff = roff;
      }
      return j;
    };
    StepJob<T> s;
    s.ystride = lay.ystride;
    s.partials = parts();
    s.nz = g->nz;
    s.bitmap_nodes = lay.bitmap_nodes;
    s.buffer_bytes = lay.buffer_bytes;
    par = 0;
    s.blocks = blocks;
    s.Yp = Y(1);   // not read
    s.Yn = Y(0);
    s.mask = g->mask + static_cast<int64_t>(mbuf) * lay.group * g->d.n;
    s.anymask = g->anymask + static_cast<int64_t>(mbuf) * lay.group * awords;
    HIP_TRY(launch_step<T>(g->d, B, s, st));
    s.mask = nullptr;
    s.anymask = nullptr;
    auto next_masks = [&]() {
      const MaskJob mj = mask_job(next ? *next : BlockList{}, blocks, 1 - mbuf);
      g->mask_pending = mj.set;
      g->mask_pending_buf = 1 - mbuf;
      return mj;
    };
    pending = job(2);
    for (int ell = 3; ell <= L; ++ell) {
      // the first dense step skips the rows the two-hop step left at zero (B = 64);
      // the later ones gather every neighbour row and, where no block is at a last
      // step of which few rows are read, are the launches the stats count.  Every
      // kTimeEvery-th of those is timed by events that take the row kernel's own start
      // and end; the others run without events.
      s.skip = ell == 3 && B == 64;
      s.last = 0;
      if (acc && B == 64) {
        int at = 0;
        for (int i = 0; i < blocks.nb; ++i) {
          if (lend[i] < ell) continue;
          // the rows made: one per half-edge and source, no gain where the graph has fewer
          // (TGT L = 3, ms without / with: complete graph n = 250 0.43 / 0.77, G(n, m) 500
          // nodes and 25,000 edges 0.15 / 0.19; 3,000 and 60,000 0.18 / 0.17)
          const int rows = blocks.b[i].kend - blocks.b[i].kbeg + B;
          if (lend[i] == ell && !((keep >> i) & 1u) && rows <= g->d.n) s.last |= 1u << at;
          ++at;
        }
      }
      const bool dense = !s.skip && s.last == 0;   // every row of every block
      s.blocks = having(ell);
      const int launches = B == 64 ? 1 : s.blocks.nb;   // of one block each below 64
      for (int i = 0; i < launches; ++i) {
        s.ev[i] = {};
        if (timing && dense && (stats.prop_launches + i) % kTimeEvery == 0) {
          const int rc = event_pair(&s.ev[i].start, &s.ev[i].stop);
          if (rc) return rc;
        }
      }
      s.Yp = Y(par);
      s.Yn = Y(1 - par);
      s.acc = pending;
      s.mj = ell == 3 ? next_masks() : MaskJob{};
      HIP_TRY(launch_step<T>(g->d, B, s, st));
      if (dense) {
        stats.prop_launches += launches;
        stats.prop_bytes += step_bytes() * s.blocks.nb;
      }
      par = 1 - par;
      pending = job(ell);
    }
    if (L == 2) HIP_TRY(launch_mask_update(g->d, B, next_masks(), st));
    return SC_OK;
  }

  // one more dense step without accumulation (switch-step planning)
  int advance(const BlockList& blocks) {
    StepJob<T> s;
    s.blocks = blocks;
    s.Yp = Y(par);
    s.Yn = Y(1 - par);
    s.ystride = lay.ystride;
    s.partials = parts();
    s.nz = g->nz;
    s.bitmap_nodes = lay.bitmap_nodes;
    s.buffer_bytes = lay.buffer_bytes;
    HIP_TRY(launch_step<T>(g->d, B, s, st));
    par = 1 - par;
    return SC_OK;
  }

  // states at l = 0 (indicators) or l = 1 (one hop) when the walk tail starts that early
  int init_low(const BlockList& blocks, int ell) {
    par = 0;
    for (int i = 0; i < blocks.nb; ++i) {
      T* y = Y(0) + blocks.b[i].buf * lay.ystride;
      HIP_TRY(hipMemsetAsync(y, 0, static_cast<size_t>(g->d.n) * B * sizeof(T), st));
      k_init_low<T><<<B, 64, 0, st>>>(g->d.n, blocks.b[i].s0, B, ell, g->d.rowptr, g->d.col,
                                      inv_deg_host_sel<T>(g->d), y);
      HIP_TRY(hipGetLastError());
    }
    return SC_OK;
  }

  // a block's source range, slot range and largest truncation
  BlockRef block_ref(int b, const int32_t* tau_row, int* tmax) const {
    const int64_t n = g->d.n;
    BlockRef r;
    r.s0 = b * B;
    const int s1 = static_cast<int>(std::min<int64_t>(n, static_cast<int64_t>(r.s0) + B));
    r.kbeg = g->rowptr_h[r.s0];
    r.kend = g->rowptr_h[s1];
    if (tmax) {
      int t = 0;
      for (int x = r.s0; x < s1; ++x) t = std::max(t, tau_row[x]);
      *tmax = t;
    }
    return r;
  }
};

// learned closure run (method SC_LEARNED)
int run_learned(sc_graph* g, double eps, const sc_options& o, double* out_user, sc_stats* st);

}  // namespace sc
