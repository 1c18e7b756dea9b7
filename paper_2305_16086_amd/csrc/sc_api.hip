// Host side of libsc: graph ingest and validation, the truncation policy,
// the TGT / TGT+ orchestration over source blocks, and lambda* by Lanczos.
//
// Every piece of arithmetic of the method runs in the kernels of
// kernels_tgt.hip / kernels_plus.hip; this file only builds the CSR, sizes
// buffers, chooses launch parameters and sequences the launches.

#include <algorithm>
#include <limits>
#include <chrono>
#include <mutex>
#include <unordered_map>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "sc_host.hpp"

namespace sc {

namespace {
thread_local std::string g_last_error = "no error";
}  // namespace

int fail(int code, const std::string& msg) {
  g_last_error = msg;
  return code;
}

namespace {
std::mutex g_alloc_mu;
std::unordered_map<void*, size_t> g_alloc_sizes;
size_t g_alloc_live = 0;
}  // namespace

hipError_t tracked_malloc_bytes(void** p, size_t bytes) {
  *p = nullptr;
  std::lock_guard<std::mutex> lk(g_alloc_mu);
  if (const char* lim = std::getenv("SC_DEVICE_BYTES_LIMIT")) {
    const double cap = std::atof(lim);
    if (cap > 0.0 && static_cast<double>(g_alloc_live) + static_cast<double>(bytes) > cap)
      return hipErrorOutOfMemory;
  }
  const hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();   // a caller that goes on with less must not find it later
    *p = nullptr;
    return e;
  }
  g_alloc_sizes[*p] = bytes;
  g_alloc_live += bytes;
  return hipSuccess;
}

hipError_t tracked_free(void* p) {
  if (!p) return hipSuccess;
  {
    std::lock_guard<std::mutex> lk(g_alloc_mu);
    auto it = g_alloc_sizes.find(p);
    if (it != g_alloc_sizes.end()) {
      g_alloc_live -= it->second;
      g_alloc_sizes.erase(it);
    }
  }
  return hipFree(p);
}

size_t tracked_live_bytes() {
  std::lock_guard<std::mutex> lk(g_alloc_mu);
  return g_alloc_live;
}

}  // namespace sc

using sc::dev_alloc;
using sc::dev_free;
using sc::fail;

void sc_graph::release() {
  dev_free(d.rowptr);
  dev_free(d.col);
  dev_free(d.deg);
  dev_free(d.slot_row);
  dev_free(d.slot_half);
  dev_free(d.half_slot);
  dev_free(d.inv_deg_f);
  dev_free(d.inv_deg_d);
  dev_free(d.tasks);
  dev_free(d.wg_tasks);
  dev_free(d.slice_grp);
  dev_free(d.slice_row);
  dev_free(d.slice_nb);
  dev_free(d.slice_inv_f);
  dev_free(d.slice_inv_d);
  dev_free(d.giant);
  dev_free(rank_d);
  if (Y) (void)sc::tracked_free(Y);
  Y = nullptr;
  if (tau_host) (void)hipHostFree(tau_host);
  tau_host = nullptr;
  for (auto& e : call_ev) {
    if (e) (void)hipEventDestroy(e);
    e = nullptr;
  }
  if (tail_stream) (void)hipStreamDestroy(tail_stream);
  tail_stream = nullptr;
  for (auto& e : pipe_ev) {
    if (e) (void)hipEventDestroy(e);
    e = nullptr;
  }
  if (partials) (void)sc::tracked_free(partials);
  partials = nullptr;
  dev_free(mask);
  dev_free(anymask);
  dev_free(gacc);
  dev_free(tau_slot);
  dev_free(tau_row);
  dev_free(nr_slot);
  dev_free(spec_lam);
  dev_free(spec_phi);
  dev_free(tail.cs);
  dev_free(tail.col);
  dev_free(tail.chunk_off);
  dev_free(tail.part);
  dev_free(tail.ctl);
  tail = sc::TailScratch{};
  tail_blocks = 0;
  dev_free(work);
  dev_free(plan_work);
  dev_free(nz);
  dev_free(d.col16);
  dev_free(out_dev);
  dev_free(tau_out_dev);
  dev_free(nr_out_dev);
  if (rdiag) (void)sc::tracked_free(rdiag);
  if (roff) (void)sc::tracked_free(roff);
  sc::dev_free(src.Q);
  sc::dev_free(src.S);
  sc::dev_free(src.slot_ctl);
  sc::dev_free(src.tilde_row);
  sc::dev_free(src.pos_slot);
  sc::dev_free(src.pos_w);
  sc::dev_free(src.nr_pos);
  sc::dev_free(src.chunk_off);
  sc::dev_free(src.part);
  sc::dev_free(src.ctl);
  sc::dev_free(src.totals);
  sc::dev_free(src.heavy);
  sc::dev_free(src.list);
  sc::dev_free(src.hoff);
  src = SourceBuffers{};
  rdiag = roff = nullptr;
  rbytes = 0;
  dev_free(feat);
  dev_free(zpred);
  dev_free(cl_s0);
  dev_free(fb);
  dev_free(block_flag);
  for (auto& e : events) (void)hipEventDestroy(e);
  events.clear();
}

// ====================================================================== graph build

int sc::build_host_csr(int64_t n, int64_t m, const int64_t* u, const int64_t* v, unsigned flags,
                       HostCSR& out) {
  if (!u || !v) return fail(SC_EINVAL, "edge arrays are NULL");
  if (n < 2 || m < 1) return fail(SC_EINVAL, "need n >= 2 and m >= 1");
  if (n >= (1ll << 31) || 2 * m >= (1ll << 31))
    return fail(SC_EINVAL, "n and 2m must be below 2^31");
  for (int64_t e = 0; e < m; ++e) {
    if (u[e] < 0 || u[e] >= n || v[e] < 0 || v[e] >= n)
      return fail(SC_EINVAL, "edge " + std::to_string(e) + " has a node id out of [0, n)");
    if (u[e] == v[e]) return fail(SC_ESELFLOOP, "edge " + std::to_string(e) + " is a self-loop");
  }
  const int32_t N = static_cast<int32_t>(n);
  const int64_t H = 2 * m;
  std::vector<int32_t> hsrc, hdst;
  std::vector<int32_t> order, tmp;
  try {
    hsrc.resize(H);
    hdst.resize(H);
    order.resize(H);
    tmp.resize(H);
  } catch (const std::bad_alloc&) {
    return fail(SC_ENOMEM, "host allocation failed");
  }
  for (int64_t e = 0; e < m; ++e) {
    hsrc[e] = static_cast<int32_t>(u[e]);
    hdst[e] = static_cast<int32_t>(v[e]);
    hsrc[e + m] = static_cast<int32_t>(v[e]);
    hdst[e + m] = static_cast<int32_t>(u[e]);
  }
  // two stable counting sorts: by neighbour, then by source -> rows sorted by neighbour
  std::vector<int64_t> cnt(static_cast<size_t>(N) + 1);
  auto counting_sort = [&](const std::vector<int32_t>& key, const std::vector<int32_t>& in,
                           std::vector<int32_t>& outv) {
    std::fill(cnt.begin(), cnt.end(), 0);
    for (int64_t i = 0; i < H; ++i) ++cnt[key[in[i]] + 1];
    for (int32_t x = 0; x < N; ++x) cnt[x + 1] += cnt[x];
    for (int64_t i = 0; i < H; ++i) outv[cnt[key[in[i]]]++] = in[i];
  };
  std::iota(order.begin(), order.end(), 0);
  counting_sort(hdst, order, tmp);
  counting_sort(hsrc, tmp, order);

  // rows, duplicates
  std::vector<int32_t> rowptr(N + 1, 0), col, slot_half, half_slot(H);
  col.reserve(H);
  slot_half.reserve(H);
  int64_t i = 0;
  for (int32_t x = 0; x < N; ++x) {
    rowptr[x] = static_cast<int32_t>(col.size());
    while (i < H && hsrc[order[i]] == x) {
      const int32_t h = order[i];
      if (!col.empty() && static_cast<int64_t>(col.size()) > rowptr[x] && col.back() == hdst[h]) {
        if (!(flags & SC_MERGE_DUPS)) {
          const int64_t e = h % m;
          return fail(SC_EDUP, "edge " + std::to_string(e) + " repeats an earlier edge");
        }
        half_slot[h] = static_cast<int32_t>(col.size()) - 1;
      } else {
        half_slot[h] = static_cast<int32_t>(col.size());
        col.push_back(hdst[h]);
        slot_half.push_back(h);
      }
      ++i;
    }
  }
  rowptr[N] = static_cast<int32_t>(col.size());
  const int64_t S = static_cast<int64_t>(col.size());
  std::vector<int32_t> deg(N), slot_row(S);
  for (int32_t x = 0; x < N; ++x) {
    deg[x] = rowptr[x + 1] - rowptr[x];
    for (int32_t k = rowptr[x]; k < rowptr[x + 1]; ++k) slot_row[k] = x;
  }

  // connected and non-bipartite (BFS 2-colouring)
  {
    std::vector<int8_t> colour(N, -1);
    std::vector<int32_t> queue;
    queue.reserve(N);
    queue.push_back(0);
    colour[0] = 0;
    bool odd_cycle = false;
    for (size_t qh = 0; qh < queue.size(); ++qh) {
      const int32_t x = queue[qh];
      for (int32_t k = rowptr[x]; k < rowptr[x + 1]; ++k) {
        const int32_t y = col[k];
        if (colour[y] < 0) {
          colour[y] = static_cast<int8_t>(1 - colour[x]);
          queue.push_back(y);
        } else if (colour[y] == colour[x]) {
          odd_cycle = true;
        }
      }
    }
    if (static_cast<int64_t>(queue.size()) != N)
      return fail(SC_EDISCONNECTED, "graph is not connected");
    if (!odd_cycle) return fail(SC_EBIPARTITE, "graph is bipartite");
  }

  // gather tasks: workgroup tasks (heavy rows, giant-row chunks) first, then
  // wave tasks for the light rows
  std::vector<sc::Task> tasks, wg_tasks;
  std::vector<sc::HeavyRow> giant;
  int32_t nparts = 0;
  for (int32_t x = 0; x < N; ++x) {
    if (deg[x] > sc::kGiant) {
      sc::HeavyRow hr{x, nparts, 0, 0};
      for (int32_t b = rowptr[x]; b < rowptr[x + 1]; b += sc::kGiantChunk) {
        wg_tasks.push_back({x, b, std::min(b + sc::kGiantChunk, rowptr[x + 1]), nparts++});
        ++hr.nparts;
      }
      giant.push_back(hr);
    } else if (deg[x] > sc::kChunk) {
      wg_tasks.push_back({x, rowptr[x], rowptr[x + 1], -1});
    } else {
      tasks.push_back({x, rowptr[x], rowptr[x + 1], -1});
    }
  }
  std::vector<float> inv_f(N);
  std::vector<double> inv_d(N);
  for (int32_t x = 0; x < N; ++x) {
    inv_f[x] = 1.0f / static_cast<float>(deg[x]);
    inv_d[x] = 1.0 / static_cast<double>(deg[x]);
  }
  out.n = N;
  out.m = m;
  out.nslots = S;
  out.rowptr = std::move(rowptr);
  out.col = std::move(col);
  out.deg = std::move(deg);
  out.slot_row = std::move(slot_row);
  out.slot_half = std::move(slot_half);
  out.half_slot = std::move(half_slot);
  out.tasks = std::move(tasks);
  out.wg_tasks = std::move(wg_tasks);
  out.giant = std::move(giant);
  out.nparts = nparts;
  out.inv_f = std::move(inv_f);
  out.inv_d = std::move(inv_d);
  return SC_OK;
}

int sc::upload_csr(const HostCSR& h, DeviceGraph& d) {
  d.n = h.n;
  d.m = h.m;
  d.nslots = h.nslots;
  d.ntasks = static_cast<int32_t>(h.tasks.size());
  d.nwg = static_cast<int32_t>(h.wg_tasks.size());
  d.ngiant = static_cast<int32_t>(h.giant.size());
  d.nparts = h.nparts;
  auto up = [&](auto** dst, const auto& src) -> hipError_t {
    hipError_t e = dev_alloc(dst, src.size());
    if (e != hipSuccess) return e;
    if (src.empty()) return hipSuccess;
    return hipMemcpy(*dst, src.data(), src.size() * sizeof(src[0]), hipMemcpyHostToDevice);
  };
  hipError_t e = hipSuccess;
  if (e == hipSuccess) e = up(&d.rowptr, h.rowptr);
  if (e == hipSuccess) e = up(&d.col, h.col);
  if (e == hipSuccess) e = up(&d.deg, h.deg);
  if (e == hipSuccess) e = up(&d.slot_row, h.slot_row);
  if (e == hipSuccess) e = up(&d.slot_half, h.slot_half);
  if (e == hipSuccess) e = up(&d.half_slot, h.half_slot);
  if (e == hipSuccess) e = up(&d.inv_deg_f, h.inv_f);
  if (e == hipSuccess) e = up(&d.inv_deg_d, h.inv_d);
  if (e == hipSuccess) e = up(&d.tasks, h.tasks);
  if (e == hipSuccess) e = up(&d.wg_tasks, h.wg_tasks);
  if (e == hipSuccess) e = up(&d.giant, h.giant);
  if (e != hipSuccess)
    return fail(e == hipErrorOutOfMemory ? SC_ENOMEM : SC_EHIP,
                std::string("graph upload: ") + hipGetErrorString(e));
  return SC_OK;
}

int sc::graph_from_csr(HostCSR& h, sc_graph** out) {
  sc_graph* g = new (std::nothrow) sc_graph();
  if (!g) return fail(SC_ENOMEM, "host allocation failed");
  (void)hipGetDevice(&g->device);
  const int rc = sc::upload_csr(h, g->d);
  if (rc) {
    g->release();
    delete g;
    return rc;
  }
  g->rowptr_h = std::move(h.rowptr);
  g->deg_h = std::move(h.deg);
  *out = g;
  return SC_OK;
}

namespace {

// Breadth-first visiting order of the nodes (ids valid, n >= 1): started at
// the highest-degree node (lowest id among equals), each node's neighbours
// taken in ascending id; unreached nodes follow in ascending id.
void bfs_order(int64_t n, int64_t m, const int64_t* u, const int64_t* v, std::vector<int32_t>& label) {
  std::vector<int64_t> off(n + 1, 0);
  for (int64_t e = 0; e < m; ++e) {
    ++off[u[e] + 1];
    ++off[v[e] + 1];
  }
  for (int64_t x = 0; x < n; ++x) off[x + 1] += off[x];
  std::vector<int32_t> adj(static_cast<size_t>(2 * m));
  {
    // rows in edge order, then transposed: walking the rows in ascending x and
    // appending x to each neighbour's row leaves every row in ascending id
    std::vector<int32_t> first(static_cast<size_t>(2 * m));
    std::vector<int64_t> pos(off.begin(), off.end() - 1);
    for (int64_t e = 0; e < m; ++e) {
      first[pos[u[e]]++] = static_cast<int32_t>(v[e]);
      first[pos[v[e]]++] = static_cast<int32_t>(u[e]);
    }
    pos.assign(off.begin(), off.end() - 1);
    for (int64_t x = 0; x < n; ++x)
      for (int64_t k = off[x]; k < off[x + 1]; ++k) adj[pos[first[k]]++] = static_cast<int32_t>(x);
  }
  int64_t s = 0;
  for (int64_t x = 1; x < n; ++x)
    if (off[x + 1] - off[x] > off[s + 1] - off[s]) s = x;
  std::vector<unsigned char> seen(n, 0);
  label.clear();
  label.reserve(n);
  seen[s] = 1;
  label.push_back(static_cast<int32_t>(s));
  for (size_t q = 0; q < label.size(); ++q) {
    const int32_t x = label[q];
    for (int64_t k = off[x]; k < off[x + 1]; ++k) {
      const int32_t y = adj[k];
      if (!seen[y]) {
        seen[y] = 1;
        label.push_back(y);
      }
    }
  }
  for (int64_t x = 0; x < n; ++x)
    if (!seen[x]) label.push_back(static_cast<int32_t>(x));
}

}  // namespace

extern "C" int sc_build_graph(int64_t n, int64_t m, const int64_t* u, const int64_t* v,
                              unsigned flags, sc_graph** out) {
  if (!out) return fail(SC_EINVAL, "out handle pointer is NULL");
  *out = nullptr;
  const unsigned order_flags = flags & (SC_DEGREE_ORDER | SC_BFS_ORDER);
  if (order_flags == (SC_DEGREE_ORDER | SC_BFS_ORDER))
    return fail(SC_EINVAL, "SC_DEGREE_ORDER and SC_BFS_ORDER exclude each other");
  const unsigned build_flags = flags & ~(SC_DEGREE_ORDER | SC_BFS_ORDER);
  sc::HostCSR h;
  bool ranges_ok = order_flags && u && v && n >= 2 && n < (1ll << 31) && m >= 1 &&
                   2 * m < (1ll << 31);
  for (int64_t e = 0; ranges_ok && e < m; ++e)
    ranges_ok = u[e] >= 0 && u[e] < n && v[e] >= 0 && v[e] < n;
  if (!ranges_ok) {
    // the caller's ids (or input errors, reported by the build)
    const int rc = sc::build_host_csr(n, m, u, v, build_flags, h);
    if (rc) return rc;
    return sc::graph_from_csr(h, out);
  }
  // renumber (stored node y is the caller's label[y]); the edge order is kept
  std::vector<int32_t> rank, label;
  std::vector<int64_t> u2, v2;
  try {
    if (order_flags == SC_BFS_ORDER) {
      bfs_order(n, m, u, v, label);
    } else {   // descending degree, ties by ascending id
      std::vector<int64_t> deg(n, 0);
      for (int64_t e = 0; e < m; ++e) {
        ++deg[u[e]];
        ++deg[v[e]];
      }
      label.resize(n);
      std::iota(label.begin(), label.end(), 0);
      std::stable_sort(label.begin(), label.end(),
                       [&](int32_t a, int32_t b) { return deg[a] > deg[b]; });
    }
    rank.resize(n);
    for (int64_t y = 0; y < n; ++y) rank[label[y]] = static_cast<int32_t>(y);
    u2.resize(m);
    v2.resize(m);
    for (int64_t e = 0; e < m; ++e) {
      u2[e] = rank[u[e]];
      v2[e] = rank[v[e]];
    }
  } catch (const std::bad_alloc&) {
    return fail(SC_ENOMEM, "host allocation failed");
  }
  int rc = sc::build_host_csr(n, m, u2.data(), v2.data(), build_flags, h);
  if (rc) return rc;
  u2 = std::vector<int64_t>();
  v2 = std::vector<int64_t>();
  sc_graph* g = nullptr;
  rc = sc::graph_from_csr(h, &g);
  if (rc) return rc;
  const hipError_t e = sc::dev_alloc(&g->rank_d, static_cast<size_t>(n));
  const hipError_t e2 = e == hipSuccess ? hipMemcpy(g->rank_d, rank.data(), n * sizeof(int32_t),
                                                    hipMemcpyHostToDevice)
                                        : e;
  if (e2 != hipSuccess) {
    sc_free_graph(g);
    return fail(e2 == hipErrorOutOfMemory ? SC_ENOMEM : SC_EHIP,
                std::string("graph upload: ") + hipGetErrorString(e2));
  }
  g->rank_h = std::move(rank);
  g->label_h = std::move(label);
  *out = g;
  return SC_OK;
}

extern "C" int sc_graph_size(const sc_graph* g, int64_t* n, int64_t* m) {
  if (!g) return fail(SC_EINVAL, "graph is NULL");
  if (n) *n = g->d.n;
  if (m) *m = g->d.m;
  return SC_OK;
}

extern "C" void sc_free_graph(sc_graph* g) {
  if (!g) return;
  int cur = 0;
  (void)hipGetDevice(&cur);
  (void)hipSetDevice(g->device);
  (void)hipDeviceSynchronize();
  g->release();
  (void)hipSetDevice(cur);
  delete g;
}

// ====================================================================== lambda* by Lanczos

namespace {

// Device side of one or two Lanczos runs (kernels_lanczos.hip), driven in windows of
// steps: advance() enqueues a window and the copy of alpha and beta behind it, take()
// makes the oldest window's values readable.  With two windows under way the host
// evaluates one while the device works on the next.
struct LanczosDriver {
  sc::LanczosArgs a;
  std::vector<double*> owned;
  double* host = nullptr;          // pinned [2 windows][alpha, beta][runs][kcols]
  hipEvent_t ev[2] = {};
  hipStream_t st = nullptr;
  int kmax = 0;
  int enqueued = 0;                // steps enqueued
  int upto[2] = {};                // last step of the window in copy q
  int issued = 0, taken = 0;       // windows (issued - taken <= 2)

  ~LanczosDriver() {
    for (double* p : owned) (void)sc::tracked_free(p);
    if (host) (void)hipHostFree(host);
    for (auto& e : ev)
      if (e) (void)hipEventDestroy(e);
  }

  hipError_t alloc(double** p, size_t count) {
    const hipError_t e = dev_alloc(p, count);
    if (e == hipSuccess) owned.push_back(*p);
    return e;
  }

  // Column 0 of the basis: the top eigenvector sqrt(d / 2m) (eigenvalue 1, deflated by
  // the re-orthogonalisation); w[0]: a fixed pseudo-random unit vector orthogonal to
  // it, run r from seed seed0 + r.
  hipError_t start(const sc::DeviceGraph& dg, const int32_t* deg_host, int seed0, int runs, int kmax_,
                   hipStream_t st_) {
    st = st_;
    kmax = kmax_;
    const int64_t n = dg.n;
    a.n = n;
    a.runs = runs;
    a.rows = sc::lanczos_rows(n);
    a.chunks = static_cast<int>((n + a.rows - 1) / a.rows);
    a.kcols = kmax + 2;
    a.rowptr = dg.rowptr;
    a.col = dg.col;
    a.vstride = static_cast<int64_t>(a.kcols) * n;
    double *sid = nullptr, *small = nullptr;
    const size_t parts = static_cast<size_t>(runs) * a.chunks * a.kcols;
    hipError_t e = alloc(&a.V, static_cast<size_t>(runs) * a.vstride);
    if (e == hipSuccess) e = alloc(&a.w[0], static_cast<size_t>(runs) * n);
    if (e == hipSuccess) e = alloc(&a.w[1], static_cast<size_t>(runs) * n);
    if (e == hipSuccess) e = alloc(&sid, n);
    if (e == hipSuccess) e = alloc(&a.part[0], parts);
    if (e == hipSuccess) e = alloc(&a.part[1], parts);
    if (e == hipSuccess) e = alloc(&small, static_cast<size_t>(runs) * (a.chunks + 2 * a.kcols));
    if (e == hipSuccess)
      e = hipHostMalloc(reinterpret_cast<void**>(&host),
                        2 * static_cast<size_t>(runs) * 2 * a.kcols * sizeof(double));
    for (auto& x : ev)
      if (e == hipSuccess) e = hipEventCreateWithFlags(&x, hipEventDisableTiming);
    if (e != hipSuccess) return e;
    a.sid = sid;
    a.alpha = small;
    a.beta = small + static_cast<size_t>(runs) * a.kcols;
    a.norm = a.beta + static_cast<size_t>(runs) * a.kcols;
    std::vector<double> hv(n), sidh(n), v0(n);
    const double two_m = static_cast<double>(dg.nslots);
    for (int64_t x = 0; x < n; ++x) {
      hv[x] = std::sqrt(deg_host[x] / two_m);
      sidh[x] = 1.0 / std::sqrt(static_cast<double>(deg_host[x]));
    }
    e = hipMemcpyAsync(sid, sidh.data(), n * sizeof(double), hipMemcpyHostToDevice, st);
    for (int r = 0; r < runs && e == hipSuccess; ++r) {
      uint64_t z = 0x9E3779B97F4A7C15ull * (2 * static_cast<uint64_t>(seed0 + r) + 1);
      double dot = 0.0;
      for (int64_t x = 0; x < n; ++x) {
        z += 0x9E3779B97F4A7C15ull;
        uint64_t q = z;
        q = (q ^ (q >> 30)) * 0xBF58476D1CE4E5B9ull;
        q = (q ^ (q >> 27)) * 0x94D049BB133111EBull;
        q ^= q >> 31;
        v0[x] = (static_cast<double>(q >> 11) * (1.0 / 9007199254740992.0)) * 2.0 - 1.0;
        dot += v0[x] * hv[x];
      }
      double nrm = 0.0;
      for (int64_t x = 0; x < n; ++x) {
        v0[x] -= dot * hv[x];
        nrm += v0[x] * v0[x];
      }
      nrm = std::sqrt(nrm);
      for (int64_t x = 0; x < n; ++x) v0[x] /= nrm;
      e = hipMemcpyAsync(a.V + r * a.vstride, hv.data(), n * sizeof(double), hipMemcpyHostToDevice, st);
      if (e == hipSuccess)
        e = hipMemcpyAsync(a.w[0] + r * n, v0.data(), n * sizeof(double), hipMemcpyHostToDevice, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);   // v0 is drawn again
    }
    return e;
  }

  // The first kProbes windows of kProbe steps are waited for one by one and only looked at
  // for their end: where the Krylov space closes at once (complete graphs, hubs joined to
  // everything) the steps of full windows would be for nothing (lambda* of the complete
  // graph on 129 nodes 1.17 -> 0.25 ms, of 70 hubs joined to 6,000 nodes 2.9 -> 0.7).
  static constexpr int kProbe = 2, kProbes = 2;
  bool probing() const { return taken <= kProbes; }   // the window just taken was one
  // enqueues what is to follow it, the last probe's window completing the first full one
  hipError_t after_probe(int window) {
    return enqueued >= kmax ? hipSuccess
                            : advance(taken < kProbes ? kProbe : window - kProbes * kProbe);
  }

  // enqueues a window of up to `steps` steps
  hipError_t advance(int steps) {
    const int last = std::min(enqueued + steps, kmax);
    hipError_t e = hipSuccess;
    for (int j = enqueued + 1; j <= last && e == hipSuccess; ++j) e = sc::launch_lanczos_step(a, j, st);
    enqueued = last;
    if (e == hipSuccess) e = sc::launch_lanczos_beta(a, last, st);
    const size_t words = static_cast<size_t>(a.runs) * 2 * a.kcols;
    const int q = issued & 1;
    if (e == hipSuccess)
      e = hipMemcpyAsync(host + q * words, a.alpha, words * sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipEventRecord(ev[q], st);
    upto[q] = last;
    ++issued;
    return e;
  }

  // waits for the oldest window; its values are in copy *q up to step *last
  hipError_t take(int* q, int* last) {
    *q = taken & 1;
    *last = upto[*q];
    ++taken;
    return hipEventSynchronize(ev[*q]);
  }
  double alpha(int q, int run, int j) const {
    return host[(static_cast<size_t>(q) * 2 * a.runs + run) * a.kcols + j];
  }
  double beta(int q, int run, int j) const {
    return host[(static_cast<size_t>(q) * 2 * a.runs + a.runs + run) * a.kcols + j];
  }
  // first step in (from, to] with beta below 1e-12 (the Krylov space is exhausted; what
  // follows it is not used), else 0
  int exhausted(int q, int run, int from, int to) const {
    for (int j = from + 1; j <= to; ++j)
      if (!(beta(q, run, j) >= 1e-12)) return j;
    return 0;
  }
};

// Eigenvalues of the symmetric tridiagonal matrix (diagonal d[0..k), off-diagonal
// e[0..k-1)) by implicit QL iterations with Wilkinson-type shifts (Wilkinson and
// Reinsch; Golub and Van Loan, implicit symmetric tridiagonal QR).  d receives
// the eigenvalues (unordered) and zlast the last components of their vectors.
// Returns false if an eigenvalue needs more than 60 iterations.
bool tridiag_eigen(std::vector<double>& d, std::vector<double> e, std::vector<double>& zlast) {
  const int k = static_cast<int>(d.size());
  e.resize(k, 0.0);
  e[k - 1] = 0.0;
  zlast.assign(k, 0.0);
  zlast[k - 1] = 1.0;
  const double ulp = std::numeric_limits<double>::epsilon();
  for (int l = 0; l < k; ++l) {
    for (int iter = 0;; ++iter) {
      int m = l;
      for (; m < k - 1; ++m)   // first negligible off-diagonal at or after l
        if (std::fabs(e[m]) <= ulp * (std::fabs(d[m]) + std::fabs(d[m + 1]))) break;
      if (m == l) break;
      if (iter == 60) return false;
      // shift from the leading 2 x 2 block, then chase the bulge from m up to l
      double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double r = std::sqrt(g * g + 1.0);
      g = d[m] - d[l] + e[l] / (g + std::copysign(r, g));
      double sn = 1.0, cs = 1.0, p = 0.0;
      bool split = false;
      for (int i = m - 1; i >= l; --i) {
        const double f = sn * e[i];
        const double b = cs * e[i];
        r = std::sqrt(f * f + g * g);   // entries of N are at most 1: no overflow
        e[i + 1] = r;
        if (r == 0.0) {   // the matrix splits: deflate and restart from l
          d[i + 1] -= p;
          e[m] = 0.0;
          split = true;
          break;
        }
        sn = f / r;
        cs = g / r;
        g = d[i + 1] - p;
        r = (d[i] - g) * sn + 2.0 * cs * b;
        p = sn * r;
        d[i + 1] = g + p;
        g = cs * r - b;
        const double t = zlast[i + 1];
        zlast[i + 1] = sn * zlast[i] + cs * t;
        zlast[i] = cs * zlast[i] - sn * t;
      }
      if (split) continue;
      d[l] -= p;
      e[l] = g;
      e[m] = 0.0;
    }
  }
  return true;
}

// Eigenvectors of the same matrix for the count eigenvalues lam (any order) by inverse
// iteration (Golub and Van Loan, section 8.2.2; the tridiagonal systems by Gaussian
// elimination with partial pivoting), each orthogonalised against the vectors already
// found whose eigenvalues lie within 1e-3: row c of z (count x k) is the vector of
// lam[c].  O(k) per vector, where accumulating the QL rotations costs O(k^2).
void tridiag_vectors(const std::vector<double>& d, const std::vector<double>& e,
                     const double* lam, int count, std::vector<double>& z) {
  const int k = static_cast<int>(d.size());
  z.assign(static_cast<size_t>(count) * k, 0.0);
  const double tiny = std::numeric_limits<double>::epsilon();
  std::vector<double> u0(k), u1(k), u2(k), l(k), x(k);
  std::vector<char> swapped(k);
  uint64_t seed = 0x9E3779B97F4A7C15ull;
  for (int c = 0; c < count; ++c) {
    double* v = z.data() + static_cast<size_t>(c) * k;
    // P (T - lam I) = L U, U with two superdiagonals
    double a0 = d[0] - lam[c], a1 = k > 1 ? e[0] : 0.0, a2 = 0.0;
    for (int i = 0; i + 1 < k; ++i) {
      const double b0 = e[i], b1 = d[i + 1] - lam[c], b2 = i + 2 < k ? e[i + 1] : 0.0;
      if (std::fabs(b0) > std::fabs(a0)) {
        swapped[i] = 1;
        l[i] = a0 / b0;
        u0[i] = b0;
        u1[i] = b1;
        u2[i] = b2;
        a0 = a1 - l[i] * b1;
        a1 = a2 - l[i] * b2;
      } else {
        swapped[i] = 0;
        if (a0 == 0.0) a0 = tiny;
        l[i] = b0 / a0;
        u0[i] = a0;
        u1[i] = a1;
        u2[i] = a2;
        a0 = b1 - l[i] * a1;
        a1 = b2 - l[i] * a2;
      }
      a2 = 0.0;
    }
    u0[k - 1] = std::fabs(a0) < tiny ? tiny : a0;
    for (int i = 0; i < k; ++i) {
      seed = seed * 6364136223846793005ull + 1442695040888963407ull;
      x[i] = static_cast<double>(seed >> 11) * (1.0 / 9007199254740992.0) - 0.5;
    }
    for (int it = 0; it < 4; ++it) {
      if (it > 0)   // the start vector stands for L applied to a random one
        for (int i = 0; i + 1 < k; ++i) {
          if (swapped[i]) std::swap(x[i], x[i + 1]);
          x[i + 1] -= l[i] * x[i];
        }
      for (int i = k - 1; i >= 0; --i) {
        double s = x[i];
        if (i + 1 < k) s -= u1[i] * x[i + 1];
        if (i + 2 < k) s -= u2[i] * x[i + 2];
        x[i] = s / u0[i];
      }
      auto normalise = [&]() {
        double m = 0.0, s = 0.0;
        for (double t : x) m = std::max(m, std::fabs(t));
        for (double& t : x) {
          t /= m;
          s += t * t;
        }
        s = 1.0 / std::sqrt(s);
        for (double& t : x) t *= s;
      };
      normalise();
      bool close = false;
      for (int q = 0; q < c; ++q) {
        if (std::fabs(lam[q] - lam[c]) > 1e-3) continue;
        close = true;
        const double* w = z.data() + static_cast<size_t>(q) * k;
        double dot = 0.0;
        for (int i = 0; i < k; ++i) dot += w[i] * x[i];
        for (int i = 0; i < k; ++i) x[i] -= dot * w[i];
      }
      if (close) normalise();
    }
    std::copy(x.begin(), x.end(), v);
  }
}

// Number of eigenvalues below x (Sturm sequence); e2: squared off-diagonal.
int sturm_count(const std::vector<double>& d, const std::vector<double>& e2, double x) {
  int cnt = 0;
  double q = 1.0;
  for (size_t i = 0; i < d.size(); ++i) {
    q = d[i] - x - (i > 0 ? e2[i - 1] / q : 0.0);
    if (q == 0.0) q = 1e-300;
    cnt += q < 0.0;
  }
  return cnt;
}

// Residual estimate |beta_last z_last| of the Ritz pair at the boundary of `passes`: the
// smallest t in [lo, hi] for which passes(t) holds, by bisection to 1e-13, times sign.
// O(k) per probe: a check far from convergence costs no QL sweep over all eigenvalues.
template <typename F>
double boundary_residual(const std::vector<double>& d, const std::vector<double>& e, double beta_last,
                         double lo, double hi, double sign, F passes, double* theta = nullptr) {
  while (hi - lo > 1e-13) {
    const double mid = 0.5 * (lo + hi);
    (passes(mid) ? hi : lo) = mid;
  }
  std::vector<double> z;
  const double t = sign * 0.5 * (lo + hi);
  if (theta) *theta = t;
  tridiag_vectors(d, e, &t, 1, z);
  return std::fabs(beta_last * z.back());
}

std::vector<double> squares(const std::vector<double>& e) {
  std::vector<double> s(e);
  for (double& x : s) x *= x;
  return s;
}

// extreme Ritz estimate: max over the two ends of |theta| + residual, where the
// residual of a Ritz pair is |beta_last * (last component of its vector)|
// (eigenvalues and last components by implicit QL, O(k^2) per check); *plain is the
// larger |theta| alone
double ritz_bound(const std::vector<double>& alpha, const std::vector<double>& beta, int k,
                  double beta_last, double* worst_res, double* plain) {
  std::vector<double> d(alpha.begin(), alpha.begin() + k), zl;
  std::vector<double> e(beta.begin(), beta.begin() + std::min<size_t>(beta.size(), k));
  if (!tridiag_eigen(d, e, zl)) {
    *worst_res = 1.0;   // no answer: report as unconverged
    *plain = 1.0;
    return 1.0;
  }
  int imax = 0, imin = 0;
  for (int i = 1; i < k; ++i) {
    if (d[i] > d[imax]) imax = i;
    if (d[i] < d[imin]) imin = i;
  }
  const double rmax = std::fabs(beta_last * zl[imax]);
  const double rmin = std::fabs(beta_last * zl[imin]);
  *worst_res = std::max(rmax, rmin);
  *plain = std::max(std::fabs(d[imax]), std::fabs(d[imin]));
  return std::max(std::fabs(d[imax]) + rmax, std::fabs(d[imin]) + rmin);
}

// `runs` Lanczos runs side by side from seeds seed0, ...: lambda* estimate and whether
// both ends passed the residual test, per run.
int lambda_runs(sc_graph* g, hipStream_t st, int kmax, int seed0, int runs, double* result,
                bool* converged) {
  const int64_t n = g->d.n;
  constexpr int kWindow = 20;
  LanczosDriver lz;
  const hipError_t e0 = lz.start(g->d, g->deg_h.data(), seed0, runs, kmax, st);
  if (e0 != hipSuccess)
    return fail(e0 == hipErrorOutOfMemory ? SC_ENOMEM : SC_EHIP, "lanczos allocation failed");
  std::vector<double> al, be;
  std::vector<char> done(runs, 0);
  int open = runs;   // runs not done
  HIP_TRY(lz.advance(lz.kProbe));
  for (int checked = 0; checked < kmax && open > 0;) {
    if (lz.taken >= lz.kProbes && lz.enqueued < kmax)
      HIP_TRY(lz.advance(kWindow));   // beside the evaluation
    int q = 0, upto = 0;
    HIP_TRY(lz.take(&q, &upto));
    for (int r = 0; r < runs; ++r) {
      if (done[r]) continue;
      const int ex = lz.exhausted(q, r, checked, upto);
      const int j = ex ? ex : upto;
      const double b_j = lz.beta(q, r, j);
      const bool closed = ex || j == n - 1;   // the Krylov space is all there is
      const bool last = closed || j == kmax;
      if (lz.probing() && !last) continue;   // checked every kWindow steps
      al.resize(j);
      be.resize(j - 1);
      for (int i = 1; i <= j; ++i) al[i - 1] = lz.alpha(q, r, i);
      for (int i = 1; i < j; ++i) be[i - 1] = lz.beta(q, r, i);
      double res = 0.0;
      if (!last) {   // an end still far from converged ends the check here
        const int k = j;
        const std::vector<double> e2 = squares(be);
        res = boundary_residual(al, be, b_j, -1.1, 1.1, 1.0,
                                [&](double t) { return sturm_count(al, e2, t) == k; });
        if (res > 1e-7) continue;
        res = boundary_residual(al, be, b_j, -1.1, 1.1, 1.0,
                                [&](double t) { return sturm_count(al, e2, t) > 0; });
        if (res > 1e-7) continue;
      }
      double plain = 0.0;
      result[r] = ritz_bound(al, be, j, closed ? 0.0 : b_j, &res, &plain);
      converged[r] = closed || res < 1e-9;
      // at the step limit the residual can reach past 1, where it bounds nothing: the
      // Ritz value alone then, reported as not converged
      if (last && !converged[r] && result[r] >= 1.0) result[r] = plain;
      if (last || converged[r]) {
        done[r] = 1;
        --open;
      }
    }
    checked = upto;
    if (lz.probing() && open > 0) HIP_TRY(lz.after_probe(kWindow));
  }
  HIP_TRY(hipStreamSynchronize(st));
  return SC_OK;
}

}  // namespace

int sc::compute_lambda_star(sc_graph* g, hipStream_t st, double* out) {
  // two Lanczos runs from independent start vectors; the larger estimate is kept (a
  // start vector nearly orthogonal to the extreme eigenvector would make one run
  // under-estimate), converged only if both runs passed the residual test.  Side by
  // side, they share the launches; where there is no memory for both bases, one after
  // the other with the same results (each basis up to 600 steps, held to 4 GiB)
  const int64_t n = g->d.n;
  const int64_t kcap = std::max<int64_t>(40, (int64_t(1) << 29) / std::max<int64_t>(n, 1) - 2);
  const int kmax = static_cast<int>(std::min<int64_t>({n - 1, 600, kcap}));
  double result[2] = {-1.0, -1.0};
  bool converged[2] = {};
  int rc = lambda_runs(g, st, kmax, 0, 2, result, converged);
  if (rc == SC_ENOMEM) {
    rc = lambda_runs(g, st, kmax, 0, 1, result, converged);
    if (rc == SC_OK) rc = lambda_runs(g, st, kmax, 1, 1, result + 1, converged + 1);
  }
  if (rc) return rc;
  for (double r : result)
    if (!(r > 0.0) || !(r < 1.0))
      return fail(SC_EINVAL, "lambda* estimate outside (0, 1): " + std::to_string(r) +
                                 " (graph bipartite or too small?)");
  *out = std::max(result[0], result[1]);
  g->lambda_converged = (converged[0] && converged[1]) ? 1 : 0;
  return SC_OK;
}

int sc::graph_lambda_star(sc_graph* g, hipStream_t st, double* lam) {
  if (g->lambda_star <= 0.0) {
    double v = 0.0;
    const int rc = compute_lambda_star(g, st, &v);
    if (rc != SC_OK) return rc;
    g->lambda_star = v;
  }
  *lam = g->lambda_star;
  return SC_OK;
}

// Lanczos with full re-orthogonalisation (twice) on N = D^-1/2 A D^-1/2 with
// the trivial eigenvector deflated.  Every 25 steps the Ritz values of the
// tridiagonal matrix are checked: the run stops when the omega - 1 of largest
// |theta| have residual estimates |beta_j y_j| <= tol (or after max_iter steps,
// or when the Krylov space is exhausted).  The longest prefix (|theta|
// descending) of pairs within tol is kept, with the trivial pair in front.
int sc::lanczos_spectrum(sc_graph* g, int omega, int max_iter, double tol, hipStream_t st,
                         int* kept, double* worst) {
  const sc::DeviceGraph& dg = g->d;
  const int64_t n = dg.n;
  // the basis is held whole: at most ~16 GiB of it
  const int64_t cap = std::max<int64_t>(omega + 8, (int64_t(16) << 30) / (8 * n) - 2);
  const int kmax = static_cast<int>(std::min<int64_t>({n - 1, static_cast<int64_t>(max_iter), cap}));
  constexpr int kWindow = 25;
  LanczosDriver lz;
  hipError_t e = lz.start(dg, g->deg_h.data(), 0, 1, kmax, st);
  if (e != hipSuccess)
    return fail(e == hipErrorOutOfMemory ? SC_ENOMEM : SC_EHIP, "spectrum: allocation failed");
  const int want = omega - 1;
  // Ritz pairs ordered by |theta| descending (ties: theta descending)
  auto order_of = [](const std::vector<double>& th) {
    std::vector<int> idx(th.size());
    for (size_t i = 0; i < idx.size(); ++i) idx[i] = static_cast<int>(i);
    std::sort(idx.begin(), idx.end(), [&](int a, int b) {
      const double fa = std::fabs(th[a]), fb = std::fabs(th[b]);
      return fa > fb || (fa == fb && th[a] > th[b]);
    });
    return idx;
  };
  std::vector<double> alpha, beta, th, zl;
  int steps = 0;
  double b_last = 0.0;
  HIP_TRY(lz.advance(lz.kProbe));
  for (int checked = 0;;) {
    if (lz.taken >= lz.kProbes && lz.enqueued < kmax)
      HIP_TRY(lz.advance(kWindow));   // beside the evaluation
    int q = 0, upto = 0;
    HIP_TRY(lz.take(&q, &upto));
    const int ex = lz.exhausted(q, 0, checked, upto);
    steps = ex ? ex : upto;
    b_last = lz.beta(q, 0, steps);
    if (!(b_last >= 0.0)) b_last = 0.0;
    alpha.resize(steps);
    beta.resize(steps - 1);
    for (int i = 1; i <= steps; ++i) alpha[i - 1] = lz.alpha(q, 0, i);
    for (int i = 1; i < steps; ++i) beta[i - 1] = lz.beta(q, 0, i);
    checked = upto;
    if (ex || steps == kmax) break;
    if (lz.probing()) {
      HIP_TRY(lz.after_probe(kWindow));
    } else if (steps >= want) {
      // the pair of want-th largest |theta| first: the largest t with fewer than `want`
      // eigenvalues of magnitude above it
      const std::vector<double> e2 = squares(beta);
      auto above = [&](double t) {
        return steps - sturm_count(alpha, e2, t) + sturm_count(alpha, e2, -t);
      };
      double at = 0.0;
      const double rp = boundary_residual(alpha, beta, b_last, 0.0, 1.1, 1.0,
                                          [&](double t) { return above(t) < want; }, &at);
      const double rn = boundary_residual(alpha, beta, b_last, at, at, -1.0,
                                          [](double) { return true; });
      // the pair's sign is not known: the nearer eigenvalue answers with its own residual,
      // the other end's start vector converges to some other pair
      if (std::min(rp, rn) > 100.0 * tol) continue;
      th = alpha;
      if (!tridiag_eigen(th, beta, zl)) break;
      const std::vector<int> idx = order_of(th);
      bool done = true;
      for (int c = 0; c < want && done; ++c) done = std::fabs(b_last * zl[idx[c]]) <= tol;
      if (done) break;
    }
  }
  // Ritz pairs of the final tridiagonal matrix: all eigenvalues, the vectors of those kept
  th = alpha;
  if (!tridiag_eigen(th, beta, zl))
    return fail(SC_EINVAL, "spectrum: tridiagonal eigenvalues did not converge");
  const std::vector<int> idx = order_of(th);
  const bool exact = b_last < 1e-12;   // invariant subspace: the Ritz pairs are eigenpairs
  int p = 0;
  double wres = 0.0;
  while (p < want && p < steps) {
    const double r = exact ? 0.0 : std::fabs(b_last * zl[idx[p]]);
    if (r > tol) break;
    wres = std::max(wres, r);
    ++p;
  }
  if (p == 0)
    return fail(SC_EINVAL, "spectrum: no Ritz pair reached the tolerance (raise max_iter)");
  const int om = p + 1;
  const int p32 = (p + kRitzCols - 1) / kRitzCols * kRitzCols;
  std::vector<double> lam(om);
  lam[0] = 1.0;
  for (int c = 0; c < p; ++c) lam[1 + c] = th[idx[c]];
  std::vector<double> Z;
  tridiag_vectors(alpha, beta, lam.data() + 1, p, Z);
  std::vector<double> Y(static_cast<size_t>(steps) * p32, 0.0);
  for (int i = 0; i < steps; ++i)
    for (int c = 0; c < p; ++c) Y[static_cast<size_t>(i) * p32 + c] = Z[static_cast<size_t>(c) * steps + i];
  double* Yd = nullptr;
  double* lam_d = nullptr;
  double* phi_d = nullptr;
  e = dev_alloc(&Yd, Y.size());
  if (e == hipSuccess) e = dev_alloc(&lam_d, om);
  if (e == hipSuccess) e = dev_alloc(&phi_d, static_cast<size_t>(n) * om);
  if (e == hipSuccess)
    e = hipMemcpyAsync(Yd, Y.data(), Y.size() * sizeof(double), hipMemcpyHostToDevice, st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(lam_d, lam.data(), om * sizeof(double), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = sc::launch_ritz(n, n, lz.a.V, steps, Yd, p32, p, om, phi_d, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  dev_free(Yd);
  if (e != hipSuccess) {
    dev_free(lam_d);
    dev_free(phi_d);
    return fail(e == hipErrorOutOfMemory ? SC_ENOMEM : SC_EHIP,
                std::string("spectrum: ") + hipGetErrorString(e));
  }
  dev_free(g->spec_lam);
  dev_free(g->spec_phi);
  g->spec_lam = lam_d;
  g->spec_phi = phi_d;
  g->spec_omega = om;
  g->spec_lam_h = lam;
  ++g->spec_version;
  *kept = om;
  *worst = wres;
  return SC_OK;
}

extern "C" int sc_compute_spectrum(sc_graph* g, int omega, int max_iter, double tol,
                                   int* omega_kept, double* max_residual) {
  if (!g) return fail(SC_EINVAL, "graph is NULL");
  if (omega < 2 || omega > sc::kMaxOmega) return fail(SC_EINVAL, "omega must lie in [2, 256]");
  if (omega > g->d.n) omega = static_cast<int>(g->d.n);
  if (max_iter <= 0) max_iter = 2048;
  if (!(tol > 0.0)) tol = 1e-8;
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != g->device) (void)hipSetDevice(g->device);
  int kept = 0;
  double worst = 0.0;
  const int rc = sc::no_throw(
      [&] { return sc::lanczos_spectrum(g, omega, max_iter, tol, nullptr, &kept, &worst); });
  if (cur != g->device) (void)hipSetDevice(cur);
  if (rc) return rc;
  if (omega_kept) *omega_kept = kept;
  if (max_residual) *max_residual = worst;
  return SC_OK;
}

extern "C" int sc_set_spectrum(sc_graph* g, int omega, const double* lambda, const double* phi) {
  if (!g || !lambda || !phi) return fail(SC_EINVAL, "NULL argument");
  if (omega < 2 || omega > sc::kMaxOmega || omega > g->d.n)
    return fail(SC_EINVAL, "omega must lie in [2, min(n, 256)]");
  if (std::fabs(lambda[0] - 1.0) > 1e-8)
    return fail(SC_EINVAL, "lambda[0] must be the trivial eigenvalue 1");
  for (int k = 1; k < omega; ++k) {
    if (!(std::fabs(lambda[k]) < 1.0))
      return fail(SC_EINVAL, "non-trivial eigenvalues must lie in (-1, 1)");
    if (k >= 2 && std::fabs(lambda[k]) > std::fabs(lambda[k - 1]) * (1.0 + 1e-12))
      return fail(SC_EINVAL, "eigenvalues must be ordered by |lambda| descending");
  }
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != g->device) (void)hipSetDevice(g->device);
  const size_t cells = static_cast<size_t>(g->d.n) * omega;
  std::vector<double> stored;   // rows in the stored node order (renumbered graphs)
  if (!g->rank_h.empty()) {
    try {
      stored.resize(cells);
    } catch (const std::bad_alloc&) {
      if (cur != g->device) (void)hipSetDevice(cur);
      return fail(SC_ENOMEM, "host allocation failed");
    }
    for (int64_t x = 0; x < g->d.n; ++x)
      std::memcpy(stored.data() + static_cast<size_t>(g->rank_h[x]) * omega,
                  phi + static_cast<size_t>(x) * omega, omega * sizeof(double));
  }
  const double* phi_src = stored.empty() ? phi : stored.data();
  double* lam_d = nullptr;
  double* phi_d = nullptr;
  hipError_t e = sc::dev_alloc(&lam_d, omega);
  if (e == hipSuccess) e = sc::dev_alloc(&phi_d, cells);
  if (e == hipSuccess) e = hipMemcpy(lam_d, lambda, omega * sizeof(double), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(phi_d, phi_src, cells * sizeof(double), hipMemcpyHostToDevice);
  if (cur != g->device) (void)hipSetDevice(cur);
  if (e != hipSuccess) {
    sc::dev_free(lam_d);
    sc::dev_free(phi_d);
    return fail(e == hipErrorOutOfMemory ? SC_ENOMEM : SC_EHIP,
                std::string("set spectrum: ") + hipGetErrorString(e));
  }
  sc::dev_free(g->spec_lam);
  sc::dev_free(g->spec_phi);
  g->spec_lam = lam_d;
  g->spec_phi = phi_d;
  g->spec_omega = omega;
  g->spec_lam_h.assign(lambda, lambda + omega);
  ++g->spec_version;
  return SC_OK;
}

extern "C" int sc_get_spectrum(const sc_graph* g, int* omega, double* lambda, double* phi) {
  if (!g || !omega) return fail(SC_EINVAL, "NULL argument");
  *omega = g->spec_omega;
  if (g->spec_omega == 0) return SC_OK;
  if (lambda) std::memcpy(lambda, g->spec_lam_h.data(), g->spec_omega * sizeof(double));
  if (phi) {
    const int omega_s = g->spec_omega;
    const size_t cells = static_cast<size_t>(g->d.n) * omega_s;
    std::vector<double> stored;   // rows in the stored node order (renumbered graphs)
    if (!g->rank_h.empty()) {
      try {
        stored.resize(cells);
      } catch (const std::bad_alloc&) {
        return fail(SC_ENOMEM, "host allocation failed");
      }
    }
    int cur = 0;
    (void)hipGetDevice(&cur);
    if (cur != g->device) (void)hipSetDevice(g->device);
    const hipError_t e = hipMemcpy(stored.empty() ? phi : stored.data(), g->spec_phi,
                                   cells * sizeof(double), hipMemcpyDeviceToHost);
    if (cur != g->device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return fail(SC_EHIP, std::string("get spectrum: ") + hipGetErrorString(e));
    for (int64_t x = 0; !stored.empty() && x < g->d.n; ++x)
      std::memcpy(phi + static_cast<size_t>(x) * omega_s,
                  stored.data() + static_cast<size_t>(g->rank_h[x]) * omega_s,
                  omega_s * sizeof(double));
  }
  return SC_OK;
}

extern "C" int sc_lambda_star(sc_graph* g, double* lam) {
  if (!g || !lam) return fail(SC_EINVAL, "NULL argument");
  return sc::no_throw([&] { return sc::graph_lambda_star(g, nullptr, lam); });
}

extern "C" int sc_walk_trace(sc_graph* g, int32_t i, int32_t j, int64_t r, int32_t length,
                             uint64_t seed, int32_t* nodes_host) {
  if (!g || (!nodes_host && length > 0)) return fail(SC_EINVAL, "NULL argument");
  if (i < 0 || j < 0 || i >= g->d.n || j >= g->d.n) return fail(SC_EINVAL, "node id out of range");
  if (r < 0 || r > 0xFFFFFFFFll) return fail(SC_EINVAL, "walk index must lie in [0, 2^32)");
  if (length < 0 || length > (1 << 20)) return fail(SC_EINVAL, "length must lie in [0, 2^20]");
  if (length == 0) return SC_OK;
  const bool renumbered = !g->rank_h.empty();
  if (renumbered) {   // the stored nodes
    i = g->rank_h[i];
    j = g->rank_h[j];
  }
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != g->device) (void)hipSetDevice(g->device);
  int32_t* d = nullptr;
  int rc = SC_OK;
  {
    auto body = [&]() -> int {
      HIP_TRY(sc::dev_alloc(&d, 2 * static_cast<size_t>(length)));
      HIP_TRY(sc::launch_walk_trace(g->d, i, j, static_cast<uint32_t>(r), length, seed, d, nullptr));
      HIP_TRY(hipMemcpy(nodes_host, d, 2 * static_cast<size_t>(length) * sizeof(int32_t),
                        hipMemcpyDeviceToHost));
      return SC_OK;
    };
    rc = body();
  }
  sc::dev_free(d);
  if (cur != g->device) (void)hipSetDevice(cur);
  if (rc == SC_OK && renumbered)   // back to the caller's ids
    for (int64_t t = 0; t < 2 * static_cast<int64_t>(length); ++t) nodes_host[t] = g->label_h[nodes_host[t]];
  return rc;
}

// ====================================================================== all-edge SC

extern "C" void sc_default_options(sc_options* o) {
  if (!o) return;
  std::memset(o, 0, sizeof(*o));
  o->method = SC_TGT;
  o->precision = 0;
  o->block = 0;
  o->gamma = 10;
  o->delta = 0.0;
  o->seed = 0x5C5Cull;
  o->tilde_tau = -1;
  o->max_L = 255;
  o->lambda_star = 0.0;
  o->mlp = nullptr;
  o->infer_bf16 = 1;
  o->force_fallback = 0;
  o->sources = nullptr;
  o->nsources = 0;
  o->switch_rule = 0;
}

namespace sc {

PipeLayout pipe_layout(const sc_graph* g, int B, size_t tsize, int sets) {
  PipeLayout l;
  l.sets = sets;
  if (const char* b = std::getenv("SC_STEP_BITMAP_NODES"))   // other limits (tests)
    l.bitmap_nodes = std::max(0ll, std::min(240000ll, std::atoll(b)));
  if (const char* b = std::getenv("SC_STEP_BUFFER_BYTES"))
    l.buffer_bytes = std::min<uint64_t>(kBufferBytes, std::max(0ll, std::atoll(b)));
  const int64_t n = g->d.n;
  l.ystride = (n * B + 63) / 64 * 64;
  const size_t yb = static_cast<size_t>(l.ystride) * tsize;
  const int64_t nblocks = (n + B - 1) / B;
  int64_t group = static_cast<int64_t>(kGroupBytes / (2 * yb));
  group = std::max<int64_t>(group, kMinGroup);
  while (group > 1 && 2 * sets * group * yb > kPipeBudgetBytes) --group;
  group = std::min<int64_t>({group, nblocks, kMaxGroup});
  if (g->group_limit > 0)
    group = std::min<int64_t>(group, std::max<int64_t>(1, g->group_limit / (2 * yb)));
  // Where steps go by slices: whole rounds of the 8 XCDs (a block is tsize / 2 slices when
  // B = 64), or a count of slices that divides them, since the 6 slices of 3 blocks would
  // leave two XCDs idle (BA n = 600,000, k = 2, by slices: TGT L = 3 940 ms with 3 blocks,
  // 774 with 4; TGT+ 2,792 with 3, 2,385 with 2).  Steps by whole rows take any count (TGT+
  // 1,954 ms with 2 blocks, 1,828 with 3; n = 300,000, k = 3, L = 5: 580 with 4, 559 with 6).
  if (n <= l.bitmap_nodes) {
    const int64_t unit = std::max<int64_t>(1, 16 / static_cast<int64_t>(tsize));
    if (group > unit && group < nblocks) group = group / unit * unit;
    while (group < unit && group < nblocks && unit % group) --group;
  }
  l.group = static_cast<int>(group);
  l.tail_group = static_cast<int>(std::min<int64_t>(
      group, std::max<int64_t>(1, static_cast<int64_t>(kTailBytes / col_scratch_bytes(col_parts(n))))));
  return l;
}

namespace {

template <typename P>
hipError_t grow_zeroed(P** p, size_t* have, size_t want, hipStream_t st) {
  if (*p && *have >= want) return hipSuccess;
  dev_free(*p);
  *have = 0;
  hipError_t e = dev_alloc(p, want);
  if (e == hipSuccess) e = hipMemsetAsync(*p, 0, want * sizeof(P), st);
  if (e == hipSuccess) *have = want;
  return e;
}

// The sliced lists of DeviceGraph: rows of at most kChunk slots by degree
// (descending, ties by id), groups of 8.
int build_slice_lists(sc_graph* g, hipStream_t st) {
  DeviceGraph& d = g->d;
  if (d.slice_nb) return SC_OK;
  const int32_t n = d.n;
  std::vector<int32_t> first(kChunk + 2, 0), rows;
  std::vector<int2> grp;
  try {
    for (int32_t x = 0; x < n; ++x)
      if (g->deg_h[x] <= kChunk) ++first[kChunk - g->deg_h[x] + 1];
    for (int k = 0; k <= kChunk; ++k) first[k + 1] += first[k];
    const int32_t light = first[kChunk + 1];
    const int32_t ngrp = (light + 7) / 8;
    rows.assign(static_cast<size_t>(ngrp) * 8, n);
    for (int32_t x = 0; x < n; ++x)
      if (g->deg_h[x] <= kChunk) rows[first[kChunk - g->deg_h[x]]++] = x;
    grp.resize(ngrp);
    int64_t off = 0;
    for (int32_t k = 0; k < ngrp; ++k) {
      const int32_t width = (g->deg_h[rows[8 * k]] + 3) / 4 * 4;
      grp[k] = make_int2(static_cast<int>(off), width);   // below 2^31 / 8 + n / 8 chunks
      off += (width + 7) / 8;
    }
    std::vector<float> invf(rows.size(), 0.0f);
    std::vector<double> invd(rows.size(), 0.0);
    for (size_t r = 0; r < rows.size(); ++r)
      if (rows[r] < n) {
        invf[r] = 1.0f / static_cast<float>(g->deg_h[rows[r]]);
        invd[r] = 1.0 / static_cast<double>(g->deg_h[rows[r]]);
      }
    d.nslice_grp = ngrp;
    auto up = [&](auto** dst, const auto& src) -> hipError_t {
      hipError_t e = dev_alloc(dst, src.size());
      if (e == hipSuccess && !src.empty())
        e = hipMemcpyAsync(*dst, src.data(), src.size() * sizeof(src[0]), hipMemcpyHostToDevice, st);
      return e;
    };
    hipError_t e = up(&d.slice_grp, grp);
    if (e == hipSuccess) e = up(&d.slice_row, rows);
    if (e == hipSuccess) e = up(&d.slice_inv_f, invf);
    if (e == hipSuccess) e = up(&d.slice_inv_d, invd);
    int32_t* nb = nullptr;
    if (e == hipSuccess) e = dev_alloc(&nb, 64 * static_cast<size_t>(off));
    if (e == hipSuccess) {
      d.slice_nb = nb;
      e = launch_fill_slices(d, st);
    }
    const hipError_t done = hipStreamSynchronize(st);   // the host arrays end here
    if (e == hipSuccess) e = done;
    if (e != hipSuccess) {   // nothing is kept: a later call finds all of it or none
      dev_free(d.slice_grp);
      dev_free(d.slice_row);
      dev_free(d.slice_inv_f);
      dev_free(d.slice_inv_d);
      dev_free(d.slice_nb);
      return fail(e == hipErrorOutOfMemory ? SC_ENOMEM : SC_EHIP,
                  std::string("neighbour lists: ") + hipGetErrorString(e));
    }
  } catch (const std::bad_alloc&) {
    return fail(SC_ENOMEM, "host allocation failed");
  }
  return SC_OK;
}

}  // namespace

int ensure_narrow_ids(sc_graph* g, hipStream_t st) {
  sc::DeviceGraph& d = g->d;
  if (d.col16 || d.n > 65536) return SC_OK;
  uint16_t* c = nullptr;
  hipError_t e = sc::dev_alloc(&c, static_cast<size_t>(d.nslots));
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    return SC_OK;
  }
  if (e == hipSuccess) e = sc::launch_narrow(d.col, c, d.nslots, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);   // once: later calls may use other streams
  if (e != hipSuccess) {
    sc::dev_free(c);
    return sc::fail(SC_EHIP, std::string("narrow ids: ") + hipGetErrorString(e));
  }
  d.col16 = c;
  return SC_OK;
}

bool shrink_groups(sc_graph* g, int B, size_t tsize, hipStream_t st) {
  const PipeLayout l = pipe_layout(g, B, tsize, 1);
  if (l.group <= 1) return false;
  // what the failed call has enqueued still reads the buffers
  if (hipStreamSynchronize(st) != hipSuccess) return false;
  if (g->tail_stream && hipStreamSynchronize(g->tail_stream) != hipSuccess) return false;
  g->group_limit = 2 * static_cast<size_t>(l.ystride) * tsize * (l.group / 2);
  if (g->Y) (void)tracked_free(g->Y);
  g->Y = nullptr;
  g->ybytes = 0;
  if (g->partials) (void)tracked_free(g->partials);
  g->partials = nullptr;
  g->pbytes = 0;
  dev_free(g->nz);
  g->nz_bytes = 0;
  dev_free(g->mask);
  g->mask_words = 0;
  dev_free(g->anymask);
  g->anymask_words = 0;
  g->mask_clean = false;
  g->mask_pending = BlockList{};
  dev_free(g->tail.col);
  g->tail_blocks = 0;
  return true;
}

int ensure_buffers(sc_graph* g, int B, size_t tsize, int sets, hipStream_t st) {
  using namespace sc;
  const int64_t n = g->d.n;
  const int64_t S = static_cast<int64_t>(g->rowptr_h[n]);
  const PipeLayout lay = pipe_layout(g, B, tsize, sets);
  const size_t yb = 2 * static_cast<size_t>(lay.bufs()) * lay.ystride * tsize;
  if (yb > g->ybytes) {
    if (g->Y) (void)sc::tracked_free(g->Y);
    g->Y = nullptr;
    g->ybytes = 0;
    HIP_TRY(sc::tracked_malloc(&g->Y, yb));
    g->ybytes = yb;
  }
  if (B == 64) {
    const int rc = build_slice_lists(g, st);
    if (rc) return rc;
    const size_t nzb = static_cast<size_t>(lay.bufs()) * (tsize / 2) * flag_stride(n);
    HIP_TRY(grow_zeroed(&g->nz, &g->nz_bytes, nzb, st));
  }
  const size_t pb = static_cast<size_t>(lay.bufs()) * std::max(g->d.nparts, 1) * B * tsize;
  if (pb > g->pbytes) {
    if (g->partials) (void)sc::tracked_free(g->partials);
    g->partials = nullptr;
    g->pbytes = 0;
    HIP_TRY(sc::tracked_malloc(&g->partials, pb));
    g->pbytes = pb;
  }
  const size_t mw = 2 * static_cast<size_t>(lay.group) * n;
  const size_t aw = 2 * static_cast<size_t>(lay.group) * ((n + 31) / 32);
  if (!g->mask_clean || mw > g->mask_words || aw > g->anymask_words) {
    // new words, or a call that failed between setting bits and clearing them
    g->mask_clean = false;
    g->mask_pending = BlockList{};
    if (mw > g->mask_words) {
      dev_free(g->mask);
      g->mask_words = 0;
      HIP_TRY(dev_alloc(&g->mask, mw));
      g->mask_words = mw;
    }
    if (aw > g->anymask_words) {
      dev_free(g->anymask);
      g->anymask_words = 0;
      HIP_TRY(dev_alloc(&g->anymask, aw));
      g->anymask_words = aw;
    }
    HIP_TRY(launch_fill_u64(reinterpret_cast<uint64_t*>(g->mask),
                            static_cast<int64_t>(g->mask_words), 0, st));
    HIP_TRY(launch_fill_u32(g->anymask, static_cast<int64_t>(g->anymask_words), 0, st));
    g->mask_clean = true;
  }
  if (!g->gacc) HIP_TRY(dev_alloc(&g->gacc, S));
  if (!g->tau_slot) HIP_TRY(dev_alloc(&g->tau_slot, S));
  if (!g->tau_row) HIP_TRY(dev_alloc(&g->tau_row, n + 4));
  if (!g->nr_slot) HIP_TRY(dev_alloc(&g->nr_slot, S));
  if (!g->work) HIP_TRY(dev_alloc(&g->work, 4));   // [0..1] walk totals, [2] capped halves (learned)
  if (!g->plan_work) HIP_TRY(dev_alloc(&g->plan_work, 4 * 2 * 64));
  if (!g->out_dev) HIP_TRY(dev_alloc(&g->out_dev, g->d.m));
  if (!g->tau_host)
    HIP_TRY(hipHostMalloc(reinterpret_cast<void**>(&g->tau_host),
                          (static_cast<size_t>(n) + 8) * sizeof(int32_t)));
  for (auto& e : g->call_ev)
    if (!e) HIP_TRY(hipEventCreate(&e));
  return SC_OK;
}

int ensure_tail(sc_graph* g, int blocks, bool walks) {
  const int64_t n = g->d.n, S = g->d.nslots;
  TailScratch& t = g->tail;
  if (!t.ctl) {
    t.nparts = col_parts(n);
    t.col_bytes = col_scratch_bytes(t.nparts);
    // flattened walks: the chunk sums of a launch (a block whose sums do not fit
    // walks one slot per wave)
    t.capacity = std::min<int64_t>(int64_t(1) << 22, 4 * S + 65536);
    if (const char* cap = std::getenv("SC_WALK_CHUNK_CAPACITY"))   // smaller buffer (tests)
      t.capacity = std::max<int64_t>(1, std::min<int64_t>(t.capacity, std::atoll(cap)));
    HIP_TRY(dev_alloc(&t.ctl, static_cast<size_t>(kMaxGroup)));
  }
  if (!t.cs) HIP_TRY(dev_alloc(&t.cs, static_cast<size_t>(kMaxGroup) * 64));
  if (static_cast<size_t>(blocks) > g->tail_blocks) {
    dev_free(t.col);
    g->tail_blocks = 0;
    HIP_TRY(dev_alloc(&t.col, t.col_bytes * blocks));
    g->tail_blocks = blocks;
  }
  if (walks) {
    if (!t.chunk_off) HIP_TRY(dev_alloc(&t.chunk_off, S + n / 16 + 2));
    if (!t.part) HIP_TRY(dev_alloc(&t.part, static_cast<size_t>(t.capacity)));
  }
  return SC_OK;
}

int ensure_pipeline(sc_graph* g) {
  if (!g->tail_stream) HIP_TRY(hipStreamCreateWithFlags(&g->tail_stream, hipStreamNonBlocking));
  for (auto& e : g->pipe_ev)
    if (!e) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  return SC_OK;
}

}  // namespace sc

namespace {

using sc::Runner;

// Switch-step cost model.  The traversal of a block runs on the critical
// stream, its tail (candidate summary, walk counts, walks) on the tail stream,
// so a block costs about max(traversal, tail) plus an interference share of
// the shorter one.  Constants are whole-GPU rates measured on MI355X with one
// block per launch; a block of a group takes less of each, in about the same
// proportions, and the choice (which the results depend on) has stayed the best
// one (BA n = 100,000, eps = 1e-3, ms with switch steps 3, 4, 5, 6: 439, 174, 223,
// 294, 4 chosen; G(n, m) n = 10,000 with 3, 4, 5: 2.09, 2.69, 2.02, 5 chosen).
// The environment can override them for tuning.
struct CostModel {
  double gather_bw;     // bytes/s of neighbour-row gathers in a dense step
  double step_fixed;    // s of fixed cost per dense step
  double twohop_frac;   // two-hop step cost relative to a dense step
  double skip_frac;     // first dense step (zero rows skipped, B = 64) relative to a dense step
  double tail_fixed;    // s of a block's tail launches besides the walks (their
                        // chain of small launches under the traversal's load) ...
  double tail_per_node; // ... plus this many s per node (passes over the block state)
  double walk_step;     // s per single-walk step
  double overlap;       // share of the shorter stream that still costs time
};

CostModel cost_model() {
  CostModel c{7.5e12, 3.0e-6, 0.3, 0.6, 5.5e-5, 3.5e-10, 2.5e-11, 0.25};
  if (const char* s = std::getenv("SC_COST_GATHER_BW")) c.gather_bw = std::atof(s);
  if (const char* s = std::getenv("SC_COST_STEP_FIXED")) c.step_fixed = std::atof(s);
  if (const char* s = std::getenv("SC_COST_SKIP_FRAC")) c.skip_frac = std::atof(s);
  if (const char* s = std::getenv("SC_COST_TAIL_FIXED")) c.tail_fixed = std::atof(s);
  if (const char* s = std::getenv("SC_COST_TAIL_PER_NODE")) c.tail_per_node = std::atof(s);
  if (const char* s = std::getenv("SC_COST_WALK_STEP")) c.walk_step = std::atof(s);
  if (const char* s = std::getenv("SC_COST_OVERLAP")) c.overlap = std::atof(s);
  return c;
}

// The switch step by the cost model: walk steps at every candidate, sampled on up to
// four blocks (traversed as one group).
template <typename T>
int plan_switch(sc_graph* g, Runner<T>& R, const int32_t* tau_row, int Lmax, int gamma,
                double coef, int64_t nr_cap, int* tilde_out) {
  const int B = R.B;
  const int64_t n = g->d.n;
  hipStream_t st = R.st;
  const int nblocks = static_cast<int>((n + B - 1) / B);
  const CostModel cm = cost_model();
  const double dense = cm.step_fixed + static_cast<double>(g->d.nslots) * B * sizeof(T) / cm.gather_bw;
  const double tail0 = cm.tail_fixed + cm.tail_per_node * static_cast<double>(n);
  const int nsamp = std::min(nblocks, 4);
  constexpr int kSlots = 2 * 64;   // counters of a sample
  std::vector<double> cost(Lmax + 1, 0.0);
  std::vector<unsigned long long> wk(static_cast<size_t>(nsamp) * kSlots, 0ull);
  std::vector<int> tmaxs(nsamp, 0);
  HIP_TRY(hipMemsetAsync(g->plan_work, 0, nsamp * kSlots * sizeof(unsigned long long), st));
  const int step = std::min({nsamp, R.lay.bufs(), R.lay.group, R.lay.tail_group});
  int rc = sc::ensure_tail(g, step, false);
  if (rc) return rc;
  for (int s = 0; s < nsamp; s += step) {
    sc::BlockList list;
    int tmax_of[sc::kMaxGroup], sample_of[sc::kMaxGroup], to2[sc::kMaxGroup];
    int tmax_all = 0;
    for (int si = s; si < std::min(nsamp, s + step); ++si) {
      sc::BlockRef r = R.block_ref(static_cast<int>((si + 0.5) * nblocks / nsamp), tau_row, &tmaxs[si]);
      if (tmaxs[si] < 3) continue;
      r.buf = list.nb;
      tmax_of[list.nb] = tmaxs[si];
      sample_of[list.nb] = si;
      to2[list.nb] = 2;
      tmax_all = std::max(tmax_all, tmaxs[si]);
      list.b[list.nb++] = r;
    }
    if (list.nb == 0) continue;
    rc = R.traverse(list, to2, false, nullptr);
    if (rc) return rc;
    for (int ell = 2; ell < tmax_all && ell <= Lmax && ell < 64; ++ell) {
      sc::BlockList on;   // the samples that have a step beyond ell
      int on_sample[sc::kMaxGroup];
      for (int i = 0; i < list.nb; ++i)
        if (ell < tmax_of[i]) {
          on_sample[on.nb] = sample_of[i];
          on.b[on.nb++] = list.b[i];
        }
      if (ell > 2) {
        rc = R.advance(on);
        if (rc) return rc;
      }
      HIP_TRY(sc::launch_colstats<T>(g->d, on, B, gamma, R.Y(R.par), R.lay.ystride, g->tail, st));
      HIP_TRY(sc::launch_walk_counts<T>(g->d, on, B, ell, gamma, coef, nr_cap, R.Y(R.par),
                                        R.lay.ystride, g->tail, g->tau_slot, g->nr_slot, st));
      for (int i = 0; i < on.nb; ++i) {
        sc::BlockList one;
        one.nb = 1;
        one.b[0] = on.b[i];
        HIP_TRY(sc::launch_work_totals(one, ell, g->tau_slot, g->nr_slot,
                                       g->plan_work + on_sample[i] * kSlots + 2 * ell, 0, st));
      }
    }
  }
  HIP_TRY(hipMemcpyAsync(wk.data(), g->plan_work, wk.size() * sizeof(unsigned long long),
                         hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  for (int si = 0; si < nsamp; ++si) {
    const int tmax = tmaxs[si];
    for (int ell = 2; ell <= Lmax; ++ell) {
      const int steps = std::min(ell, tmax);
      const double first = B == 64 ? cm.skip_frac : 1.0;   // l = 3
      const double trav =
          steps >= 2 ? cm.step_fixed +
                           dense * (cm.twohop_frac + (steps >= 3 ? first + (steps - 3) : 0.0))
                     : 0.0;
      // switch points beyond the 64 counter slots are not candidates
      const double tail =
          ell < tmax
              ? (ell < 64 ? tail0 + static_cast<double>(wk[si * kSlots + 2 * ell + 1]) * cm.walk_step
                          : 1e30)
              : cm.step_fixed;
      cost[ell] += std::max(trav, tail) + cm.overlap * std::min(trav, tail);
    }
  }
  int tilde = Lmax;
  for (int ell = 2; ell <= Lmax; ++ell)
    if (cost[ell] < cost[tilde]) tilde = ell;
  *tilde_out = tilde;
  return SC_OK;
}

template <typename T>
int run_method(sc_graph* g, double eps, int L, const sc_options& o, double* out_user,
               sc_stats* st_user) {
  const int64_t n = g->d.n, m = g->d.m;
  hipStream_t st = static_cast<hipStream_t>(o.stream);
  const int B = o.block > 0 ? o.block : 64;
  if (B != 16 && B != 32 && B != 64) return fail(SC_EINVAL, "block must be 16, 32 or 64");
  const bool plus = o.method == SC_TGT_PLUS;
  const int gamma = o.gamma < 0 ? 10 : o.gamma;
  if (gamma > sc::kMaxGamma) return fail(SC_EINVAL, "gamma above 16 is not supported");
  int max_L = o.max_L > 0 ? o.max_L : 255;
  if (max_L % 2 == 0) --max_L;
  // TGT has no tails: its groups follow one another in one set of states
  const int sets = plus ? sc::kPipeSets : 1;
  int rc = sc::ensure_buffers(g, B, sizeof(T), sets, st);
  if (rc) return rc;
  const bool dev_ptrs = (o.flags & SC_DEVICE_PTRS) != 0;

  g->mask_clean = false;   // set again once the call's last clear is enqueued
  Runner<T> R{g, B, sets, st, (o.flags & SC_TIME_KERNELS) != 0};
  const sc::PipeLayout& lay = R.lay;
  R.stats.block = B;
  R.stats.tilde_tau = -1;
  R.stats.tilde_min = -1;
  R.stats.tilde_max = -1;
  R.stats.lambda_converged = -1;
  HIP_TRY(hipEventRecord(g->call_ev[0], st));

  // truncation policy: uniform L, CalTau with the graph's spectrum (Algorithm 1),
  // or the lambda*-bound (Algorithm 1 line 1)
  double lam = 0.0;
  int Lodd = 0;
  const bool spectral = L == 0 && (o.flags & SC_TAU_SPECTRAL) != 0;
  if (spectral && g->spec_omega < 2)
    return fail(SC_EINVAL, "SC_TAU_SPECTRAL needs a spectrum (sc_compute_spectrum or sc_set_spectrum)");
  if (L > 0) {
    Lodd = (L % 2 == 1) ? L : L + 1;
  } else if (spectral) {
    lam = std::fabs(g->spec_lam_h[1]);
  } else {
    if (o.lambda_star > 0.0) {
      lam = o.lambda_star;
    } else {
      rc = sc::graph_lambda_star(g, st, &lam);
      if (rc) return rc;
      R.stats.lambda_converged = g->lambda_converged;
    }
    if (!(lam > 0.0 && lam < 1.0)) return fail(SC_EINVAL, "lambda* must lie in (0, 1)");
  }
  R.stats.lambda_star = lam;
  const double eps_tau = plus ? eps / 2.0 : eps;
  // the capped count follows the rows' truncations, so that one copy brings both; it is
  // zeroed behind that copy for the next call
  const int64_t n_even = (n + 1) / 2 * 2;
  unsigned long long* capped = reinterpret_cast<unsigned long long*>(g->tau_row + n_even);
  unsigned long long* reset = nullptr;
  bool have_gacc = false;
  int32_t* const tau_row = g->tau_host;   // pinned: [n] row truncations, then the capped count
  if (L > 0) {
    // every edge has tau = Lodd: nothing to read back
    HIP_TRY(sc::launch_tau(g->d, Lodd, eps_tau, lam, max_L, g->tau_slot, g->tau_row, st, nullptr));
    std::fill(tau_row, tau_row + n, Lodd);
    R.stats.L_used = R.stats.L_min = Lodd;
  } else {
    if (!g->capped_clean)
      HIP_TRY(sc::launch_fill_u64(reinterpret_cast<uint64_t*>(capped), 1, 0, st));
    g->capped_clean = false;
    reset = capped;
    if (spectral)
      HIP_TRY(sc::launch_caltau(g->d, g->spec_lam, g->spec_phi, g->spec_omega, eps_tau, max_L,
                                g->tau_slot, g->tau_row, st, capped));
    else
      HIP_TRY(sc::launch_tau(g->d, Lodd, eps_tau, lam, max_L, g->tau_slot, g->tau_row, st, capped));
    const unsigned long long* capped_h =
        reinterpret_cast<const unsigned long long*>(tau_row + n_even);
    HIP_TRY(hipMemcpyAsync(tau_row, g->tau_row, (n_even + 2) * sizeof(int32_t),
                           hipMemcpyDeviceToHost, st));
    if (!plus) {   // what does not wait for the host goes ahead
      HIP_TRY(sc::launch_gacc_init(g->d, g->tau_slot, 1, g->gacc, st, nullptr, reset));
      have_gacc = true;
    }
    HIP_TRY(hipStreamSynchronize(st));
    R.stats.L_capped = static_cast<int64_t>(*capped_h / 2);   // both halves of an edge share tau
    int Lmax = 0, Lmin = 1 << 30;
    for (int64_t x = 0; x < n; ++x) {
      Lmax = std::max(Lmax, tau_row[x]);
      Lmin = std::min(Lmin, tau_row[x]);
    }
    R.stats.L_used = Lmax;
    R.stats.L_min = Lmin;
  }
  const int Lmax = R.stats.L_used;
  const int nblocks = static_cast<int>((n + B - 1) / B);

  int tilde = Lmax;
  double coef = 0.0;
  const int64_t nr_cap = (1ll << 31) - 1;
  if (plus) {
    const double delta = o.delta > 0.0 ? o.delta : 1.0 / static_cast<double>(n);
    // Eq. 13 constant; m counts distinct edges
    coef = 8.0 * std::log(static_cast<double>(g->d.nslots) / delta) / (eps * eps);
    const sc_graph::PlanKey key{eps,  L,     max_L, lam, B, static_cast<int>(sizeof(T)), gamma,
                                delta, spectral ? g->spec_version : 0};
    if (o.tilde_tau >= 0) {
      tilde = std::min(o.tilde_tau, Lmax);
    } else if (g->plan_valid && g->plan_key == key) {
      tilde = g->plan_tilde;   // the switch step depends only on the graph and these options
    } else {
      rc = plan_switch<T>(g, R, tau_row, Lmax, gamma, coef, nr_cap, &tilde);
      if (rc) return rc;
      g->plan_key = key;
      g->plan_tilde = tilde;
      g->plan_valid = true;
    }
    R.stats.tilde_tau = tilde;
    R.stats.tilde_min = tilde;
    R.stats.tilde_max = tilde;
  }
  if (!have_gacc)
    HIP_TRY(sc::launch_gacc_init(g->d, g->tau_slot, (plus && tilde < 1) ? 0 : 1, g->gacc, st,
                                 plus ? g->nr_slot : nullptr, reset));
  if (reset) g->capped_clean = true;
  R.ev_used = 0;
  R.stats.prop_launches = 0;
  R.stats.prop_bytes = 0.0;

  // Groups of blocks in source order.  A block whose edges all stop at tau <= 1 has
  // only the l = 0, 1 terms, which the accumulator initialisation already holds, and
  // is in no group.
  struct Group {
    sc::BlockList all, trav, tail;   // tail: blocks with edges beyond the switch step
    int lend[sc::kMaxGroup];         // last traversal step per block of trav
    uint32_t keep = 0;               // blocks of trav whose last state a tail reads
  };
  std::vector<Group> groups;
  bool any_tail = false;
  int max_tail = 0;
  for (int b = 0; b < nblocks; ++b) {
    int tmax;
    sc::BlockRef r = R.block_ref(b, tau_row, &tmax);
    const int lend = plus ? std::min(tmax, tilde) : tmax;
    const bool tail = plus && tmax > tilde;
    if (lend < 2 && !tail) continue;
    if (groups.empty() || groups.back().all.nb == lay.group) groups.emplace_back();
    Group& gr = groups.back();
    r.buf = static_cast<int>((groups.size() - 1) % lay.sets) * lay.group + gr.all.nb;
    gr.all.b[gr.all.nb++] = r;
    if (lend >= 2) {
      gr.lend[gr.trav.nb] = lend;
      if (tail) gr.keep |= 1u << gr.trav.nb;
      gr.trav.b[gr.trav.nb++] = r;
    }
    if (tail) {
      gr.tail.b[gr.tail.nb++] = r;
      any_tail = true;
      max_tail = std::max(max_tail, gr.tail.nb);
    }
  }
  if (any_tail) {
    rc = sc::ensure_tail(g, std::min(max_tail, lay.tail_group), true);
    if (rc) return rc;
  }
  // Pipeline: the traversals run on the caller's stream, a group's tails (candidate
  // summary, walk counts, walks) on the tail stream beside the next group's traversal.
  // The tails of a group wait for its traversal, and the traversal of group q waits
  // for the tails of group q - kPipeSets, whose states it reuses.  Blocks touch
  // disjoint slots of gacc and nr_slot.
  hipStream_t sb = st;
  if (any_tail) {
    rc = sc::ensure_pipeline(g);
    if (rc) return rc;
    sb = g->tail_stream;
    HIP_TRY(hipEventRecord(g->pipe_ev[0], st));
    HIP_TRY(hipStreamWaitEvent(sb, g->pipe_ev[0], 0));
  }
  const auto host0 = std::chrono::steady_clock::now();
  bool tail_recorded[sc::kPipeSets] = {};
  for (size_t q = 0; q < groups.size(); ++q) {
    const Group& gr = groups[q];
    const int qset = static_cast<int>(q % lay.sets);
    if (tail_recorded[qset])
      HIP_TRY(hipStreamWaitEvent(st, g->pipe_ev[1 + sc::kPipeSets + qset], 0));
    R.st = st;
    rc = R.traverse(gr.trav, gr.lend, true, g->gacc,
                    q + 1 < groups.size() ? &groups[q + 1].trav : nullptr, gr.keep);
    if (rc) return rc;
    if (gr.tail.nb == 0) {
      rc = R.flush_acc();
      if (rc) return rc;
      continue;
    }
    // the last step's accumulation rides on the candidate summary's first launch when
    // every block of the group that still has it pending is summarised there
    const bool fuse_acc = R.pending.list.nb == gr.tail.nb;
    if (!fuse_acc) {
      rc = R.flush_acc();
      if (rc) return rc;
    }
    const sc::AccJob last = R.pending;
    R.pending = sc::AccJob{};
    HIP_TRY(hipEventRecord(g->pipe_ev[1 + qset], st));
    HIP_TRY(hipStreamWaitEvent(sb, g->pipe_ev[1 + qset], 0));
    R.st = sb;
    if (tilde < 2) {
      rc = R.init_low(gr.tail, tilde);
      if (rc) return rc;
    }
    for (int t = 0; t < gr.tail.nb; t += lay.tail_group) {
      sc::BlockList part;
      for (int i = t; i < std::min(gr.tail.nb, t + lay.tail_group); ++i) part.b[part.nb++] = gr.tail.b[i];
      HIP_TRY(sc::launch_colstats<T>(g->d, part, B, gamma, R.Y(R.par), lay.ystride, g->tail, sb,
                                     fuse_acc ? &last : nullptr));
      HIP_TRY(sc::launch_walk_counts<T>(g->d, part, B, tilde, gamma, coef, nr_cap, R.Y(R.par),
                                        lay.ystride, g->tail, g->tau_slot, g->nr_slot, sb));
      HIP_TRY(sc::launch_walks<T>(g->d, part, B, tilde, o.seed, R.Y(R.par), lay.ystride,
                                  g->tau_slot, g->nr_slot, g->gacc, g->tail, sb));
    }
    HIP_TRY(hipEventRecord(g->pipe_ev[1 + sc::kPipeSets + qset], sb));
    tail_recorded[qset] = true;
    R.st = st;
  }
  R.st = st;
  R.stats.host_ms =
      std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - host0).count();
  if (any_tail) {
    HIP_TRY(hipEventRecord(g->pipe_ev[0], sb));
    HIP_TRY(hipStreamWaitEvent(st, g->pipe_ev[0], 0));
  }
  rc = R.flush_masks();
  if (rc) return rc;
  g->mask_clean = true;
  double* out_dev = dev_ptrs ? out_user : g->out_dev;
  HIP_TRY(sc::launch_combine(g->d, g->gacc, out_dev, st));
  HIP_TRY(hipEventRecord(g->call_ev[1], st));

  // traces
  int32_t* tau_o = nullptr;
  int64_t* nr_o = nullptr;
  if (o.tau_out) {
    if (!dev_ptrs && !g->tau_out_dev) HIP_TRY(dev_alloc(&g->tau_out_dev, m));
    tau_o = dev_ptrs ? o.tau_out : g->tau_out_dev;
  }
  if (o.nr_out) {
    if (!dev_ptrs && !g->nr_out_dev) HIP_TRY(dev_alloc(&g->nr_out_dev, 2 * m));
    nr_o = dev_ptrs ? o.nr_out : g->nr_out_dev;
  }
  HIP_TRY(sc::launch_trace(g->d, g->tau_slot, plus ? g->nr_slot : nullptr, tau_o, nr_o, st));
  std::vector<int32_t> tilde_h;
  if (o.tilde_tau_out) {
    tilde_h.resize(n);
    for (int64_t x = 0; x < n; ++x)   // in the caller's ids
      tilde_h[x] = plus ? tilde : tau_row[g->rank_h.empty() ? x : g->rank_h[x]];
    if (dev_ptrs)
      HIP_TRY(hipMemcpyAsync(o.tilde_tau_out, tilde_h.data(), n * sizeof(int32_t),
                             hipMemcpyHostToDevice, st));
    else
      std::memcpy(o.tilde_tau_out, tilde_h.data(), n * sizeof(int32_t));
  }
  unsigned long long wk[2] = {0, 0};
  if (any_tail) {
    unsigned long long* work = g->work;
    HIP_TRY(sc::launch_fill_u64(reinterpret_cast<uint64_t*>(work), 2, 0, st));
    sc::BlockList whole;
    whole.nb = 1;
    whole.b[0].kend = static_cast<int>(g->d.nslots);
    HIP_TRY(sc::launch_work_totals(whole, tilde, g->tau_slot, g->nr_slot, work, 0, st));
    HIP_TRY(hipMemcpyAsync(wk, work, sizeof(wk), hipMemcpyDeviceToHost, st));
  }
  if (!dev_ptrs) {
    HIP_TRY(hipMemcpyAsync(out_user, out_dev, m * sizeof(double), hipMemcpyDeviceToHost, st));
    if (o.tau_out)
      HIP_TRY(hipMemcpyAsync(o.tau_out, tau_o, m * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    if (o.nr_out)
      HIP_TRY(hipMemcpyAsync(o.nr_out, nr_o, 2 * m * sizeof(int64_t), hipMemcpyDeviceToHost, st));
  }
  HIP_TRY(hipStreamSynchronize(st));
  float ms = 0.0f;
  HIP_TRY(hipEventElapsedTime(&ms, g->call_ev[0], g->call_ev[1]));
  R.stats.total_ms = ms;
  R.stats.walks = plus ? static_cast<int64_t>(wk[0]) : 0;
  R.stats.walk_steps = plus ? static_cast<int64_t>(wk[1]) : 0;
  if (R.timing) {
    double tot = 0.0;
    for (size_t i = 0; i + 1 < R.ev_used; i += 2) {
      float t = 0.0f;
      HIP_TRY(hipEventElapsedTime(&t, g->events[i], g->events[i + 1]));
      tot += t;
    }
    R.stats.prop_ms = tot;
    R.stats.prop_timed = static_cast<int64_t>(R.ev_used / 2);
  }
  if (st_user) *st_user = R.stats;
  return SC_OK;
}

}  // namespace

extern "C" int sc_all_edges_ex(sc_graph* g, double eps, int L, const sc_options* o, double* out,
                               sc_stats* st) {
  if (!g) return fail(SC_EINVAL, "graph is NULL");
  if (!out) return fail(SC_EINVAL, "out is NULL");
  if (!(eps > 0.0 && eps < 1.0)) return fail(SC_EINVAL, "eps must lie in (0, 1)");
  if (L < 0) return fail(SC_EINVAL, "L must be >= 0");
  sc_options opt;
  if (o)
    opt = *o;
  else
    sc_default_options(&opt);
  if (opt.method != SC_TGT && opt.method != SC_TGT_PLUS && opt.method != SC_LEARNED)
    return fail(SC_EINVAL, "unknown method");
  if (opt.precision != 0 && opt.precision != 1) return fail(SC_EINVAL, "precision must be 0 or 1");
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != g->device) (void)hipSetDevice(g->device);
  if (opt.method == SC_LEARNED && (opt.flags & SC_TAU_SPECTRAL))
    return fail(SC_ENOTIMPL, "SC_TAU_SPECTRAL is not supported with SC_LEARNED");
  const bool per_source = (opt.flags & SC_PER_SOURCE) != 0;
  if (per_source && opt.method != SC_TGT_PLUS)
    return fail(SC_ENOTIMPL, "SC_PER_SOURCE runs TGT+ (method 1) only");
  if (opt.sources && !per_source) return fail(SC_EINVAL, "a source list needs SC_PER_SOURCE");
  const int rc = sc::no_throw([&] {
    if (per_source) return sc::run_per_source(g, eps, L, opt, out, st);
    if (opt.method == SC_LEARNED) return sc::run_learned(g, eps, opt, out, st);
    return sc::with_smaller_groups(
        g, opt.block > 0 ? opt.block : 64, opt.precision == 1 ? sizeof(double) : sizeof(float),
        static_cast<hipStream_t>(opt.stream), [&] {
          return opt.precision == 1 ? run_method<double>(g, eps, L, opt, out, st)
                                    : run_method<float>(g, eps, L, opt, out, st);
        });
  });
  if (cur != g->device) (void)hipSetDevice(cur);
  return rc;
}

extern "C" int sc_all_edges(sc_graph* g, double eps, int L, double* out) {
  sc_options o;
  sc_default_options(&o);
  o.method = L == 0 ? SC_TGT_PLUS : SC_TGT;
  return sc_all_edges_ex(g, eps, L, &o, out, nullptr);
}

extern "C" const char* sc_strerror(int code) {
  switch (code) {
    case SC_OK: return "ok";
    case SC_EINVAL: return "invalid argument";
    case SC_ESELFLOOP: return "self-loop in edge list";
    case SC_EDUP: return "duplicate edge";
    case SC_EDISCONNECTED: return "graph is not connected";
    case SC_EBIPARTITE: return "graph is bipartite";
    case SC_ENOMEM: return "out of memory";
    case SC_EHIP: return "HIP runtime error";
    case SC_ENOTIMPL: return "not implemented";
    default: return "unknown error code";
  }
}

extern "C" const char* sc_last_error(void) { return sc::g_last_error.c_str(); }

extern "C" const char* sc_version(void) { return "sc-mi355x 0.1 (gfx950)"; }
