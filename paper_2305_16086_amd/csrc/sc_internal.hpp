// Internal declarations shared by the host orchestration and the kernel
// translation units of libsc.  Not part of the public ABI (see include/sc.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "sc.h"

namespace sc {

// Row tasks of the gather kernels: a row with at most kChunk slots is one
// wave's task, a row with up to kGiant slots one workgroup's task, and a
// giant row is cut into workgroup chunks of kGiantChunk slots whose partial
// sums a fix-up pass adds in chunk order (deterministic, no atomics).
constexpr int kChunk = 256;
constexpr int kGiant = 4096;
constexpr int kGiantChunk = 1024;
constexpr int kWavesPerBlock = 4;     // 256-thread workgroups
constexpr int kMaxGamma = 16;         // candidate lists kept in registers

struct Task {
  int32_t row;
  int32_t beg;      // first CSR slot
  int32_t end;      // one past the last CSR slot
  int32_t part;     // -1: whole row; else index of this chunk's partial-sum row
};

struct HeavyRow {
  int32_t row;
  int32_t part0;    // first partial row
  int32_t nparts;   // number of chunks
  int32_t pad;
};

// Per-column summary of q = p_tilde(., s_c) used by Algorithm 3 / Lemma 4.3.
struct ColStats {
  double maxV, minV;     // max / min over all nodes
  double rho;            // upper bound on rho_i (Eq. 16), safe reading of Alg. 3
  double maxN, minN;     // max / min over N(s_c)
};

// A block's state is cut into slices of one 128-byte line per row (32 FP32 or 16 FP64
// columns).  Work that reads one slice is laid out so that workgroup w, which runs on
// XCD w mod 8, takes slice w mod 8 (+ 8, 16, ...) of the launch: an XCD's 4 MB L2 then
// holds lines of one slice at a time.  Each slice has slice_wgs workgroups in the
// whole rounds of 8 slices; the remaining 1..7 slices have rem_wgs each, on 8, 4, 2 or
// 1 XCDs.
struct SliceGrid {
  int nslices = 0, slice_wgs = 0, rem_wgs = 0;
  // XCDs per slice when rem (1..7) slices share the eight
  __host__ __device__ static int rem_xcds(int rem) {
    return rem > 4 ? 1 : rem > 2 ? 2 : rem > 1 ? 4 : 8;
  }
  __host__ __device__ int size() const {
    const int rem = nslices & 7;
    const int k = rem ? rem_xcds(rem) : 1;
    return 8 * (nslices >> 3) * slice_wgs + (rem ? 8 * ((rem_wgs + k - 1) / k) : 0);
  }
  // slice, workgroup of the slice and workgroups of the slice of workgroup w; false: none
  __device__ bool decode(int w, int* sl, int* wg, int* wgs) const {
    const int x = w & 7, j = w >> 3;
    const int rounds = nslices >> 3, rem = nslices & 7;
    if (j < rounds * slice_wgs) {
      *sl = x + 8 * (j / slice_wgs);
      *wg = j % slice_wgs;
      *wgs = slice_wgs;
      return true;
    }
    const int k = rem_xcds(rem);
    if (x / k >= rem) return false;
    *sl = 8 * rounds + x / k;
    *wg = (j - rounds * slice_wgs) * k + x % k;
    *wgs = rem_wgs;
    return *wg < rem_wgs;
  }
};

// The source blocks of one launch.  Block i covers sources s0 .. s0 + B - 1 (CSR
// slots [kbeg, kend)) and keeps its state at buf * ystride of the Y arrays.
constexpr int kMaxGroup = 32;
struct BlockRef {
  int32_t s0 = 0, kbeg = 0, kend = 0, buf = 0;
};
struct BlockList {
  int32_t nb = 0;
  BlockRef b[kMaxGroup];
};

// Per-edge accumulation job of a group: the slots of every listed block gain the
// step-ell term.  With rdiag set instead, the job records p_ell(s,s) and p_ell(j,s)
// of every slot into rdiag / roff (T[slots][L0 + 1], the learned closure's
// recordings).
struct AccJob {
  BlockList list;                // nb == 0: no job
  int32_t wg0[kMaxGroup] = {};   // prefix of workgroup counts (filled at launch)
  int32_t ell = 0;
  const int32_t* tau = nullptr;
  double* gacc = nullptr;
  void* rdiag = nullptr;
  void* roff = nullptr;
};

// Neighbour-bit update of the two-hop masks: set the bits of the blocks of `set` in
// mask set buf, clear those of `clear` in set 1 - buf.  A set holds `slots` blocks'
// arrays, block i of a group at position i.
struct MaskJob {
  BlockList set, clear;
  int32_t buf = 0;
  int64_t slots = 0, awords = 0;
  unsigned long long* mask = nullptr;   // [2][slots][n]
  unsigned* anymask = nullptr;          // [2][slots][awords]
};

struct DeviceGraph {
  int32_t n = 0;
  int64_t m = 0;                 // input edges (halves 0..2m-1)
  int64_t nslots = 0;            // CSR slots (2 x distinct edges)
  int32_t* rowptr = nullptr;     // [n+1]
  int32_t* col = nullptr;        // [2m] neighbours, ascending per row
  int32_t* deg = nullptr;        // [n]
  int32_t* slot_row = nullptr;   // [2m] row of each slot
  int32_t* slot_half = nullptr;  // [2m] slot -> half id (e, or e + m for (v_e -> u_e))
  int32_t* half_slot = nullptr;  // [2m] half id -> slot
  float* inv_deg_f = nullptr;    // [n]
  double* inv_deg_d = nullptr;   // [n]
  Task* tasks = nullptr;         // [ntasks] wave tasks (B < 64): rows with <= kChunk slots
  int32_t ntasks = 0;
  // sliced lists for B = 64 (built with the first such run): the light rows sorted by
  // degree (descending) in groups of 8; group g's ids in chunks of 8 slots, chunk q at
  // slice_nb[64 (grp[g].x + q)], row r's slot 8 q + k at 8 r + k of it, n where the row
  // has ended; a group is as wide as its longest row, rounded up to 4 (grp[g].y)
  int2* slice_grp = nullptr;     // [nslice_grp]
  int32_t nslice_grp = 0;
  int32_t* slice_row = nullptr;  // [8 * nslice_grp] rows (n: none)
  int32_t* slice_nb = nullptr;
  float* slice_inv_f = nullptr;  // [8 * nslice_grp] 1/degree
  double* slice_inv_d = nullptr;
  Task* wg_tasks = nullptr;      // [nwg] workgroup tasks: heavy rows, giant-row chunks
  int32_t nwg = 0;
  HeavyRow* giant = nullptr;     // [ngiant] rows cut into chunks
  int32_t ngiant = 0;
  int32_t nparts = 0;            // total partial rows
  // col in 16 bits for the walks (built with the first per-source run where n <= 65,536)
  uint16_t* col16 = nullptr;     // [2m]
};

// One graph of a batch as the persistent kernel sees it (device pointers).
// Rows sorted by degree (descending) form groups of 64.  Row i of group gi
// has a record rec[(gi * 64 + i) * RW ...] of RW = 4 + 8 / K words: (row,
// degree, cb, 0) followed by its first kBatchSlots neighbour ids, K = 2 ids
// of 16 bits per word when narrow (n < 65535), else K = 1; its slots from
// kBatchSlots on sit column-major in nb, word w at nb[cb + w * 64].  Rows are
// padded with the zero row n up to their group's largest degree rounded up
// to kBatchSlots; records past the last row read (n, 0, 0, 0, n ...).
struct BatchGraph {
  int32_t n = 0;
  int32_t B = 0;                    // source-block width of this graph's items
  int32_t ngroups = 0;
  int32_t narrow = 0;               // 1: two 16-bit ids per neighbour word
  const int32_t* rowptr = nullptr;
  const int32_t* col = nullptr;
  const int32_t* slot_row = nullptr;
  const int32_t* tau_slot = nullptr;
  const int32_t* tau_row = nullptr;
  const float* inv_f = nullptr;
  const double* inv_d = nullptr;
  const uint32_t* rec = nullptr;
  const uint32_t* nb = nullptr;
  const float* grp_invf = nullptr;  // 1/degree of the records' rows (0 past the last)
  const double* grp_invd = nullptr;
  double* gacc = nullptr;
  // truncation and output of the run (prologue / epilogue kernels)
  const int32_t* deg = nullptr;
  const int32_t* half_slot = nullptr;
  double* out = nullptr;            // device output, m doubles
  int32_t m = 0;
  int32_t L = 0;                    // odd uniform truncation, 0: Theorem 3.2, -1: tau_slot
                                    // and tau_row already hold CalTau's lengths
  int32_t max_L = 0;
  int32_t active = 0;               // 1: graph takes part in the run
  double eps = 0.0;
  double lam = 0.0;
};

constexpr int kBatchSlots = 8;          // neighbour slots per gather batch (group widths padded to it)
constexpr int kBatchWordPad = 8 * 64;   // spare words after the last group

struct BatchItem {
  int32_t graph;
  int32_t s0;
};

// --------------------------------------------------------------- kernels (launch wrappers)
// All wrappers enqueue on `st` and return the hipError_t of the launch.

// gacc[k] = 1/d_s - [tau_k >= 1] * 1/(d_s d_j): the l = 0 and l = 1 terms of
// Eq. 9, whose probabilities are known in closed form (p_0 = e_s,
// p_1(s,s) = 0, p_1(j,s) = 1/d_j).
// include_l1 = 0 leaves the l = 1 term to the walk tail (TGT+ with tilde_tau = 0).
// Also nr[k] = 0 and *capped = 0 (either may be null).
hipError_t launch_gacc_init(const DeviceGraph& g, const int32_t* tau_slot, int include_l1,
                            double* gacc, hipStream_t st, int64_t* nr = nullptr,
                            unsigned long long* capped = nullptr);

// tau per slot: uniform L (odd) when L > 0, else the lambda* bound of
// Theorem 3.2 with Upsilon = Delta = 0.  Also the per-row maximum.
// CalTau (Algorithm 1, Eq. 6-8) for every slot with the omega eigenpairs of
// D^-1/2 A D^-1/2 of largest |lambda| (lam[omega], phi[n][omega] node-major on
// the device, pair 0 the trivial one); tau capped at the odd max_L.
constexpr int kMaxOmega = 256;
// capped (may be null): += half-edges whose automatic tau was cut to max_L.
hipError_t launch_caltau(const DeviceGraph& g, const double* lam, const double* phi, int omega,
                         double eps_tau, int max_L, int32_t* tau_slot, int32_t* tau_row,
                         hipStream_t st, unsigned long long* capped = nullptr);
// Ritz vectors phi[x][1..p] = V[:, 1..steps] Y (Y: steps x p32 row-major, p32 a multiple of
// kRitzCols), phi[x][0] = V[x]
constexpr int kRitzCols = 32;
hipError_t launch_ritz(int64_t n, int64_t ld, const double* V, int steps, const double* Y,
                       int p32, int p, int omega, double* phi, hipStream_t st);
hipError_t launch_tau(const DeviceGraph& g, int L, double eps_tau, double lam, int max_L,
                      int32_t* tau_slot, int32_t* tau_row, hipStream_t st,
                      unsigned long long* capped = nullptr);

// Mask update in a launch of its own.
hipError_t launch_mask_update(const DeviceGraph& g, int B, const MaskJob& mj, hipStream_t st);

// Fills DeviceGraph::slice_nb from the CSR (the other slice arrays are set).
hipError_t launch_fill_slices(const DeviceGraph& g, hipStream_t st);

// Bytes between the row-flag arrays of StepJob::nz.
inline int64_t flag_stride(int64_t n) { return (n + 63) / 64 * 64; }
// Nodes up to which a launch goes by slices, each on its own XCDs, and the two-hop step and
// the step after it test a bitmap in LDS.  Beyond, an L2 holds little of a slice and the
// memory-side cache not all the states of a group: the chip takes one slice (in those two
// steps, one block's whole rows) after the other.  BA, ms per call by slices / in order, k
// edges per node; FP32 TGT L = 5: n = 100,000 k = 3 69 / 69, k = 10 136 / 151; 130,000 117 /
// 112, 237 / 252; 160,000 181 / 165, 376 / 388; 200,000 294 / 252, 612 / 617.  TGT+ (lambda* =
// 0.7): 100,000 172 / 167, 85 / 88; 130,000 284 / 272, 139 / 138; 160,000 429 / 402, 211 / 201;
// 200,000 694 / 615, 308 / 300.  FP64 TGT L = 5: 60,000 51 / 50, 89 / 102; 100,000 138 / 124, 273 /
// 289; 160,000 361 / 298, 751 / 751.
constexpr int64_t kBitmapNodes = 140000;
// State bytes that a buffer descriptor's 32-bit offsets reach.
constexpr uint64_t kBufferBytes = 0xFFFFFC00ull;

// One step of a group of blocks: Yn = P Yp, or with mask the two-hop state
// Yn = P P Y0 of the indicators from the neighbour masks.  acc accumulates the
// states held in Yp and mj updates masks, carried as extra workgroups when B = 64.
template <typename T>
struct StepJob {
  BlockList blocks;
  const T* Yp = nullptr;         // [buf][n * B], ystride elements apart
  T* Yn = nullptr;
  int64_t ystride = 0;
  T* partials = nullptr;         // [buf][nparts * B]
  // B = 64: the two-hop step writes nz[buf][slice][x] = (the 128-byte slice of row x
  // has a nonzero; always 1 for heavy rows), flag_stride(n) bytes per slice; with skip,
  // rows flagged 0 are exact zeros in Yp and are not gathered
  uint8_t* nz = nullptr;
  bool skip = false;
  int64_t bitmap_nodes = kBitmapNodes;
  uint64_t buffer_bytes = kBufferBytes;
  // B = 64: bit i: of block i's new state only the rows of its sources and their
  // neighbours are read (its last step with nothing but the accumulation to follow);
  // the light ones among the other rows are not written
  uint32_t last = 0;
  const unsigned long long* mask = nullptr;   // two-hop: [i][n]
  const unsigned* anymask = nullptr;          // [i][ceil(n/32)]
  AccJob acc;
  MaskJob mj;
  // the row kernel's own start and end (B < 64: those of each block's kernel)
  struct Events {
    hipEvent_t start = nullptr, stop = nullptr;
  };
  Events ev[kMaxGroup];
};
template <typename T>
hipError_t launch_step(const DeviceGraph& g, int B, const StepJob<T>& job, hipStream_t st);

// The accumulation in a launch of its own.
template <typename T>
hipError_t launch_accumulate(const DeviceGraph& g, int B, const AccJob& acc, const T* Y,
                             int64_t ystride, hipStream_t st);

// Work buffers of the tails of a group, one set per block of the list.
struct TailScratch {
  ColStats* cs = nullptr;         // [blocks][64]
  char* col = nullptr;            // [blocks] col_bytes each
  size_t col_bytes = 0;
  int nparts = 0;                 // row chunks of the candidate summary
  int64_t* chunk_off = nullptr;   // [slots + blocks of the graph]; a block's at kbeg + s0 / B
  double* part = nullptr;         // [capacity] chunk sums, shared by the blocks of a launch
  int64_t capacity = 0;
  int64_t* ctl = nullptr;         // [blocks] chunks
};
// Row chunks of the candidate summary of an n-node graph (a power of two; at most
// kColParts) and the bytes of its scratch per block.
constexpr int kColParts = 2048;
int col_parts(int64_t n);
size_t col_scratch_bytes(int nparts);

// The tail kernels take every block of the list in one launch; block i's state is at
// Y + buf * ystride.
// Algorithm 3 summary per column (top-gamma, rho bound, extremes); acc (optional): the
// accumulation of those states, carried by the first launch.
template <typename T>
hipError_t launch_colstats(const DeviceGraph& g, const BlockList& blocks, int B, int gamma,
                           const T* Y, int64_t ystride, const TailScratch& ts, hipStream_t st,
                           const AccJob* acc = nullptr);

// n_r per slot (Eq. 13 with chi of Eq. 17 / Eq. 15); 0 where tau_k <= tilde.
template <typename T>
hipError_t launch_walk_counts(const DeviceGraph& g, const BlockList& blocks, int B, int tilde,
                              int gamma, double coef, int64_t nr_cap, const T* Y, int64_t ystride,
                              const TailScratch& ts, const int32_t* tau_slot, int64_t* nr_slot,
                              hipStream_t st);

// work[stride * i] += walk pairs, work[stride * i + 1] += single-walk steps of block i
hipError_t launch_work_totals(const BlockList& blocks, int tilde, const int32_t* tau_slot,
                              const int64_t* nr_slot, unsigned long long* work, int stride,
                              hipStream_t st);

// Walk tail: gacc[k] += mean_r X_r (Eq. 11) for the blocks' slots (a block whose
// chunk sums end beyond ts.capacity, those of the blocks before it counted, walks one
// slot per wave).
template <typename T>
hipError_t launch_walks(const DeviceGraph& g, const BlockList& blocks, int B, int tilde,
                        uint64_t seed, const T* Y, int64_t ystride, const int32_t* tau_slot,
                        const int64_t* nr_slot, double* gacc, const TailScratch& ts,
                        hipStream_t st);
// the nodes of walk pair r of half-edge (i, j) over len steps: nodes[0, len)
// from i, nodes[len, 2 len) from j (device memory)
hipError_t launch_walk_trace(const DeviceGraph& g, int i, int j, uint32_t r, int len,
                             uint64_t seed, int32_t* nodes, hipStream_t st);

// out[e] = gacc[slot(u_e->v_e)] + gacc[slot(v_e->u_e)] (Algorithm 2 line 12).
hipError_t launch_combine(const DeviceGraph& g, const double* gacc, double* out,
                          hipStream_t st);

// Trace outputs in input order.
hipError_t launch_trace(const DeviceGraph& g, const int32_t* tau_slot, const int64_t* nr_slot,
                        int32_t* tau_out, int64_t* nr_out, hipStream_t st);

// --------------------------------------------------------------- per-source TGT+
// Frontier-sparse traversal with the per-source switch step of Eq. 14, one
// workgroup per source (kernels_sparse.hip).  Columns are 64-bit fixed point
// Q[y] = p_l(i, y) / d_y in units of 2^-63, one pair of n-word columns and one
// pair of n-entry support lists per workgroup slot.

// Graphs of up to this many nodes keep both columns in LDS (64 KB, two workgroups a CU):
// the pushes are LDS atomics then (3,000 nodes, 3,000 sources in two launches: 589 -> 425 us).
constexpr int kSrcLdsColumns = 4096;

// A source between two of its steps (see the heavy kernels): the state at l = ell, and
// what the step being made collects.
struct SrcHeavy {
  int64_t li = 0;                 // list entry
  int32_t row = 0, slot = 0;
  int32_t ell = 0, cnt = 0, parity = 0, done = 0;
  uint64_t pushed = 0, vol = 0, qmx = 0, qmn = 0, qmx_i = 0, qmn_i = 0;
  double rho = 0.0, rhs = 0.0;    // rho-hat and Eq. 14's right side at ell
  int32_t cntn = 0, pad_ = 0;
  unsigned long long vol_n = 0, mx_n = 0, mn_n = ~0ull;
};

struct SrcArgs {
  int32_t n = 0;
  const int32_t* rowptr = nullptr;
  const int32_t* col = nullptr;
  const int32_t* tau_slot = nullptr;
  const int32_t* tau_row = nullptr;
  const int32_t* srcs = nullptr;   // source list (null: node k is entry k)
  const int64_t* hoff = nullptr;   // [nsrc + 1] prefix of the listed sources' degrees (null: rowptr)
  int64_t list_base = 0;           // first list entry of this launch (workgroup w takes entry base + w)
  int64_t nsrc = 0;                // list length
  int64_t pos_base = 0;            // hoff[list_base]: positions are relative to it
  uint64_t* Q = nullptr;           // [2 * slots * n], all zero between sources
  int32_t* S = nullptr;            // [2 * slots * n]
  int32_t* slot_ctl = nullptr;     // [2 * slots]: final support size, which column holds it
  int32_t* tilde_row = nullptr;    // [n] switch step per source
  int64_t* nr_slot = nullptr;      // [2m] walk pairs per CSR slot
  double* gacc = nullptr;          // [2m] per-half sums (l = 0 term already in)
  int32_t* pos_slot = nullptr;     // [positions] CSR slot of each position
  int32_t* pos_w = nullptr;        // [positions] workgroup slot holding its source's column
  int64_t* nr_pos = nullptr;       // [positions] walk pairs
  unsigned long long* totals = nullptr;   // walk pairs, walk steps, pushed entries, min / max tilde
  double coef = 0.0;               // 8 ln(2m / delta) / eps^2 (Eq. 13)
  int64_t nr_cap = 0;
  int gamma = 10;
  int rule = 0;                    // 0: Eq. 14 as printed (walk pairs), 1: walk steps
  int force_tilde = -1;            // >= 0: switch at min(force_tilde, tau_p) instead
  SrcHeavy* heavy = nullptr;       // [sources of the launch] (null: each ends in its head)
  int32_t* heavy_ctl = nullptr;    // [2] sources in heavy, of those not done
  uint64_t heavy_vol = 0;          // a push of more edges is left to the heavy kernels
};

struct SrcWalkArgs {
  int32_t n = 0;
  int64_t P = 0;                   // positions of this wave
  const int32_t* rowptr = nullptr;
  const int32_t* col = nullptr;
  const uint16_t* col16 = nullptr;   // as DeviceGraph's
  const int32_t* slot_row = nullptr;
  const int32_t* tau_slot = nullptr;
  const int32_t* tilde_row = nullptr;
  const uint64_t* Q = nullptr;
  uint64_t* Qw = nullptr;          // same memory, cleared after the walks
  const int32_t* S = nullptr;
  const int32_t* slot_ctl = nullptr;
  const int32_t* pos_slot = nullptr;
  const int32_t* pos_w = nullptr;
  const int64_t* nr_pos = nullptr;
  int64_t* chunk_off = nullptr;    // [P + 1]
  int64_t* ctl = nullptr;          // chunks, whether they fit, units drawn
  int32_t nsources = 0;            // sources of this wave
  double* part = nullptr;          // [capacity]
  int64_t capacity = 0;
  double* gacc = nullptr;
  unsigned k0 = 0, k1 = 0;         // Philox key
  // a batch of chunks [cbeg, cend) set by the host (part holds the batch from
  // index 0); cend < 0: all chunks at once, or one wave per half when they do
  // not fit the buffer (ctl[1] == 0)
  int64_t cbeg = 0, cend = -1;
  // a half with more chunks than this in the batch is summed by a whole
  // workgroup (fixed segments, then the segment sums in order)
  int64_t finish_seg = 256;
  // chunks of a batch, and per source, from which k_src_walks_lds takes it
  int64_t lds_chunks = 65536, lds_source = 96;
};

// dst[k] = src[k] (n <= 65,536)
hipError_t launch_narrow(const int32_t* src, uint16_t* dst, int64_t count, hipStream_t st);
// what a call starts from: totals (entries 3 and 6 are minima), no walks, no slot
// holding a column to clear yet (the heads clear their slot's last one), no tilde
hipError_t launch_src_init(unsigned long long* totals, int ntotals, int64_t* nr_slot, int64_t slots,
                           int32_t* slot_ctl, int64_t nctl, int32_t* tilde_row, int64_t n,
                           hipStream_t st);
hipError_t launch_src_head(const SrcArgs& a, int grid, hipStream_t st);
// `rounds` steps of the first `count` sources in heavy
hipError_t launch_src_heavy(const SrcArgs& a, int count, int rounds, hipStream_t st);
// plain fills (kernels, so that a captured sequence holds no memset nodes)
hipError_t launch_fill_u64(uint64_t* p, int64_t count, uint64_t value, hipStream_t st);
hipError_t launch_fill_u32(uint32_t* p, int64_t count, uint32_t value, hipStream_t st);
// vol[x] = sum of the degrees of x's neighbours (the first push of source x)
hipError_t launch_nbr_volume(const DeviceGraph& g, int64_t* vol, hipStream_t st);
// mm[0] = min(mm[0], min tau_row), mm[1] = max(mm[1], max tau_row)
hipError_t launch_tau_range(int n, const int32_t* tau_row, unsigned long long* mm, hipStream_t st);
// scan, walks and finish of a wave (its columns are cleared by the next head
// that takes the slot, or by launch_src_clear after the last wave)
hipError_t launch_src_walks(const SrcWalkArgs& a, hipStream_t st);
// the same in parts: the chunk scan (ctl[0] = chunks), one batch of walks with
// its finish pass; and the clearing of every used slot's final column
hipError_t launch_src_scan(const SrcWalkArgs& a, hipStream_t st);
hipError_t launch_src_walk_batch(const SrcWalkArgs& a, hipStream_t st);
hipError_t launch_src_clear(const SrcWalkArgs& a, int nslots_used, hipStream_t st);
// dst[x] = src[idx[x]] for x < n (per-node results of a renumbered graph, in the
// caller's ids)
hipError_t launch_gather_i32(const int32_t* src, const int32_t* idx, int32_t* dst, int64_t n,
                             hipStream_t st);

// --------------------------------------------------------------- learned closure
constexpr int kMlpParams = 5313;
constexpr int kFeat = 16;
constexpr int kRecSteps = 8;   // L0

template <typename T>
hipError_t launch_record_init(const DeviceGraph& g, T* rdiag, T* roff, hipStream_t st);
// Recordings of steps ell - 1 and ell of the blocks from their states at ell - 1
// (no dense step for ell); 3 <= ell <= kRecSteps.
template <typename T>
hipError_t launch_record_last(const DeviceGraph& g, const BlockList& blocks, int B, int ell,
                              const T* Y, int64_t ystride, T* rdiag, T* roff, hipStream_t st);
template <typename T>
hipError_t launch_features(const DeviceGraph& g, const T* rdiag, const T* roff, double lam,
                           float* X, double* s0, double* uK, double* lo, double* hi,
                           hipStream_t st);
hipError_t launch_targets(int64_t m, const double* s_ref, const double* s0, const double* uK,
                          float* z, float* w, hipStream_t st);
hipError_t launch_norm_stats(const float* X, int64_t N, float* norm, hipStream_t st);
hipError_t launch_feature_range(const float* X, int64_t N, float* fmin, float* fmax,
                                hipStream_t st);
// Adam's constants for one step: rate, decay rates, epsilon, bias corrections 1 - b^step.
struct AdamStep {
  float lr = 0.f, b1 = 0.f, b2 = 0.f, eps = 0.f, bc1 = 1.f, bc2 = 1.f;
};
// Partial-gradient rows (and partial losses) launch_mlp_train_step writes for nbatch samples.
int mlp_train_blocks(int64_t nbatch);
// Gradient of the weighted squared error over samples idx[0 .. nbatch) into grad (may be
// null) and, with adam, the Adam step on theta, m1, m2.
hipError_t launch_mlp_train_step(float* theta, const float* norm, const float* X, const float* z,
                                 const float* w, const int64_t* idx, int64_t nbatch,
                                 float inv_count, float* grads, float* lossp, float* grad,
                                 float* loss_out, float* m1, float* m2, const AdamStep* adam,
                                 hipStream_t st);
hipError_t launch_mlp_infer(const float* theta, const float* norm, const float* X, int64_t N,
                            int bf16, float* y, hipStream_t st);
hipError_t launch_closure_apply(const DeviceGraph& g, const float* zpred, const double* s0,
                                const double* uK, const double* lo, const double* hi,
                                const float* X, const float* fmin, const float* fmax, double eps,
                                int B, int force, double* out, unsigned char* fb,
                                int* block_flag, unsigned long long* count, hipStream_t st);
hipError_t launch_combine_masked(const DeviceGraph& g, const double* gacc,
                                 const unsigned char* fb, double* out, hipStream_t st);

// --------------------------------------------------------------- Lanczos
constexpr int kLanczosMaxRows = 2048;   // rows of a chunk
constexpr int kLanczosCols = 1024;      // basis columns of an update segment
// Buffers of `runs` Lanczos runs on an n-node graph cut into chunks of `rows` rows.
// Column 0 of a run's basis is the deflated top eigenvector; w[0] holds the unit start
// vector before step 1.  Step j writes column j, alpha[j] and beta[j - 1].
struct LanczosArgs {
  int64_t n = 0;
  int runs = 1, rows = 0, chunks = 0, kcols = 0;   // kcols: basis columns allocated
  const int32_t* rowptr = nullptr;
  const int32_t* col = nullptr;
  const double* sid = nullptr;      // [n] 1/sqrt(degree)
  double* V = nullptr;              // [runs] vstride = kcols * n, column major
  int64_t vstride = 0;
  double* w[2] = {nullptr, nullptr};      // [runs][n]
  double* part[2] = {nullptr, nullptr};   // [runs][chunks][kcols]
  double* norm = nullptr;           // [runs][chunks]
  double* alpha = nullptr;          // [runs][kcols]
  double* beta = nullptr;           // [runs][kcols]
};
int lanczos_rows(int64_t n);
hipError_t launch_lanczos_step(const LanczosArgs& a, int j, hipStream_t st);
// beta[j] after step j when no further step follows
hipError_t launch_lanczos_beta(const LanczosArgs& a, int j, hipStream_t st);

// Persistent batch kernel for items of block width B: workgroups of nt
// threads (256, 512, 1024) take items from *ticket (zero before the launch)
// until it passes nitems.  lds: block states in dyn_lds bytes of dynamic
// LDS, else in slabs of slab_elems elements per workgroup (nt = 256).
template <typename T>
hipError_t launch_batch(int nt, bool lds, int B, int grid, size_t dyn_lds, const BatchGraph* graphs,
                        const BatchItem* items, int nitems, int* ticket, T* slabs,
                        int64_t slab_elems, hipStream_t st);
template <typename T>
const void* batch_kernel_ptr(int nt, bool lds, int B);
hipError_t launch_fill_i32(int32_t* p, int count, int value, hipStream_t st);
// Truncation per slot and row, and the closed-form l = 0, 1 terms, for every
// row of the active graphs (node_off: G + 1 prefix of node counts); with mm,
// mm[0] / mm[1] take the min / max of the rows' truncations; capped (may be
// null) += half-edges whose automatic length was cut to max_L.
hipError_t launch_batch_prologue(const BatchGraph* graphs, const int64_t* node_off, int G,
                                 int64_t total_rows, int32_t* mm, unsigned long long* capped,
                                 hipStream_t st);
// out[e] = g(u_e, v_e) + g(v_e, u_e) for every edge of the active graphs.
hipError_t launch_batch_combine(const BatchGraph* graphs, const int64_t* edge_off, int G,
                                int64_t total_edges, hipStream_t st);

}  // namespace sc
