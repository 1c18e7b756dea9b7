// Deterministic traversal kernels (Algorithm 2) for blocks of B sources.
//
// Layout: a block's state Y is node-major, Y[x * B + c] = p_l(x, s0 + c), so
// gathering a neighbour row reads B contiguous values.  Every floating-point
// reduction has a fixed order (no floating-point atomics), so results are
// bit-reproducible: a row with at most kChunk neighbours adds them in slot
// order; a heavier row is one workgroup's task (its four waves take interleaved
// 64-slot pieces and add their sums in wave order through LDS); a row above
// kGiant neighbours is cut into workgroup chunks whose partial sums a fix-up
// pass adds in chunk order.
//
// B = 64 runs a group of blocks per launch (k_step).  B = 16 and 32 run one
// block per launch (k_twohop, k_propagate).
#include "sc_internal.hpp"
#include "accumulate.hpp"
#include <hip/hip_ext.h>
#include "tau.hpp"

#include <algorithm>
#include <cfloat>
#include <climits>

namespace sc {

namespace {

constexpr int kThreads = 64 * kWavesPerBlock;

inline unsigned grid_for(int64_t items, int per_block) {
  return static_cast<unsigned>((items + per_block - 1) / per_block);
}

// ------------------------------------------------------------------ closed-form l = 0, 1 terms
__global__ void k_gacc_init(int64_t nslots, const int32_t* __restrict__ slot_row,
                            const int32_t* __restrict__ col, const double* __restrict__ inv_deg,
                            const int32_t* __restrict__ tau, int include_l1,
                            double* __restrict__ gacc, int64_t* __restrict__ nr,
                            unsigned long long* __restrict__ capped) {
  const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k == 0 && capped) *capped = 0ull;
  if (k >= nslots) return;
  if (nr) nr[k] = 0;
  const int s = slot_row[k];
  const int j = col[k];
  double v = inv_deg[s];                          // l = 0: p_0(s,s)/d_s, p_0(j,s) = 0
  if (include_l1 && tau[k] >= 1)
    v -= inv_deg[j] * inv_deg[s];                 // l = 1: p_1(s,s) = 0, p_1(j,s) = 1/d_j
  gacc[k] = v;
}

// ------------------------------------------------------------------ truncation lengths
// One wave per row: the lanes stride over the row's slots (hub rows too) and a
// butterfly max gives the row's longest truncation.
__global__ __launch_bounds__(kThreads) void k_tau(int n, const int32_t* __restrict__ rowptr,
                                                  const int32_t* __restrict__ col,
                                                  const int32_t* __restrict__ deg, int L,
                                                  double eps_tau, double lam, int max_L,
                                                  int32_t* __restrict__ tau_slot,
                                                  int32_t* __restrict__ tau_row,
                                                  unsigned long long* __restrict__ capped) {
  const int x = blockIdx.x * kWavesPerBlock + static_cast<int>(threadIdx.x) / 64;
  const int lane = static_cast<int>(threadIdx.x) & 63;
  if (x >= n) return;   // uniform per wave
  int tmax = 0;
  int ncap = 0;
  const double di = static_cast<double>(deg[x]);
  const int end = rowptr[x + 1];
  for (int k = rowptr[x] + lane; k < end; k += 64) {
    int t = tau_uncapped(L, di, static_cast<double>(deg[col[k]]), eps_tau, lam);
    if (L <= 0 && t > max_L) {
      t = max_L;
      ++ncap;
    }
    tau_slot[k] = t;
    tmax = t > tmax ? t : tmax;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const int o = __shfl_xor(tmax, off, 64);
    tmax = o > tmax ? o : tmax;
    ncap += __shfl_xor(ncap, off, 64);
  }
  if (lane == 0) {
    tau_row[x] = tmax;
    if (capped && ncap > 0) atomicAdd(capped, static_cast<unsigned long long>(ncap));
  }
}

// ------------------------------------------------------------------ CalTau (Algorithm 1)
// One wave per row x; for every slot (x -> j) the lanes hold the eigenpairs
// k = 2 .. omega-1 (1-based; up to kMaxOmega / 64 per lane) and the sums of
// Eq. 7 and Eq. 8 close with a fixed butterfly, so both halves of an edge get
// the same tau.  lam[omega], phi[n][omega] node-major, pair 1 the trivial one.
__device__ inline double wave_sum_d(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__global__ __launch_bounds__(kThreads) void k_caltau(
    int n, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const int32_t* __restrict__ deg, const double* __restrict__ lam,
    const double* __restrict__ phi, int omega, double eps_tau, int max_L,
    int32_t* __restrict__ tau_slot, int32_t* __restrict__ tau_row,
    unsigned long long* __restrict__ capped) {
  constexpr int P = kMaxOmega / 64;
  const int x = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (x >= n) return;
  bool on[P];
  double lk[P], ax[P];
  const double dx = static_cast<double>(deg[x]);
  const double sx = sqrt(dx);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int k = lane + 64 * p;   // 0-based index; the captured pairs are 1 .. omega-2
    on[p] = k >= 1 && k <= omega - 2;
    lk[p] = on[p] ? lam[k] : 0.0;
    ax[p] = on[p] ? phi[static_cast<size_t>(x) * omega + k] / sx : 0.0;
  }
  const double lw = fabs(lam[omega - 1]);
  const double shrink = 1.0 - lw * lw;
  const double log_inv = log(1.0 / lw);
  int tmax = 0;
  int ncap = 0;   // slots of this row cut to max_L (same on every lane)
  for (int s = rowptr[x]; s < rowptr[x + 1]; ++s) {
    const int j = col[s];
    const double dj = static_cast<double>(deg[j]);
    const double sj = sqrt(dj);
    double coef[P], pw[P], sq[P];
    double ups = 0.0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int k = lane + 64 * p;
      const double a = on[p] ? ax[p] - phi[static_cast<size_t>(j) * omega + k] / sj : 0.0;
      const double w = a * a;
      ups += w * (1.0 + lk[p]);
      coef[p] = on[p] ? w / (1.0 - lk[p]) : 0.0;
      sq[p] = lk[p] * lk[p];
      pw[p] = sq[p];   // lambda_k^(t+1) at t = 1
    }
    ups = wave_sum_d(ups);                                 // Eq. 7
    const double num = 1.0 / dx + 1.0 / dj - 2.0 / (dx * dj) - ups;
    int t = 1;
    while (t <= max_L) {
      double dl = 0.0;
#pragma unroll
      for (int p = 0; p < P; ++p) dl += coef[p] * pw[p];
      const double delta = wave_sum_d(dl);                 // Eq. 8 at t
      bool more;                                           // t <= Eq. 6 (Algorithm 1 line 5)
      if (eps_tau - delta <= 0.0) {
        more = true;                                       // Eq. 6 = +infinity
      } else if (num <= 0.0) {
        more = false;                                      // Eq. 6 = -infinity
      } else {
        const double f = ceil(log(num / ((eps_tau - delta) * shrink)) / log_inv - 1.0);
        more = static_cast<double>(t) <= f;
      }
      if (!more) break;
      t += 2;
#pragma unroll
      for (int p = 0; p < P; ++p) pw[p] *= sq[p];
    }
    const int tau = t > max_L ? max_L : t;
    if (lane == 0) tau_slot[s] = tau;
    ncap += t > max_L ? 1 : 0;
    tmax = tau > tmax ? tau : tmax;
  }
  if (lane == 0) {
    tau_row[x] = tmax;
    if (capped && ncap > 0) atomicAdd(capped, static_cast<unsigned long long>(ncap));
  }
}

// Ritz vectors of the Lanczos basis: phi[x][1 + c] = sum_i V[i + 1][x] Y[i][c]
// for c < p (Y: steps x p32 row-major, zero-padded to a multiple of 32
// columns); column 0 of phi is V's column 0 (the trivial eigenvector).

__global__ __launch_bounds__(256) void k_ritz(int64_t n, int64_t ld, const double* __restrict__ V,
                                              int steps, const double* __restrict__ Y, int p32,
                                              int p, int omega, double* __restrict__ phi) {
  const int64_t x = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (x >= n) return;
  const int c0 = blockIdx.y * kRitzCols;
  double acc[kRitzCols];
#pragma unroll
  for (int c = 0; c < kRitzCols; ++c) acc[c] = 0.0;
  for (int i = 0; i < steps; ++i) {
    const double v = V[static_cast<size_t>(i + 1) * ld + x];
    const double* yr = Y + static_cast<size_t>(i) * p32 + c0;
#pragma unroll
    for (int c = 0; c < kRitzCols; ++c) acc[c] += v * yr[c];
  }
#pragma unroll
  for (int c = 0; c < kRitzCols; ++c)
    if (c0 + c < p) phi[static_cast<size_t>(x) * omega + 1 + c0 + c] = acc[c];
  if (blockIdx.y == 0) phi[static_cast<size_t>(x) * omega] = V[x];
}

// ------------------------------------------------------------------ indicator masks
// Wave w of the set part marks bit c of mask[u] (and the node's bit in the
// filter) for every u in N(s0 + c), c = w mod B, of block w / B of `set` in mask
// set `buf`; the waves after them zero what the blocks of `clear` marked in the
// other set.  A block's words only ever hold that block's bits, so clearing may
// zero whole words.
__device__ inline void mask_update_wave(int w, int lane, int n, int B, const MaskJob& mj,
                                        const int32_t* __restrict__ rowptr,
                                        const int32_t* __restrict__ col) {
  const bool set = w < mj.set.nb * B;
  if (!set) w -= mj.set.nb * B;
  const BlockList& bl = set ? mj.set : mj.clear;
  const int i = w / B, c = w % B;
  if (i >= bl.nb) return;
  const int s = bl.b[i].s0 + c;
  if (s >= n) return;
  const int64_t at = static_cast<int64_t>(set ? mj.buf : 1 - mj.buf) * mj.slots + i;
  unsigned long long* mk = mj.mask + at * n;
  unsigned* am = mj.anymask + at * mj.awords;
  const unsigned long long bit = 1ull << c;
  for (int k = rowptr[s] + lane; k < rowptr[s + 1]; k += 64) {
    const int u = col[k];
    if (set) {
      atomicOr(&mk[u], bit);
      atomicOr(&am[u >> 5], 1u << (u & 31));
    } else {
      mk[u] = 0ull;
      am[u >> 5] = 0u;
    }
  }
}

__global__ void k_mask_update(int n, int B, MaskJob mj, const int32_t* __restrict__ rowptr,
                              const int32_t* __restrict__ col) {
  mask_update_wave(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6), threadIdx.x & 63, n, B, mj,
                   rowptr, col);
}

// ------------------------------------------------------------------ wave helpers
template <typename T, int B>
__device__ inline T reduce_groups(T v) {
  // lanes c, c+B, c+2B, ... hold partial sums of column c; butterfly in a fixed order
#pragma unroll
  for (int off = B; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// wave-uniform broadcast of lane jj's value through a scalar register
__device__ inline float bcast(float v, int jj) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), jj));
}
__device__ inline double bcast(double v, int jj) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(static_cast<int>(b & 0xFFFFFFFFll), jj);
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), jj);
  return __longlong_as_double((static_cast<long long>(hi) << 32) |
                              static_cast<long long>(static_cast<unsigned>(lo)));
}

// Pointers the row kernels need (passed by value).
template <typename T>
struct RowArgs {
  const Task* tasks;          // wave tasks: one light row each (B < 64)
  int ntasks;
  const Task* wg_tasks;       // workgroup tasks (heavy rows, giant-row chunks)
  int nwg;
  const int32_t* col;
  const T* inv_deg;
  T* partials;
};

// Workgroup a of the accumulation of the blocks in `list`: block by the prefix
// of their workgroup counts, one slot per thread.
template <typename T, int B>
__device__ inline void accumulate_group(const AccJob& acc, const int32_t* __restrict__ slot_row,
                                        const int32_t* __restrict__ col,
                                        const double* __restrict__ inv_deg_d, const T* Y,
                                        int64_t ystride, int a) {
  int i = 0;
  while (i + 1 < acc.list.nb && a >= acc.wg0[i + 1]) ++i;   // uniform per workgroup
  const BlockRef br = acc.list.b[i];
  const int k = br.kbeg + (a - acc.wg0[i]) * kThreads + static_cast<int>(threadIdx.x);
  if (k < br.kend)
    accumulate_half<T, B>(acc, br.s0, slot_row, col, inv_deg_d, Y + br.buf * ystride, k);
}

// Sum over the 64-slot pieces first, first + step, ... of [beg, end) of the
// neighbour rows of Yp (column c); lanes c, c+B, ... share a column and are
// combined at the end.  kSkip (B = 64): rows whose flags in nz (one array of nzs
// bytes per slice) are all zero are exact zeros in Yp and are not gathered.
template <typename T, int B, bool kSkip = false>
__device__ inline T gather_pieces(const RowArgs<T>& a, const T* __restrict__ Yp, int beg, int end,
                                  int first, int step, int lane, int c, int gq,
                                  const uint8_t* nz = nullptr, int64_t nzs = 0) {
  constexpr int G = 64 / B;
  constexpr int kBatch = sizeof(T) == 4 ? 32 : 16;   // gathers in flight per lane
  constexpr int kSlices = static_cast<int>(sizeof(T)) / 2;   // of 128 bytes per 64-column row
  static_assert(!kSkip || G == 1, "zero-row skipping needs one column per lane");
  T acc = T(0);
  for (int base = beg + 64 * first; base < end; base += 64 * step) {
    const int cnt = min(64, end - base);
    const int myu = lane < cnt ? a.col[base + lane] : 0;
    if (kSkip) {
      // gather only the slots whose row is nonzero, in slot order: the skipped
      // rows are exact zeros, so the sum is that of the full slot loop
      unsigned any = 0;
      if (lane < cnt) {
#pragma unroll
        for (int q = 0; q < kSlices; ++q) any |= nz[q * nzs + myu];
      }
      unsigned long long rem = __ballot(any != 0);
      while (rem) {
        T v[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
          v[q] = T(0);
          if (rem) {
            const int l = __builtin_ctzll(rem);
            rem &= rem - 1ull;
            const int u = __builtin_amdgcn_readlane(myu, l);
            v[q] = Yp[static_cast<size_t>(u) * B + c];
          }
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) acc += v[q];
      }
    } else if (G == 1) {
      for (int jj = 0; jj < cnt; jj += kBatch) {
        T v[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
          const int l = jj + q;   // wave-uniform
          const int u = __builtin_amdgcn_readlane(myu, l & 63);
          v[q] = l < cnt ? Yp[static_cast<size_t>(u) * B + c] : T(0);
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) acc += v[q];
      }
    } else {
      // uniform trip count: every lane takes part in each shuffle (a shuffle
      // from an inactive lane would read 0), the add is predicated instead
      for (int j0 = 0; j0 < cnt; j0 += G) {
        const int jj = j0 + gq;
        const int u = __shfl(myu, jj, 64);
        if (jj < cnt) acc += Yp[static_cast<size_t>(u) * B + c];
      }
    }
  }
  return reduce_groups<T, B>(acc);
}

// Same traversal for the two-hop step: neighbour u contributes 1/d_u to column
// c when bit c of mask[u] is set (u is a neighbour of source c).
template <typename T, int B>
__device__ inline T twohop_pieces(const RowArgs<T>& a, const unsigned long long* __restrict__ mask,
                                  const unsigned* __restrict__ anymask, int beg, int end,
                                  int first, int step, int lane, int c, int gq) {
  constexpr int G = 64 / B;
  T acc = T(0);
  for (int base = beg + 64 * first; base < end; base += 64 * step) {
    const int cnt = min(64, end - base);
    const int myu = lane < cnt ? a.col[base + lane] : 0;
    // the small bitmap filters out the neighbours no column marks
    const bool hit = lane < cnt && ((anymask[myu >> 5] >> (myu & 31)) & 1u);
    const unsigned long long mym = hit ? mask[myu] : 0ull;
    const T myw = hit ? a.inv_deg[myu] : T(0);
    if (__ballot(hit) == 0ull) continue;
    if (G == 1) {
      const int mlo = static_cast<int>(mym & 0xFFFFFFFFull);
      const int mhi = static_cast<int>(mym >> 32);
      unsigned long long ph = __ballot(hit);   // only marked slots contribute, in slot order
      while (ph) {
        const int jj = __builtin_ctzll(ph);
        ph &= ph - 1ull;
        const unsigned long long mk =
            (static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readlane(mhi, jj))) << 32) |
            static_cast<unsigned>(__builtin_amdgcn_readlane(mlo, jj));
        if ((mk >> c) & 1ull) acc += bcast(myw, jj);
      }
    } else {
      for (int j0 = 0; j0 < cnt; j0 += G) {
        const int jj = j0 + gq;
        const unsigned long long mk = __shfl(mym, jj, 64);
        const T w = __shfl(myw, jj, 64);
        if (jj < cnt && ((mk >> c) & 1ull)) acc += w;
      }
    }
  }
  return reduce_groups<T, B>(acc);
}

// Workgroup task: the four waves' sums are added in wave order; a whole row
// is scaled by 1/d and stored, a giant-row chunk goes to its partial row.
template <typename T, int B>
__device__ inline void wg_finish(const RowArgs<T>& a, const Task& tk, T sum, int wave, int lane,
                                 T* __restrict__ Y) {
  __shared__ T red[kWavesPerBlock][64];
  red[wave][lane] = sum;
  __syncthreads();
  if (wave == 0 && lane < B) {
    T tot = red[0][lane];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w) tot += red[w][lane];
    if (tk.part < 0)
      Y[static_cast<size_t>(tk.row) * B + lane] = tot * a.inv_deg[tk.row];
    else
      a.partials[static_cast<size_t>(tk.part) * B + lane] = tot;
  }
}

// ------------------------------------------------------------------ one step of a group, B = 64
// The light rows of a slice (SliceGrid) are one XCD's work, so each XCD's L2 holds one
// slice of one block at a time instead of parts of whole rows of the same block in all
// eight.
//
// Light rows are read through the sliced lists of DeviceGraph (rows sorted by
// degree in groups of 8): a wave takes a group, 8 lanes x 16 bytes per row, so one
// load instruction fetches the neighbours of 8 rows; the ids of 8 rows x 8 slots
// are one coalesced load, spread within each row's lanes by ds_swizzle.  Padding is
// id n, whose offset lies past the buffer descriptor's end: such loads return zero
// and move nothing, without a branch (a vector instruction takes four cycles here,
// so at 20 slots per row the addressing and the additions cost about as much as the
// gathers).  Sums are in slot order.
//
// The two-hop step and the step after it test one bit per neighbour (is it joined
// to a source of the block; is its slice of the two-hop state nonzero) in a bitmap
// in LDS, filled once per workgroup, so these two launch as many workgroups as are
// resident and stride over the groups.  From memory such a test fetches a line per
// neighbour, as much as gathering the row.
//
// A launch covers every block of a group (up to kMaxGroup): the launch and drain of
// a step and its longest row's chain of dependent loads are paid once per group.
//
// All this is for states of which an L2 holds a good part; larger graphs go by kTwoHopBig
// and kSkipBig (whole_rows), and by kFull one slice after the other (kBitmapNodes).
enum StepMode { kFull, kSkip, kTwoHop, kTwoHopBig, kSkipBig };
constexpr bool is_twohop(int mode) { return mode == kTwoHop || mode == kTwoHopBig; }
constexpr bool is_skip(int mode) { return mode == kSkip || mode == kSkipBig; }

template <typename T>
struct StepArgs {
  int n;
  SliceGrid slices;            // light rows of the blocks' slices
  bool in_order;               // slice after slice over the whole chip instead
  int heavy_wgs;               // workgroups of the heavy tasks (multiple of 8, before the slices)
  int light_wgs;               // workgroups of the slices
  int acc_wgs;                 // workgroups of the accumulation, then the mask update
  const int2* grp;             // [ngrp] (first chunk, padded width)
  int ngrp;
  const int32_t* grow;         // [ngrp * 8] rows (n: none)
  const T* ginv;               // [ngrp * 8] 1/degree
  const int32_t* gnb;          // ids
  const T* Yp;                 // state at l - 1 / at l, block buf at buf * ystride
  T* Yn;
  int64_t ystride;
  uint8_t* nz;                 // [buf][slice][nzs]: row flags of the two-hop state
  int64_t nzs;
  const unsigned long long* mask;   // [i][n], i = position of the block in the group
  const unsigned* anymask;
  int64_t awords;
  const T* inv;                // [n] 1/degree by node
  int part_rows;               // partial-sum rows per block
  RowArgs<T> row;
  BlockList blocks;
  uint32_t last;               // see StepJob
  AccJob acc;                  // accumulation of the states in Yp (list.nb == 0: none)
  const int32_t* slot_row;
  const double* inv_deg_d;
  const int32_t* rowptr;
  MaskJob mj;
};

// lane of row r (8 lanes), step k: the value the row's lane k holds
template <int k>
__device__ inline int row_lane(int v) {
  return __builtin_amdgcn_ds_swizzle(v, 0x18 | (k << 5));
}
template <int k>
__device__ inline float row_lane_f(float v) {
  return __int_as_float(row_lane<k>(__float_as_int(v)));
}
template <int k>
__device__ inline double row_lane_f(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = row_lane<k>(static_cast<int>(b & 0xFFFFFFFFll));
  const int hi = row_lane<k>(static_cast<int>(b >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) |
                              static_cast<long long>(static_cast<unsigned>(lo)));
}

template <typename T>
struct alignas(16) Vec16 {
  T v[16 / sizeof(T)];
};
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// The block state rows are gathered from.  kWide: states of 4 GiB or more, which a
// buffer descriptor's 32-bit offsets do not reach.
template <typename T, bool kWide>
struct RowSource {
  static constexpr int kShift = sizeof(T) == 4 ? 8 : 9;   // log2 of the bytes of a row
  const char* base;
  __amdgpu_buffer_rsrc_t rsrc;
  int n;
  uint32_t coff;   // the lane's byte offset inside a row
  __device__ RowSource(const T* Y, int n_, uint32_t coff_) : n(n_), coff(coff_) {
    base = reinterpret_cast<const char*>(Y);
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0,
                                             static_cast<uint32_t>(n_) << kShift, 0x00020000);
  }
  // 16 bytes of row u, `at` bytes after the lane's own, zeros for u == n
  __device__ Vec16<T> load(int u, uint32_t at = 0) const {
    if constexpr (kWide) {
      if (u < n)
        return *reinterpret_cast<const Vec16<T>*>(base + ((static_cast<size_t>(u) << kShift) + coff + at));
      Vec16<T> z;
#pragma unroll
      for (int e = 0; e < static_cast<int>(16 / sizeof(T)); ++e) z.v[e] = T(0);
      return z;
    } else {
      const u32x4_t w = __builtin_amdgcn_raw_buffer_load_b128(
          rsrc, (static_cast<uint32_t>(u) << kShift) + coff + at, 0, 0);
      return __builtin_bit_cast(Vec16<T>, w);
    }
  }
};

// Steps [0, K) of a chunk: the loads in flight together, then added in slot order.
template <typename T, int K, typename Src>
__device__ inline void load_chunk(const Src& src, int ids, Vec16<T>* v) {
  v[0] = src.load(row_lane<0>(ids));
  v[1] = src.load(row_lane<1>(ids));
  v[2] = src.load(row_lane<2>(ids));
  v[3] = src.load(row_lane<3>(ids));
  if constexpr (K == 8) {
    v[4] = src.load(row_lane<4>(ids));
    v[5] = src.load(row_lane<5>(ids));
    v[6] = src.load(row_lane<6>(ids));
    v[7] = src.load(row_lane<7>(ids));
  }
}

template <typename T, int K>
__device__ inline void add_chunk(const Vec16<T>* v, T (&acc)[16 / sizeof(T)]) {
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int e = 0; e < static_cast<int>(16 / sizeof(T)); ++e) acc[e] += v[k].v[e];
}

// two-hop: neighbour u adds 1/d_u to the columns whose source it is joined to; hits:
// the lanes whose neighbour has any such column
template <typename T, int k>
__device__ inline void twohop_step(unsigned long long hits, unsigned m, T w, int c,
                                   T (&acc)[16 / sizeof(T)]) {
  constexpr int V = 16 / sizeof(T);
  if ((hits & (0x0101010101010101ull << k)) == 0ull) return;   // wave-uniform
  const unsigned mk = static_cast<unsigned>(row_lane<k>(static_cast<int>(m))) >> (c * V);
  const T wk = row_lane_f<k>(w);
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] += ((mk >> e) & 1u) ? wk : T(0);
}

// twohop_step for all slices of a row (m: the neighbour's whole mask)
template <typename T, int k>
__device__ inline void twohop_all(unsigned long long hits, unsigned long long m, T w, int c,
                                  T (&acc)[sizeof(T) / 2][16 / sizeof(T)]) {
  constexpr int V = 16 / sizeof(T), C = 8 * V, kSlices = 64 / C;
  if ((hits & (0x0101010101010101ull << k)) == 0ull) return;   // wave-uniform
  const unsigned lo = static_cast<unsigned>(row_lane<k>(static_cast<int>(m)));
  const unsigned hi = static_cast<unsigned>(row_lane<k>(static_cast<int>(m >> 32)));
  const T wk = row_lane_f<k>(w);
#pragma unroll
  for (int h = 0; h < kSlices; ++h) {
    const unsigned mk = (h * C < 32 ? lo : hi) >> ((h * C & 31) + c * V);
#pragma unroll
    for (int e = 0; e < V; ++e) acc[h][e] += ((mk >> e) & 1u) ? wk : T(0);
  }
}

// The next K of the slots of each row's chunk that `live` (bits of the row's 8 slots)
// names, all slices of their rows: the loads in flight together, behind them what
// `meanwhile` issues, then added in slot order.  Dead slots cost no load: a row has its
// own k-th live slot in step k, zeros where it has none.
template <typename T, int K, typename Src, typename F>
__device__ inline void gather_live(const Src& src, int n, int ids, unsigned& live, int lane,
                                   T (&acc)[sizeof(T) / 2][16 / sizeof(T)], F meanwhile) {
  constexpr int V = 16 / sizeof(T), kSlices = static_cast<int>(sizeof(T)) / 2;
  Vec16<T> v[K][kSlices];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int x = __shfl(ids, (lane & 56) + __builtin_ctz(live | 128u), 64);
    const int u = live ? x : n;
    live &= live - 1u;
#pragma unroll
    for (int h = 0; h < kSlices; ++h) v[k][h] = src.load(u, h * 128);
  }
  meanwhile();
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int h = 0; h < kSlices; ++h)
#pragma unroll
      for (int e = 0; e < V; ++e) acc[h][e] += v[k][h].v[e];
}

// What a wave that strides over the groups of rows has fetched of those to come: the
// list of the group after next; the list, rows, 1/degree and first ids of the next.
template <typename T>
struct GroupAhead {
  int2 g0, g1;
  int row, ids;
  T iv;
  __device__ int2 list(const StepArgs<T>& a, int x) const {
    return x < a.ngrp ? a.grp[x] : make_int2(0, 0);
  }
  __device__ void rest(const StepArgs<T>& a, int x, int lane) {   // of group x, whose list is g0
    row = a.n;
    ids = a.n;
    iv = T(0);
    if (x < a.ngrp) {
      row = a.grow[x * 8 + (lane >> 3)];
      iv = a.ginv[x * 8 + (lane >> 3)];
      if (g0.y > 0) ids = a.gnb[static_cast<int64_t>(g0.x) * 64 + lane];
    }
  }
  __device__ void start(const StepArgs<T>& a, int x, int stride, int lane) {
    g0 = list(a, x);
    g1 = list(a, x + stride);
    rest(a, x, lane);
  }
  __device__ void take(const StepArgs<T>& a, int x, int stride, int lane, int2* g, int* row_x,
                       T* iv_x, int* ids_x) {
    *g = g0;
    *row_x = row;
    *iv_x = iv;
    *ids_x = ids;
    g0 = g1;
    g1 = list(a, x + 2 * stride);
    rest(a, x + stride, lane);
  }
};

// The light rows of slice sl: groups wg * 4 + wave, + 4 wgs, ...
template <typename T, int MODE, bool kWide>
__device__ inline void light_rows(const StepArgs<T>& a, int sl, int wg, int wgs, int lane, int wave,
                                  unsigned* s_bits) {
  constexpr int V = 16 / sizeof(T);        // columns per lane
  constexpr int C = 8 * V;                 // columns per slice
  constexpr int kSlices = 64 / C;          // slices per block
  const int i = sl / kSlices, h = sl % kSlices;
  const int buf = a.blocks.b[i].buf;
  const int n = a.n;
  const int words = (n + 31) / 32;
  if constexpr (MODE == kTwoHop) {
    const unsigned* __restrict__ am = a.anymask + static_cast<size_t>(i) * a.awords;
    for (int q = threadIdx.x; q < words; q += kThreads) s_bits[q] = am[q];
    __syncthreads();
  } else if constexpr (MODE == kSkip) {
    // 32 byte flags (0 or 1) to one word; the flag array is padded to 64 bytes
    const uint4* __restrict__ nz = reinterpret_cast<const uint4*>(
        a.nz + (static_cast<size_t>(buf) * kSlices + h) * a.nzs);
    for (int q = threadIdx.x; q < words; q += kThreads) {
      const uint4 x = nz[2 * q], y = nz[2 * q + 1];
      auto four = [](unsigned w) { return (w * 0x10204080u) >> 28; };
      s_bits[q] = four(x.x) | four(x.y) << 4 | four(x.z) << 8 | four(x.w) << 12 |
                  four(y.x) << 16 | four(y.y) << 20 | four(y.z) << 24 | four(y.w) << 28;
    }
    __syncthreads();
  }
  const int r = lane >> 3, c = lane & 7;
  const uint32_t coff = static_cast<uint32_t>(h * 128 + c * 16);
  [[maybe_unused]] const RowSource<T, kWide> src(a.Yp + buf * a.ystride, n, coff);
  // The two-hop step has little to do for a group of rows but wait for the chain of its
  // list, rows and ids: the list is fetched two groups ahead, the rest one ahead (BA n =
  // 100,000, k = 3, TGT L = 3: 16.2 -> 14.4 ms a call).
  constexpr bool kAhead = MODE == kTwoHop;
  const int stride = wgs * kWavesPerBlock;
  int gi = wg * kWavesPerBlock + wave;
  [[maybe_unused]] GroupAhead<T> ahead;
  if constexpr (kAhead) ahead.start(a, gi, stride, lane);
  for (; gi < a.ngrp; gi += stride) {
    int2 g;
    int row;
    [[maybe_unused]] int first = 0;
    T iv;
    if constexpr (kAhead) {
      ahead.take(a, gi, stride, lane, &g, &row, &iv, &first);
    } else {
      g = a.grp[gi];
      row = a.grow[gi * 8 + r];
      iv = a.ginv[gi * 8 + r];
    }
    const int32_t* __restrict__ p = a.gnb + static_cast<int64_t>(g.x) * 64 + lane;
    T acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = T(0);
    if constexpr (MODE == kTwoHop) {
      const unsigned long long* __restrict__ mask = a.mask + static_cast<size_t>(i) * n;
      const int nch = (g.y + 7) >> 3;
      int next = first;
      for (int ch = 0; ch < nch; ++ch) {
        const int u = next;
        if (ch + 1 < nch) next = p[ch * 64 + 64];
        const bool hit = u < n && ((s_bits[u >> 5] >> (u & 31)) & 1u);
        if (__ballot(hit) == 0ull) continue;
        unsigned m = 0;
        T w = T(0);
        if (hit) {
          m = static_cast<unsigned>(mask[u] >> (h * C)) &
              (C == 32 ? 0xFFFFFFFFu : ((1u << (C & 31)) - 1u));
          w = a.inv[u];
        }
        const unsigned long long hits = __ballot(m != 0);
        twohop_step<T, 0>(hits, m, w, c, acc);
        twohop_step<T, 1>(hits, m, w, c, acc);
        twohop_step<T, 2>(hits, m, w, c, acc);
        twohop_step<T, 3>(hits, m, w, c, acc);
        twohop_step<T, 4>(hits, m, w, c, acc);
        twohop_step<T, 5>(hits, m, w, c, acc);
        twohop_step<T, 6>(hits, m, w, c, acc);
        twohop_step<T, 7>(hits, m, w, c, acc);
      }
    } else {
      auto live = [&](int u) {   // a zero row reads as padding
        if constexpr (MODE == kSkip)
          return u < n && ((s_bits[u >> 5] >> (u & 31)) & 1u) ? u : n;
        else
          return u;
      };
      // two chunks (16 slots of each row) in flight
      const int nf = g.y >> 3;
      const bool half = (g.y & 4) != 0;
      int q = 0;
      for (; q + 1 < nf; q += 2) {
        const int i0 = live(p[q * 64]), i1 = live(p[q * 64 + 64]);
        Vec16<T> v0[8], v1[8];
        load_chunk<T, 8>(src, i0, v0);
        load_chunk<T, 8>(src, i1, v1);
        add_chunk<T, 8>(v0, acc);
        add_chunk<T, 8>(v1, acc);
      }
      if (q < nf && half) {
        const int i0 = live(p[q * 64]), i1 = live(p[q * 64 + 64]);
        Vec16<T> v0[8], v1[4];
        load_chunk<T, 8>(src, i0, v0);
        load_chunk<T, 4>(src, i1, v1);
        add_chunk<T, 8>(v0, acc);
        add_chunk<T, 4>(v1, acc);
      } else if (q < nf) {
        Vec16<T> v0[8];
        load_chunk<T, 8>(src, live(p[q * 64]), v0);
        add_chunk<T, 8>(v0, acc);
      } else if (half) {
        Vec16<T> v0[4];
        load_chunk<T, 4>(src, live(p[q * 64]), v0);
        add_chunk<T, 4>(v0, acc);
      }
    }
    if (MODE == kTwoHop) {
      bool any = false;
#pragma unroll
      for (int e = 0; e < V; ++e) any |= acc[e] != T(0);
      const unsigned long long b = __ballot(any);
      if (c == 0 && row < n)
        a.nz[(static_cast<size_t>(buf) * kSlices + h) * a.nzs + row] =
            (b >> (8 * r)) & 0xFFull ? 1 : 0;
    }
    if (row < n) {
      Vec16<T> o;
#pragma unroll
      for (int e = 0; e < V; ++e) o.v[e] = acc[e] * iv;
      char* Yn = reinterpret_cast<char*>(a.Yn + buf * a.ystride);
      *reinterpret_cast<Vec16<T>*>(Yn + (static_cast<size_t>(row) * (64 * sizeof(T)) + coff)) = o;
    }
  }
}

// The light rows of block i in the two steps that test neighbours, beyond kBitmapNodes:
// all slices of a row at once, so that the tests, which come from memory there (the bitmap
// of the sources' neighbours; the first slice's flags, written here for whole rows), are
// made once per neighbour.  Per block of BA n = 400,000, k = 10: two-hop step 42 us, the
// step after it 92 (95 and 258 by slices and without flags; 49 and 90 with a kernel that
// takes a run of rows a wave, a lane per column).
template <typename T, int MODE>
__device__ inline void whole_rows(const StepArgs<T>& a, int i, int wg, int wgs, int lane, int wave) {
  constexpr int V = 16 / sizeof(T);
  constexpr int C = 8 * V;
  constexpr int kSlices = 64 / C;
  constexpr int kSlots = 16 / kSlices;     // slots of a row in flight (16 loads)
  const int buf = a.blocks.b[i].buf;
  const int n = a.n;
  const int r = lane >> 3, c = lane & 7;
  uint8_t* __restrict__ flags = a.nz + static_cast<size_t>(buf) * kSlices * a.nzs;
  const RowSource<T, false> src(a.Yp + buf * a.ystride, n, static_cast<uint32_t>(c * 16));
  char* __restrict__ Yn = reinterpret_cast<char*>(a.Yn + buf * a.ystride);
  const int stride = wgs * kWavesPerBlock;
  int gi = wg * kWavesPerBlock + wave;
  GroupAhead<T> ahead;
  ahead.start(a, gi, stride, lane);
  // kSkipBig: the flags of a chunk are fetched behind the gathers of the one before
  auto flag_of = [&](int u) { return MODE == kSkipBig ? flags[min(u, n - 1)] : 0; };
  [[maybe_unused]] int live = flag_of(ahead.ids);
  for (; gi < a.ngrp; gi += stride) {
    int2 g;
    int row, next;
    T iv;
    ahead.take(a, gi, stride, lane, &g, &row, &iv, &next);
    const int32_t* __restrict__ p = a.gnb + static_cast<int64_t>(g.x) * 64 + lane;
    T acc[kSlices][V];
#pragma unroll
    for (int h = 0; h < kSlices; ++h)
#pragma unroll
      for (int e = 0; e < V; ++e) acc[h][e] = T(0);
    const int nch = (g.y + 7) >> 3;
    for (int ch = 0; ch < nch; ++ch) {
      const int u = next;
      if (ch + 1 < nch) next = p[ch * 64 + 64];
      if constexpr (MODE == kTwoHopBig) {
        const unsigned* __restrict__ am = a.anymask + static_cast<size_t>(i) * a.awords;
        const bool hit = u < n && ((am[u >> 5] >> (u & 31)) & 1u);
        const unsigned long long hits = __ballot(hit);   // joined to a source of the block
        if (hits == 0ull) continue;
        unsigned long long m = 0;
        T w = T(0);
        if (hit) {
          m = a.mask[static_cast<size_t>(i) * n + u];
          w = a.inv[u];
        }
        twohop_all<T, 0>(hits, m, w, c, acc);
        twohop_all<T, 1>(hits, m, w, c, acc);
        twohop_all<T, 2>(hits, m, w, c, acc);
        twohop_all<T, 3>(hits, m, w, c, acc);
        twohop_all<T, 4>(hits, m, w, c, acc);
        twohop_all<T, 5>(hits, m, w, c, acc);
        twohop_all<T, 6>(hits, m, w, c, acc);
        twohop_all<T, 7>(hits, m, w, c, acc);
      } else {
        // the rows' live slots, four at a time
        unsigned bits = static_cast<unsigned>(__ballot(u < n && live != 0) >> (lane & 56)) & 0xFFu;
        live = flag_of(ch + 1 < nch ? next : ahead.ids);
        while (__ballot(bits != 0u) != 0ull) gather_live<T, 4>(src, n, u, bits, lane, acc, [] {});
      }
    }
    if constexpr (MODE == kTwoHopBig) {
      bool any = false;
#pragma unroll
      for (int h = 0; h < kSlices; ++h)
#pragma unroll
        for (int e = 0; e < V; ++e) any |= acc[h][e] != T(0);
      const unsigned long long b = __ballot(any);
      if (c == 0 && row < n) flags[row] = (b >> (8 * r)) & 0xFFull ? 1 : 0;
    }
    if (row < n) {
#pragma unroll
      for (int h = 0; h < kSlices; ++h) {
        Vec16<T> o;
#pragma unroll
        for (int e = 0; e < V; ++e) o.v[e] = acc[h][e] * iv;
        *reinterpret_cast<Vec16<T>*>(Yn + (static_cast<size_t>(row) * (64 * sizeof(T)) + h * 128 + c * 16)) = o;
      }
    }
  }
}

// The light rows of slice sl that the accumulation of a block's last step reads: one
// per slot (s, j) of the slice's sources, row j, and the sources' own (a row that
// several sources share is added up for each of them, to the same values).  These are
// some 10 x 64 rows of the block instead of all n, so the step costs what its longest
// rows take and the block is spared one of its dense steps (BA n = 34,401, L = 7: 33.3 ->
// 29.2 ms a call).
// Rows come from the CSR lists, 8 to a wave as in light_rows, slots in the same order.
template <typename T, bool kWide>
__device__ inline void last_rows(const StepArgs<T>& a, int sl, int wg, int wgs, int lane, int wave) {
  constexpr int V = 16 / sizeof(T);
  constexpr int C = 8 * V;
  constexpr int kSlices = 64 / C;
  const int i = sl / kSlices, h = sl % kSlices;
  const BlockRef br = a.blocks.b[i];
  const int n = a.n;
  const int c0 = br.s0 + h * C, c1 = min(n, c0 + C);
  if (c0 >= c1) return;
  const int ks = a.rowptr[c0], slots = a.rowptr[c1] - ks;
  const int r = lane >> 3, c = lane & 7;
  const uint32_t coff = static_cast<uint32_t>(h * 128 + c * 16);
  const RowSource<T, kWide> src(a.Yp + br.buf * a.ystride, n, coff);
  char* __restrict__ Yn = reinterpret_cast<char*>(a.Yn + br.buf * a.ystride);
  for (int g = wg * kWavesPerBlock + wave; g * 8 < slots + c1 - c0; g += wgs * kWavesPerBlock) {
    const int x = g * 8 + r;
    int row = x < slots ? a.row.col[ks + x] : c0 + x - slots;
    int beg = 0, d = 0;
    if (row < n) {
      beg = a.rowptr[row];
      d = a.rowptr[row + 1] - beg;
    }
    if (x >= slots + c1 - c0 || d > kChunk) {   // none, or a heavy row's task writes it
      row = n;
      d = 0;
    }
    int width = d;
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) width = max(width, __shfl_xor(width, off, 64));
    width = __builtin_amdgcn_readfirstlane(width);
    T acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = T(0);
    auto ids = [&](int q) { return q + c < d ? a.row.col[beg + q + c] : n; };
    int q = 0;
    for (; q + 8 < width; q += 16) {
      const int i0 = ids(q), i1 = ids(q + 8);
      Vec16<T> v0[8], v1[8];
      load_chunk<T, 8>(src, i0, v0);
      load_chunk<T, 8>(src, i1, v1);
      add_chunk<T, 8>(v0, acc);
      add_chunk<T, 8>(v1, acc);
    }
    if (q < width) {
      Vec16<T> v0[8];
      load_chunk<T, 8>(src, ids(q), v0);
      add_chunk<T, 8>(v0, acc);
    }
    if (row < n) {
      const T iv = a.inv[row];
      Vec16<T> o;
#pragma unroll
      for (int e = 0; e < V; ++e) o.v[e] = acc[e] * iv;
      *reinterpret_cast<Vec16<T>*>(Yn + (static_cast<size_t>(row) * (64 * sizeof(T)) + coff)) = o;
    }
  }
}

// Heavy task of one block: the four waves take interleaved 64-slot pieces, lane =
// column.
template <typename T, int MODE>
__device__ inline void heavy_rows(const StepArgs<T>& a, int i, int t, int lane, int wave) {
  constexpr int kSlices = static_cast<int>(sizeof(T)) / 2;
  const int buf = a.blocks.b[i].buf;
  const Task tk = a.row.wg_tasks[t];
  uint8_t* nz = a.nz + static_cast<size_t>(buf) * kSlices * a.nzs;
  RowArgs<T> ra = a.row;
  ra.partials += static_cast<size_t>(buf) * a.part_rows * 64;
  T sum;
  if constexpr (is_twohop(MODE)) {
    sum = twohop_pieces<T, 64>(ra, a.mask + static_cast<size_t>(i) * a.n,
                               a.anymask + static_cast<size_t>(i) * a.awords, tk.beg, tk.end, wave,
                               kWavesPerBlock, lane, lane, 0);
    if (static_cast<int>(threadIdx.x) < kSlices)   // heavy rows count as nonzero
      nz[static_cast<size_t>(threadIdx.x) * a.nzs + tk.row] = 1;
  } else {
    sum = gather_pieces<T, 64, is_skip(MODE)>(ra, a.Yp + buf * a.ystride, tk.beg, tk.end, wave,
                                              kWavesPerBlock, lane, lane, 0, nz, a.nzs);
  }
  wg_finish<T, 64>(ra, tk, sum, wave, lane, a.Yn + buf * a.ystride);
}

template <typename T, int MODE, bool kWide>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_step(StepArgs<T> a) {
  extern __shared__ unsigned s_bits[];   // one bit per node (kSkip, kTwoHop)
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int w = static_cast<int>(blockIdx.x);
  const int nb = a.blocks.nb;
  if (w < a.heavy_wgs) {
    // a block's heavy tasks on the XCDs that take its slices, where the counts divide
    int i, t;
    if (nb <= 8 && 8 % nb == 0) {
      const int k = 8 / nb;
      i = (w & 7) / k;
      t = (w >> 3) * k + (w & 7) % k;
    } else {
      i = w % nb;
      t = w / nb;
    }
    if (t < a.row.nwg) heavy_rows<T, MODE>(a, i, t, lane, wave);
    return;
  }
  w -= a.heavy_wgs;
  if (w < a.light_wgs) {
    if constexpr (MODE == kTwoHopBig || MODE == kSkipBig) {   // block after block
      const int wgs = a.slices.slice_wgs;
      whole_rows<T, MODE>(a, w / wgs, w % wgs, wgs, lane, wave);
    } else {
      int sl, wg, wgs;
      if (a.in_order) {
        wgs = a.slices.slice_wgs;
        sl = w / wgs;
        wg = w % wgs;
      } else if (!a.slices.decode(w, &sl, &wg, &wgs)) {
        return;
      }
      constexpr int kSlices = static_cast<int>(sizeof(T)) / 2;
      if constexpr (MODE != kTwoHop) {
        if ((a.last >> (sl / kSlices)) & 1u) {
          last_rows<T, kWide>(a, sl, wg, wgs, lane, wave);
          return;
        }
      }
      light_rows<T, MODE, kWide>(a, sl, wg, wgs, lane, wave, s_bits);
    }
    return;
  }
  w -= a.light_wgs;
  if (w < a.acc_wgs) {
    accumulate_group<T, 64>(a.acc, a.slot_row, a.row.col, a.inv_deg_d, a.Yp, a.ystride, w);
    return;
  }
  mask_update_wave((w - a.acc_wgs) * kWavesPerBlock + wave, lane, a.n, 64, a.mj, a.rowptr,
                   a.row.col);
}

// ------------------------------------------------------------------ one step of a block, B < 64
template <typename T, int B>
__global__ __launch_bounds__(kThreads) void k_twohop(RowArgs<T> a,
                                                     const unsigned long long* __restrict__ mask,
                                                     const unsigned* __restrict__ anymask,
                                                     T* __restrict__ Y) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int c = lane % B;
  const int gq = lane / B;
  if (static_cast<int>(blockIdx.x) < a.nwg) {
    const Task tk = a.wg_tasks[blockIdx.x];
    const T sum = twohop_pieces<T, B>(a, mask, anymask, tk.beg, tk.end, wave, kWavesPerBlock, lane, c, gq);
    wg_finish<T, B>(a, tk, sum, wave, lane, Y);
    return;
  }
  const int t = (blockIdx.x - a.nwg) * kWavesPerBlock + wave;
  if (t >= a.ntasks) return;
  const Task tk = a.tasks[t];
  const T sum = twohop_pieces<T, B>(a, mask, anymask, tk.beg, tk.end, 0, 1, lane, c, gq);
  if (gq == 0) Y[static_cast<size_t>(tk.row) * B + c] = sum * a.inv_deg[tk.row];
}

// Workgroups [0, nwg): heavy rows and giant-row chunks; then wave tasks.
template <typename T, int B>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_propagate(RowArgs<T> a, const T* __restrict__ Yp,
                                                        T* __restrict__ Yn) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int c = lane % B;
  const int gq = lane / B;
  if (static_cast<int>(blockIdx.x) < a.nwg) {
    const Task tk = a.wg_tasks[blockIdx.x];
    const T sum = gather_pieces<T, B>(a, Yp, tk.beg, tk.end, wave, kWavesPerBlock, lane, c, gq);
    wg_finish<T, B>(a, tk, sum, wave, lane, Yn);
    return;
  }
  const int t = (blockIdx.x - a.nwg) * kWavesPerBlock + wave;
  if (t >= a.ntasks) return;
  const Task tk = a.tasks[t];
  const T sum = gather_pieces<T, B>(a, Yp, tk.beg, tk.end, 0, 1, lane, c, gq);
  if (gq == 0) Yn[static_cast<size_t>(tk.row) * B + c] = sum * a.inv_deg[tk.row];
}

// Giant rows: Y[row] = inv_deg[row] * (sum of the chunk partials in chunk order),
// for block blockIdx.y of the list.
template <typename T, int B>
__global__ __launch_bounds__(kThreads) void k_fixup(const HeavyRow* __restrict__ giant, int ngiant,
                                                    const T* __restrict__ inv_deg,
                                                    const T* __restrict__ partials, int part_rows,
                                                    T* __restrict__ Y, int64_t ystride,
                                                    BlockList blocks) {
  const int lane = threadIdx.x & 63;
  const int h = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  if (h >= ngiant || lane >= B) return;
  const int buf = blocks.b[blockIdx.y].buf;
  const T* pp = partials + static_cast<size_t>(buf) * part_rows * B;
  const HeavyRow hr = giant[h];
  T acc = T(0);
  for (int p = 0; p < hr.nparts; ++p) acc += pp[static_cast<size_t>(hr.part0 + p) * B + lane];
  Y[buf * ystride + static_cast<size_t>(hr.row) * B + lane] = acc * inv_deg[hr.row];
}

// standalone accumulation (the last step of a group)
template <typename T, int B>
__global__ __launch_bounds__(kThreads) void k_accumulate(AccJob acc, const int32_t* __restrict__ slot_row,
                                                         const int32_t* __restrict__ col,
                                                         const double* __restrict__ inv_deg_d,
                                                         const T* __restrict__ Y, int64_t ystride) {
  accumulate_group<T, B>(acc, slot_row, col, inv_deg_d, Y, ystride, static_cast<int>(blockIdx.x));
}

// ------------------------------------------------------------------ sliced lists (B = 64)
// Word (group g, chunk q, row r, k) of the lists: neighbour 8 q + k of the group's
// row r, or n past its degree.
__global__ __launch_bounds__(256) void k_fill_slices(int n, int ngrp, const int2* __restrict__ grp,
                                                     const int32_t* __restrict__ grow,
                                                     const int32_t* __restrict__ rowptr,
                                                     const int32_t* __restrict__ col,
                                                     int32_t* __restrict__ gnb) {
  const int gi = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (gi >= ngrp) return;
  const int2 g = grp[gi];
  const int row = grow[gi * 8 + (lane >> 3)];
  const int beg = row < n ? rowptr[row] : 0;
  const int end = row < n ? rowptr[row + 1] : 0;
  for (int q = 0; 8 * q < g.y; ++q) {
    const int k = beg + 8 * q + (lane & 7);
    gnb[(static_cast<int64_t>(g.x) + q) * 64 + lane] = k < end ? col[k] : n;
  }
}

// ------------------------------------------------------------------ combine and traces
__global__ void k_combine(int64_t m, const int32_t* __restrict__ half_slot,
                          const double* __restrict__ gacc, double* __restrict__ out) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= m) return;
  out[e] = gacc[half_slot[e]] + gacc[half_slot[e + m]];
}

__global__ void k_trace(int64_t m, const int32_t* __restrict__ half_slot,
                        const int32_t* __restrict__ tau_slot, const int64_t* __restrict__ nr_slot,
                        int32_t* __restrict__ tau_out, int64_t* __restrict__ nr_out) {
  const int64_t h = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (h >= 2 * m) return;
  const int k = half_slot[h];
  if (tau_out && h < m) tau_out[h] = tau_slot[k];
  if (nr_out) nr_out[h] = nr_slot ? nr_slot[k] : 0;
}

}  // namespace

// ====================================================================== wrappers

hipError_t launch_gacc_init(const DeviceGraph& g, const int32_t* tau_slot, int include_l1,
                            double* gacc, hipStream_t st, int64_t* nr,
                            unsigned long long* capped) {
  const int64_t ns = g.nslots;
  k_gacc_init<<<grid_for(ns, 256), 256, 0, st>>>(ns, g.slot_row, g.col, g.inv_deg_d, tau_slot,
                                                  include_l1, gacc, nr, capped);
  return hipGetLastError();
}

hipError_t launch_tau(const DeviceGraph& g, int L, double eps_tau, double lam, int max_L,
                      int32_t* tau_slot, int32_t* tau_row, hipStream_t st,
                      unsigned long long* capped) {
  k_tau<<<grid_for(g.n, kWavesPerBlock), kThreads, 0, st>>>(
      g.n, g.rowptr, g.col, g.deg, L, eps_tau, lam, max_L, tau_slot, tau_row, capped);
  return hipGetLastError();
}

hipError_t launch_caltau(const DeviceGraph& g, const double* lam, const double* phi, int omega,
                         double eps_tau, int max_L, int32_t* tau_slot, int32_t* tau_row,
                         hipStream_t st, unsigned long long* capped) {
  if (omega < 2 || omega > kMaxOmega) return hipErrorInvalidValue;
  k_caltau<<<grid_for(g.n, kWavesPerBlock), kThreads, 0, st>>>(
      g.n, g.rowptr, g.col, g.deg, lam, phi, omega, eps_tau, max_L, tau_slot, tau_row, capped);
  return hipGetLastError();
}

hipError_t launch_ritz(int64_t n, int64_t ld, const double* V, int steps, const double* Y,
                       int p32, int p, int omega, double* phi, hipStream_t st) {
  if (p32 % kRitzCols != 0 || p > p32 || 1 + p > omega) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>((n + 255) / 256), static_cast<unsigned>(p32 / kRitzCols));
  k_ritz<<<grid, 256, 0, st>>>(n, ld, V, steps, Y, p32, p, omega, phi);
  return hipGetLastError();
}

hipError_t launch_mask_update(const DeviceGraph& g, int B, const MaskJob& mj, hipStream_t st) {
  const int waves = (mj.set.nb + mj.clear.nb) * B;
  if (waves == 0) return hipSuccess;
  k_mask_update<<<grid_for(waves, kWavesPerBlock), kThreads, 0, st>>>(g.n, B, mj, g.rowptr, g.col);
  return hipGetLastError();
}

#define SC_DISPATCH_B(B, CALL)                        \
  switch (B) {                                        \
    case 64: { constexpr int kB = 64; CALL; } break;  \
    case 32: { constexpr int kB = 32; CALL; } break;  \
    case 16: { constexpr int kB = 16; CALL; } break;  \
    default: return hipErrorInvalidValue;             \
  }
#define SC_DISPATCH_B_NARROW(B, CALL)                 \
  switch (B) {                                        \
    case 32: { constexpr int kB = 32; CALL; } break;  \
    case 16: { constexpr int kB = 16; CALL; } break;  \
    default: return hipErrorInvalidValue;             \
  }

template <typename T>
const T* inv_deg_of(const DeviceGraph& g);
template <>
const float* inv_deg_of<float>(const DeviceGraph& g) { return g.inv_deg_f; }
template <>
const double* inv_deg_of<double>(const DeviceGraph& g) { return g.inv_deg_d; }

template <typename T>
const T* slice_inv_of(const DeviceGraph& g);
template <>
const float* slice_inv_of<float>(const DeviceGraph& g) { return g.slice_inv_f; }
template <>
const double* slice_inv_of<double>(const DeviceGraph& g) { return g.slice_inv_d; }

template <typename T>
RowArgs<T> row_args(const DeviceGraph& g, T* partials) {
  RowArgs<T> a;
  a.tasks = g.tasks;
  a.ntasks = g.ntasks;
  a.wg_tasks = g.wg_tasks;
  a.nwg = g.nwg;
  a.col = g.col;
  a.inv_deg = inv_deg_of<T>(g);
  a.partials = partials;
  return a;
}

// fills the prefix of workgroup counts of an accumulation; returns their total
int plan_acc(AccJob& acc) {
  int wgs = 0;
  for (int i = 0; i < acc.list.nb; ++i) {
    acc.wg0[i] = wgs;
    wgs += static_cast<int>(grid_for(acc.list.b[i].kend - acc.list.b[i].kbeg, kThreads));
  }
  return wgs;
}

hipError_t launch_fill_slices(const DeviceGraph& g, hipStream_t st) {
  if (g.nslice_grp == 0) return hipSuccess;
  k_fill_slices<<<grid_for(g.nslice_grp, 4), 256, 0, st>>>(g.n, g.nslice_grp, g.slice_grp,
                                                           g.slice_row, g.rowptr, g.col,
                                                           g.slice_nb);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fixup(const DeviceGraph& g, int B, const BlockList& blocks, const T* partials,
                        T* Y, int64_t ystride, hipStream_t st) {
  if (g.ngiant == 0 || blocks.nb == 0) return hipSuccess;
  const dim3 grid(grid_for(g.ngiant, kWavesPerBlock), blocks.nb);
  SC_DISPATCH_B(B, (k_fixup<T, kB><<<grid, kThreads, 0, st>>>(g.giant, g.ngiant, inv_deg_of<T>(g),
                                                              partials, std::max(g.nparts, 1), Y,
                                                              ystride, blocks)));
  return hipGetLastError();
}

template <typename T>
hipError_t launch_step(const DeviceGraph& g, int B, const StepJob<T>& job, hipStream_t st) {
  const bool twohop = job.mask != nullptr;
  const int64_t awords = (static_cast<int64_t>(g.n) + 31) / 32;
  const int nb = job.blocks.nb;
  if (B != 64) {   // one launch per block; accumulation and masks in launches of their own
    for (int i = 0; i < nb; ++i) {
      const int64_t off = job.blocks.b[i].buf * job.ystride;
      const RowArgs<T> a = row_args<T>(
          g, job.partials + static_cast<size_t>(job.blocks.b[i].buf) * std::max(g.nparts, 1) * B);
      const unsigned grid = g.nwg + grid_for(g.ntasks, kWavesPerBlock);
      if (twohop) {
        SC_DISPATCH_B_NARROW(B, (k_twohop<T, kB><<<grid, kThreads, 0, st>>>(
                                    a, job.mask + static_cast<size_t>(i) * g.n,
                                    job.anymask + i * awords, job.Yn + off)));
      } else {
        SC_DISPATCH_B_NARROW(B, (hipExtLaunchKernelGGL(k_propagate<T, kB>, dim3(grid),
                                                       dim3(kThreads), 0, st, job.ev[i].start,
                                                       job.ev[i].stop, 0, a, job.Yp + off,
                                                       job.Yn + off)));
      }
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    hipError_t e = launch_accumulate<T>(g, B, job.acc, job.Yp, job.ystride, st);
    if (e == hipSuccess) e = launch_mask_update(g, B, job.mj, st);
    if (e == hipSuccess) e = launch_fixup<T>(g, B, job.blocks, job.partials, job.Yn, job.ystride, st);
    return e;
  }
  StepArgs<T> a;
  a.n = g.n;
  const int groups_wgs = static_cast<int>(grid_for(g.nslice_grp, kWavesPerBlock));
  a.slices.nslices = nb * static_cast<int>(sizeof(T) / 2);
  a.slices.slice_wgs = a.slices.rem_wgs = groups_wgs;
  size_t lds = 0;
  const bool all_last = job.last != 0 && job.last == static_cast<uint32_t>((1ull << nb) - 1);
  const bool wide = static_cast<uint64_t>(g.n) * 64 * sizeof(T) > job.buffer_bytes;
  const bool big = g.n > job.bitmap_nodes;   // no bitmap in LDS
  // (the registers of last_rows would halve the waves of kSkipBig: not with last blocks)
  const bool skip = job.skip && !all_last && !(big && (wide || job.last));
  a.in_order = big && !all_last;
  if ((twohop || skip) && big) {
    // workgroups that stride over a block's rows, as many as the chip holds
    a.slices.nslices = nb;
    a.slices.slice_wgs = std::min(groups_wgs, 256 * 8);
  } else if (twohop || skip) {
    // the same, with the bitmap: as many as are resident on the slice's XCDs (32 CUs
    // each, 160 KB of LDS, and 8 or 5 workgroups by registers)
    lds = static_cast<size_t>(awords) * 4;
    const int per_cu = static_cast<int>(
        std::max<size_t>(1, std::min<size_t>(twohop ? 8 : 5, (size_t(160) << 10) / (lds + 2048))));
    const int rem = a.slices.nslices & 7;
    a.slices.slice_wgs = std::min(groups_wgs, 32 * per_cu);
    a.slices.rem_wgs = std::min(groups_wgs, 32 * per_cu * SliceGrid::rem_xcds(rem));
  }
  if (all_last) {   // 8 rows per wave of at most a block's slots and sources
    int rows = 0;
    for (int i = 0; i < nb; ++i)
      rows = std::max(rows, job.blocks.b[i].kend - job.blocks.b[i].kbeg + B);
    const int wgs = std::min<int>(groups_wgs, (rows + 8 * kWavesPerBlock - 1) / (8 * kWavesPerBlock));
    a.slices.slice_wgs = a.slices.rem_wgs = wgs;
  }
  a.heavy_wgs = (nb * g.nwg + 7) / 8 * 8;
  a.light_wgs = a.in_order ? a.slices.nslices * a.slices.slice_wgs : a.slices.size();
  a.grp = g.slice_grp;
  a.ngrp = g.nslice_grp;
  a.grow = g.slice_row;
  a.ginv = slice_inv_of<T>(g);
  a.gnb = g.slice_nb;
  a.Yp = job.Yp;
  a.Yn = job.Yn;
  a.ystride = job.ystride;
  a.nz = job.nz;
  a.nzs = flag_stride(g.n);
  a.mask = job.mask;
  a.anymask = job.anymask;
  a.awords = awords;
  a.inv = inv_deg_of<T>(g);
  a.part_rows = std::max(g.nparts, 1);
  a.row = row_args<T>(g, job.partials);
  a.blocks = job.blocks;
  a.last = job.last;
  a.acc = job.acc;
  a.acc_wgs = plan_acc(a.acc);
  a.slot_row = g.slot_row;
  a.inv_deg_d = g.inv_deg_d;
  a.rowptr = g.rowptr;
  a.mj = job.mj;
  const int mask_wgs =
      static_cast<int>(grid_for((job.mj.set.nb + job.mj.clear.nb) * B, kWavesPerBlock));
  const int64_t grid = static_cast<int64_t>(a.heavy_wgs) + a.light_wgs + a.acc_wgs + mask_wgs;
  if (grid <= 0 || grid > INT_MAX) return hipErrorInvalidValue;
  const dim3 gd(static_cast<unsigned>(grid)), bd(kThreads);
  if (twohop && big) {
    k_step<T, kTwoHopBig, false><<<gd, bd, 0, st>>>(a);
  } else if (twohop) {
    k_step<T, kTwoHop, false><<<gd, bd, lds, st>>>(a);
  } else if (skip && big) {
    k_step<T, kSkipBig, false><<<gd, bd, 0, st>>>(a);
  } else if (skip) {
    k_step<T, kSkip, false><<<gd, bd, lds, st>>>(a);
  } else if (!wide) {
    hipExtLaunchKernelGGL((k_step<T, kFull, false>), gd, bd, 0, st, job.ev[0].start,
                          job.ev[0].stop, 0, a);
  } else {
    hipExtLaunchKernelGGL((k_step<T, kFull, true>), gd, bd, 0, st, job.ev[0].start,
                          job.ev[0].stop, 0, a);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_fixup<T>(g, B, job.blocks, job.partials, job.Yn, job.ystride, st);
}

template <typename T>
hipError_t launch_accumulate(const DeviceGraph& g, int B, const AccJob& acc, const T* Y,
                             int64_t ystride, hipStream_t st) {
  AccJob job = acc;
  const int wgs = plan_acc(job);
  if (wgs == 0) return hipSuccess;
  SC_DISPATCH_B(B, (k_accumulate<T, kB><<<wgs, kThreads, 0, st>>>(job, g.slot_row, g.col,
                                                                  g.inv_deg_d, Y, ystride)));
  return hipGetLastError();
}

hipError_t launch_combine(const DeviceGraph& g, const double* gacc, double* out,
                          hipStream_t st) {
  k_combine<<<grid_for(g.m, 256), 256, 0, st>>>(g.m, g.half_slot, gacc, out);
  return hipGetLastError();
}

hipError_t launch_trace(const DeviceGraph& g, const int32_t* tau_slot, const int64_t* nr_slot,
                        int32_t* tau_out, int64_t* nr_out, hipStream_t st) {
  if (!tau_out && !nr_out) return hipSuccess;
  k_trace<<<grid_for(2 * g.m, 256), 256, 0, st>>>(g.m, g.half_slot, tau_slot, nr_slot, tau_out,
                                                   nr_out);
  return hipGetLastError();
}

template hipError_t launch_step<float>(const DeviceGraph&, int, const StepJob<float>&, hipStream_t);
template hipError_t launch_step<double>(const DeviceGraph&, int, const StepJob<double>&, hipStream_t);
template hipError_t launch_accumulate<float>(const DeviceGraph&, int, const AccJob&, const float*,
                                             int64_t, hipStream_t);
template hipError_t launch_accumulate<double>(const DeviceGraph&, int, const AccJob&,
                                              const double*, int64_t, hipStream_t);

}  // namespace sc
