// Lanczos with full re-orthogonalisation (classical Gram-Schmidt, twice) on
// N = D^-1/2 A D^-1/2, one or two independent runs side by side (blockIdx.y).
//
// A step is four launches:
//   k_lz_apply   beta of the last step from the chunk norms, v_j = w / beta, w = N v_j;
//   k_lz_dots    per chunk of rows, its part of V^T w;
//   k_lz_orth 0  per chunk: h = sum of the parts, w -= V h, its part of V^T w again;
//   k_lz_orth 1  the same, then its part of |w|^2.
// What a workgroup needs from the others it sums itself from their parts, in chunk
// order, so nothing comes back to the host between steps (alpha and beta stay in device
// arrays that the host reads every so many steps).  The basis V is column major and a
// chunk's w stays in LDS within a launch.  Up to some 30,000 nodes a step is bound by
// its launches' chains of dependent loads, beyond by the four reads of V (n = 10,007, 260
// steps of two runs: 42 us a step, of it 27 in k_lz_orth; 380 with a launch per vector
// operation and a copy to the host for each dot product).  A chunk has at most 2,048
// rows, so above 262,144 nodes their number grows, and with its square the reads of the
// parts in k_lz_orth (from the L2s; a column's parts are 0.73 of its rows' bytes at 3 M
// nodes, 2.4 times them at 10 M).  BA n = 1,000,000: 1.8 s in all, 5.2 before.
#include "sc_internal.hpp"

namespace sc {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kApplyRows = kThreads / 8;   // rows of an SpMV workgroup
constexpr int kTile = 256;      // rows of an update tile
constexpr int kCols = 8;        // columns of a dot product in flight per wave
constexpr int kShortRow = 32;   // neighbours summed by 8 lanes

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Wave sums of eight values, halving the values with the lanes: ten exchanges instead of
// 48.  Lane l returns the sum of value 4 (l / 32) + 2 (l / 16 mod 2) + (l / 8 mod 2).
static_assert(kCols == 8, "wave_sum8");
__device__ inline double wave_sum8(double (&v)[8], int lane) {
  const bool b5 = (lane & 32) != 0, b4 = (lane & 16) != 0, b3 = (lane & 8) != 0;
  double u[4], x[2];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    u[q] = (b5 ? v[q + 4] : v[q]) + __shfl_xor(b5 ? v[q] : v[q + 4], 32, 64);
#pragma unroll
  for (int q = 0; q < 2; ++q)
    x[q] = (b4 ? u[q + 2] : u[q]) + __shfl_xor(b4 ? u[q] : u[q + 2], 16, 64);
  double t = (b3 ? x[1] : x[0]) + __shfl_xor(b3 ? x[0] : x[1], 8, 64);
#pragma unroll
  for (int off = 4; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
  return t;
}

// sum over the workgroup, the same on every thread (s_red: kWaves values)
__device__ inline double block_sum(double v, double* s_red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = s_red[0];
#pragma unroll
  for (int q = 1; q < kWaves; ++q) t += s_red[q];
  return t;
}

// part[c] = sum over the chunk's rows of V[:, c] w for c in [0, ncols)
__device__ inline void chunk_dots(const LanczosArgs& a, const double* __restrict__ V, int64_t x0,
                                  int rows, int ncols, const double* s_w,
                                  double* __restrict__ part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int c0 = wave * kCols; c0 < ncols; c0 += kWaves * kCols) {
    double acc[kCols];
#pragma unroll
    for (int q = 0; q < kCols; ++q) acc[q] = 0.0;
#pragma unroll 1
    for (int r = lane; r < rows; r += 64) {
      double v[kCols];
#pragma unroll
      for (int q = 0; q < kCols; ++q)
        v[q] = c0 + q < ncols ? V[static_cast<size_t>(c0 + q) * a.n + x0 + r] : 0.0;
      const double wr = s_w[r];
#pragma unroll
      for (int q = 0; q < kCols; ++q) acc[q] += v[q] * wr;
    }
    const double t = wave_sum8(acc, lane);
    const int c = c0 + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1);
    if ((lane & 7) == 0 && c < ncols) part[c] = t;
  }
}

// Workgroup b takes rows b, b + G, b + 2 G, ... of the G workgroups, 8 lanes per row:
// neighbouring ids (the hubs of a graph numbered by age or degree) fall to different
// workgroups.  Longer rows follow, a wave each, giant ones by the workgroup.
__global__ __launch_bounds__(kThreads) void k_lz_apply(LanczosArgs a, int j) {
  __shared__ double s_red[kWaves];
  __shared__ int s_long[kApplyRows];
  __shared__ int s_nlong;
  const int run = static_cast<int>(blockIdx.y);
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t n = a.n;
  const int64_t G = gridDim.x;
  const double* __restrict__ w_in = a.w[(j + 1) & 1] + run * n;
  double* __restrict__ w_out = a.w[j & 1] + run * n;
  if (tid == 0) s_nlong = 0;
  double inv = 1.0;
  if (j > 1) {
    double s = 0.0;
    for (int q = tid; q < a.chunks; q += kThreads) s += a.norm[run * a.chunks + q];
    const double beta = sqrt(fmax(block_sum(s, s_red), 0.0));
    inv = 1.0 / beta;
    if (blockIdx.x == 0 && tid == 0) a.beta[run * a.kcols + j - 1] = beta;
  } else {
    __syncthreads();
  }
  if (tid < kApplyRows) {   // v_j over contiguous rows
    const int64_t x = static_cast<int64_t>(blockIdx.x) * kApplyRows + tid;
    if (x < n) a.V[run * a.vstride + static_cast<int64_t>(j) * n + x] = w_in[x] * inv;
  }
  const int sub = tid & 7;
  {
    const int64_t xl = blockIdx.x + (tid >> 3) * G;
    double acc = 0.0;
    bool mine = false;
    int x = 0;
    if (xl < n) {
      x = static_cast<int>(xl);
      const int b = a.rowptr[x], e = a.rowptr[x + 1];
      mine = e - b <= kShortRow;
      if (mine) {
        int u[kShortRow / 8];
#pragma unroll
        for (int q = 0; q < kShortRow / 8; ++q) u[q] = b + sub + 8 * q < e ? a.col[b + sub + 8 * q] : -1;
#pragma unroll
        for (int q = 0; q < kShortRow / 8; ++q)
          if (u[q] >= 0) acc += a.sid[u[q]] * w_in[u[q]];
      } else if (sub == 0) {
        s_long[atomicAdd(&s_nlong, 1)] = x;
      }
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) acc += __shfl_xor(acc, off, 64);
    if (mine && sub == 0) w_out[x] = a.sid[x] * (acc * inv);
  }
  __syncthreads();
  const int nlong = s_nlong;
  bool giant = false;
  for (int q = tid >> 6; q < nlong; q += kWaves) {
    const int x = s_long[q];
    const int b = a.rowptr[x], e = a.rowptr[x + 1];
    if (e - b > kGiant) {
      giant = true;
      continue;
    }
    double acc = 0.0;
#pragma unroll 4
    for (int k = b + lane; k < e; k += 64) {
      const int u = a.col[k];
      acc += a.sid[u] * w_in[u];
    }
    acc = wave_sum(acc);
    if (lane == 0) w_out[x] = a.sid[x] * (acc * inv);
  }
  if (__syncthreads_or(giant)) {
    for (int q = 0; q < nlong; ++q) {
      const int x = s_long[q];
      const int b = a.rowptr[x], e = a.rowptr[x + 1];
      if (e - b <= kGiant) continue;   // uniform
      double acc = 0.0;
      for (int k = b + tid; k < e; k += kThreads) {
        const int u = a.col[k];
        acc += a.sid[u] * w_in[u];
      }
      const double t = block_sum(acc, s_red);
      if (tid == 0) w_out[x] = a.sid[x] * (t * inv);
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_lz_dots(LanczosArgs a, int j) {
  __shared__ double s_w[kLanczosMaxRows];
  const int run = static_cast<int>(blockIdx.y), chunk = static_cast<int>(blockIdx.x);
  const int64_t x0 = static_cast<int64_t>(chunk) * a.rows;
  const int rows = static_cast<int>(min(static_cast<int64_t>(a.rows), a.n - x0));
  const double* __restrict__ w = a.w[j & 1] + run * a.n;
  for (int r = threadIdx.x; r < rows; r += kThreads) s_w[r] = w[x0 + r];
  __syncthreads();
  chunk_dots(a, a.V + run * a.vstride, x0, rows, j + 1, s_w,
             a.part[0] + (static_cast<size_t>(run) * a.chunks + chunk) * a.kcols);
}

__global__ __launch_bounds__(kThreads) void k_lz_orth(LanczosArgs a, int j, int pass) {
  __shared__ double s_w[kLanczosMaxRows];
  __shared__ double s_h[kLanczosCols];
  __shared__ double s_p[kWaves][kTile];
  __shared__ double s_red[kWaves];
  const int run = static_cast<int>(blockIdx.y), chunk = static_cast<int>(blockIdx.x);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t n = a.n;
  const int64_t x0 = static_cast<int64_t>(chunk) * a.rows;
  const int rows = static_cast<int>(min(static_cast<int64_t>(a.rows), n - x0));
  const double* __restrict__ V = a.V + run * a.vstride;
  double* __restrict__ w = a.w[j & 1] + run * n;
  const double* __restrict__ part = a.part[pass] + static_cast<size_t>(run) * a.chunks * a.kcols;
  const int ncols = j + 1;
  for (int cs = 0; cs < ncols; cs += kLanczosCols) {   // one segment of the basis at a time
    const int nc = min(kLanczosCols, ncols - cs);
    // a column's parts over several threads where there are more threads than columns,
    // their sums in order
    double* s_t = &s_p[0][0];
    const int split = min(kThreads / nc, 8);
    const int tc = tid % nc, tp = tid / nc;
    if (tp < split) {
      double s = 0.0;
#pragma unroll 16
      for (int q = tp; q < a.chunks; q += split)
        s += part[static_cast<size_t>(q) * a.kcols + cs + tc];
      s_t[tp * nc + tc] = s;
    }
    __syncthreads();
    if (tid < nc) {
      double s = s_t[tid];
      for (int q = 1; q < split; ++q) s += s_t[q * nc + tid];
      s_h[tid] = s;
      if (cs + tid == j && chunk == 0) {
        double* al = a.alpha + run * a.kcols + j;
        *al = pass == 0 ? s : *al + s;
      }
    }
    __syncthreads();
    // each wave sums its share of the columns; the waves' sums in wave order
    const int per = (nc + kWaves - 1) / kWaves;
    const int c0 = wave * per, c1 = min(nc, c0 + per);
    for (int t = 0; t < rows; t += kTile) {
      const int tr = min(kTile, rows - t);
#pragma unroll 1
      for (int r = lane; r < tr; r += 64) {
        double acc = 0.0;
        const double* __restrict__ vp = V + static_cast<size_t>(cs) * n + x0 + t + r;
#pragma unroll 16
        for (int c = c0; c < c1; ++c) acc += vp[static_cast<size_t>(c) * n] * s_h[c];
        s_p[wave][r] = acc;
      }
      __syncthreads();
      for (int r = tid; r < tr; r += kThreads) {
        double s = s_p[0][r];
#pragma unroll
        for (int q = 1; q < kWaves; ++q) s += s_p[q][r];
        const double x = (cs == 0 ? w[x0 + t + r] : s_w[t + r]) - s;
        s_w[t + r] = x;
        if (cs + nc == ncols) w[x0 + t + r] = x;
      }
      __syncthreads();
    }
  }
  if (pass == 0) {
    chunk_dots(a, V, x0, rows, ncols, s_w,
               a.part[1] + (static_cast<size_t>(run) * a.chunks + chunk) * a.kcols);
  } else {
    double s = 0.0;
    for (int r = tid; r < rows; r += kThreads) s += s_w[r] * s_w[r];
    s = block_sum(s, s_red);
    if (tid == 0) a.norm[run * a.chunks + chunk] = s;
  }
}

// beta_j of the last step enqueued (k_lz_apply of a next step would write it)
__global__ __launch_bounds__(kThreads) void k_lz_beta(LanczosArgs a, int j) {
  __shared__ double s_red[kWaves];
  const int run = static_cast<int>(blockIdx.x);
  double s = 0.0;
  for (int q = threadIdx.x; q < a.chunks; q += kThreads) s += a.norm[run * a.chunks + q];
  const double b2 = block_sum(s, s_red);
  if (threadIdx.x == 0) a.beta[run * a.kcols + j] = sqrt(fmax(b2, 0.0));
}

}  // namespace

int lanczos_rows(int64_t n) {
  // about 128 chunks a run: with two runs a workgroup for every CU, and few enough that
  // summing every chunk's parts stays short (us per k_lz_orth with rows of
  // n / 256, n / 128 and n / 64: n = 10,007 20.9, 13.7, 15.4; 28,000 24.1, 16.9, 25.7;
  // 100,000 144, 130, 192)
  const int64_t r = (n / 128 + 63) / 64 * 64;
  return static_cast<int>(r < 64 ? 64 : r > kLanczosMaxRows ? kLanczosMaxRows : r);
}

hipError_t launch_lanczos_step(const LanczosArgs& a, int j, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(a.chunks), static_cast<unsigned>(a.runs));
  const dim3 rows(static_cast<unsigned>((a.n + kApplyRows - 1) / kApplyRows), grid.y);
  k_lz_apply<<<rows, kThreads, 0, st>>>(a, j);
  k_lz_dots<<<grid, kThreads, 0, st>>>(a, j);
  k_lz_orth<<<grid, kThreads, 0, st>>>(a, j, 0);
  k_lz_orth<<<grid, kThreads, 0, st>>>(a, j, 1);
  return hipGetLastError();
}

hipError_t launch_lanczos_beta(const LanczosArgs& a, int j, hipStream_t st) {
  k_lz_beta<<<a.runs, kThreads, 0, st>>>(a, j);
  return hipGetLastError();
}

}  // namespace sc
