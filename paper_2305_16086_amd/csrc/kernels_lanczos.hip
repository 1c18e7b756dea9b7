// Lanczos with full re-orthogonalisation (classical Gram-Schmidt, twice) on
// N = D^-1/2 A D^-1/2, one or two independent runs side by side (blockIdx.y).
//
// A step is three launches over the same chunks of rows, one workgroup per chunk:
//   k_lz_apply   beta of the last step from the chunk norms, v_j = w / beta,
//                w = N v_j, and the chunk's part of V^T w;
//   k_lz_orth 0  h = sum of the parts, w -= V h, the chunk's part of V^T w again;
//   k_lz_orth 1  the same, then the chunk's part of |w|^2.
// What a chunk's workgroup needs from the others it sums itself from their parts, in
// chunk order, so nothing comes back to the host between steps (alpha and beta stay
// in device arrays that the host reads every so many steps).  The basis V is column
// major, w of a chunk stays in LDS within a launch, and each launch reads the chunk's
// rows of V once or twice.  n = 10,007, 240 steps of two runs: 100 -> 7 ms (each dot
// product and update was a launch on a few workgroups, with three host round trips a
// step); at n = 100,000 the reads of V are the bound.
#include "sc_internal.hpp"

namespace sc {

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kTile = 256;      // rows of an update tile
constexpr int kCols = 4;        // columns of a dot product in flight per wave
constexpr int kShortRow = 128;  // neighbours summed by 8 lanes

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
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

// part[c] = sum over the chunk's rows of V[:, c] w for c in [0, ncols); column ncols - 1
// is read from last (the chunk's rows) where it is given.
__device__ inline void chunk_dots(const LanczosArgs& a, const double* __restrict__ V, int64_t x0,
                                  int rows, int ncols, const double* s_w, const double* s_last,
                                  double* __restrict__ part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int vcols = s_last ? ncols - 1 : ncols;
  for (int c0 = wave * kCols; c0 < vcols; c0 += kWaves * kCols) {
    double acc[kCols];
#pragma unroll
    for (int q = 0; q < kCols; ++q) acc[q] = 0.0;
    for (int r = lane; r < rows; r += 64) {
      double v[kCols];
#pragma unroll
      for (int q = 0; q < kCols; ++q)
        v[q] = c0 + q < vcols ? V[static_cast<size_t>(c0 + q) * a.n + x0 + r] : 0.0;
      const double wr = s_w[r];
#pragma unroll
      for (int q = 0; q < kCols; ++q) acc[q] += v[q] * wr;
    }
#pragma unroll
    for (int q = 0; q < kCols; ++q) {
      const double t = wave_sum(acc[q]);
      if (lane == 0 && c0 + q < vcols) part[c0 + q] = t;
    }
  }
  if (s_last && wave == kWaves - 1) {
    double acc = 0.0;
    for (int r = lane; r < rows; r += 64) acc += s_last[r] * s_w[r];
    acc = wave_sum(acc);
    if (lane == 0) part[ncols - 1] = acc;
  }
}

__global__ __launch_bounds__(kThreads) void k_lz_apply(LanczosArgs a, int j) {
  __shared__ double s_w[kLanczosMaxRows], s_v[kLanczosMaxRows];
  __shared__ double s_red[kWaves];
  __shared__ int s_long[kLanczosMaxRows];
  __shared__ int s_nlong;
  const int run = static_cast<int>(blockIdx.y), chunk = static_cast<int>(blockIdx.x);
  const int tid = threadIdx.x;
  const int64_t n = a.n;
  const int64_t x0 = static_cast<int64_t>(chunk) * a.rows;
  const int rows = static_cast<int>(min(static_cast<int64_t>(a.rows), n - x0));
  double* __restrict__ V = a.V + run * a.vstride;
  const double* __restrict__ w_in = a.w[(j + 1) & 1] + run * n;
  double* __restrict__ w_out = a.w[j & 1] + run * n;
  double inv = 1.0;
  if (j > 1) {
    double s = 0.0;
    for (int q = tid; q < a.chunks; q += kThreads) s += a.norm[run * a.chunks + q];
    const double beta = sqrt(fmax(block_sum(s, s_red), 0.0));
    inv = 1.0 / beta;
    if (chunk == 0 && tid == 0) a.beta[run * a.kcols + j - 1] = beta;
  }
  for (int r = tid; r < rows; r += kThreads) {
    const double v = w_in[x0 + r] * inv;
    s_v[r] = v;
    V[static_cast<size_t>(j) * n + x0 + r] = v;
  }
  if (tid == 0) s_nlong = 0;
  __syncthreads();
  // w = N v: 8 lanes per short row; the others by a wave each, giant ones by the workgroup
  const int sub = tid & 7;
  for (int r0 = 0; r0 < rows; r0 += kThreads / 8) {
    const int r = r0 + (tid >> 3);
    double acc = 0.0;
    bool mine = false;
    int x = 0;
    if (r < rows) {
      x = static_cast<int>(x0) + r;
      const int b = a.rowptr[x], e = a.rowptr[x + 1];
      mine = e - b <= kShortRow;
      if (mine) {
        for (int k = b + sub; k < e; k += 8) {
          const int u = a.col[k];
          acc += a.sid[u] * w_in[u];
        }
      } else if (sub == 0) {
        s_long[atomicAdd(&s_nlong, 1)] = r;
      }
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) acc += __shfl_xor(acc, off, 64);
    if (mine && sub == 0) s_w[r] = a.sid[x] * (acc * inv);
  }
  __syncthreads();
  const int nlong = s_nlong;
  const int lane = tid & 63;
  bool giant = false;
  for (int q = tid >> 6; q < nlong; q += kWaves) {
    const int r = s_long[q];
    const int x = static_cast<int>(x0) + r;
    const int b = a.rowptr[x], e = a.rowptr[x + 1];
    if (e - b > kGiant) {
      giant = true;
      continue;
    }
    double acc = 0.0;
    for (int k = b + lane; k < e; k += 64) {
      const int u = a.col[k];
      acc += a.sid[u] * w_in[u];
    }
    acc = wave_sum(acc);
    if (lane == 0) s_w[r] = a.sid[x] * (acc * inv);
  }
  if (__syncthreads_or(giant)) {
    for (int q = 0; q < nlong; ++q) {
      const int r = s_long[q];
      const int x = static_cast<int>(x0) + r;
      const int b = a.rowptr[x], e = a.rowptr[x + 1];
      if (e - b <= kGiant) continue;   // uniform
      double acc = 0.0;
      for (int k = b + tid; k < e; k += kThreads) {
        const int u = a.col[k];
        acc += a.sid[u] * w_in[u];
      }
      const double t = block_sum(acc, s_red);
      if (tid == 0) s_w[r] = a.sid[x] * (t * inv);
    }
    __syncthreads();
  }
  for (int r = tid; r < rows; r += kThreads) w_out[x0 + r] = s_w[r];
  chunk_dots(a, V, x0, rows, j + 1, s_w, s_v,
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
    for (int c = tid; c < nc; c += kThreads) {
      double s = 0.0;
#pragma unroll 8
      for (int q = 0; q < a.chunks; ++q) s += part[static_cast<size_t>(q) * a.kcols + cs + c];
      s_h[c] = s;
      if (cs + c == j && chunk == 0) {
        double* al = a.alpha + run * a.kcols + j;
        *al = pass == 0 ? s : *al + s;
      }
    }
    __syncthreads();
    // each wave sums an eighth of the columns; the eight sums in wave order
    const int per = (nc + kWaves - 1) / kWaves;
    const int c0 = wave * per, c1 = min(nc, c0 + per);
    for (int t = 0; t < rows; t += kTile) {
      const int tr = min(kTile, rows - t);
      for (int r = lane; r < tr; r += 64) {
        double acc = 0.0;
        const double* __restrict__ vp = V + static_cast<size_t>(cs) * n + x0 + t + r;
#pragma unroll 8
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
    chunk_dots(a, V, x0, rows, ncols, s_w, nullptr,
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
  // about 128 chunks: enough workgroups to pull the basis at the memory's rate, few
  // enough that summing every chunk's parts stays short
  const int64_t r = (n / 128 + 63) / 64 * 64;
  return static_cast<int>(r < 64 ? 64 : r > kLanczosMaxRows ? kLanczosMaxRows : r);
}

hipError_t launch_lanczos_step(const LanczosArgs& a, int j, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(a.chunks), static_cast<unsigned>(a.runs));
  k_lz_apply<<<grid, kThreads, 0, st>>>(a, j);
  k_lz_orth<<<grid, kThreads, 0, st>>>(a, j, 0);
  k_lz_orth<<<grid, kThreads, 0, st>>>(a, j, 1);
  return hipGetLastError();
}

hipError_t launch_lanczos_beta(const LanczosArgs& a, int j, hipStream_t st) {
  k_lz_beta<<<a.runs, kThreads, 0, st>>>(a, j);
  return hipGetLastError();
}

}  // namespace sc
