// Small kernels of the SCF hot path that do not depend on (nmax, lmax): the
// double-precision cross-block reductions of the coefficient sums, the force
// weights, the standalone kick-drift, fills, the batched-mode reductions and
// the adjoint's reduction of its host sums; and the engine lookup.
#include <hip/hip_runtime.h>

#include "scf_internal.h"

namespace scf {

// ---------------------------------------------------------------------------
// small kernels
// ---------------------------------------------------------------------------
// partial sums over blocks: red1[chunk][t] = sum_{b in chunk} partials[b][t] (double)
template <typename R>
__global__ void __launch_bounds__(256) reduce_kernel(const R* __restrict__ partials, int nblocks,
                                                     int T, int per_chunk, double* red1) {
  __shared__ double sh[4][64];
  const int ti = threadIdx.x & 63, kc = threadIdx.x >> 6;
  const int t = blockIdx.x * 64 + ti;
  const int b0 = blockIdx.y * per_chunk;
  int b1 = b0 + per_chunk;
  if (b1 > nblocks) b1 = nblocks;
  double s = 0.0;
  if (t < T) {
#pragma unroll 8
    for (int b = b0 + kc; b < b1; b += 4) s += double(partials[(int64_t)b * T + t]);
  }
  sh[kc][ti] = s;
  __syncthreads();
  if (kc == 0 && t < T)
    red1[(int64_t)blockIdx.y * T + t] = ((sh[0][ti] + sh[1][ti]) + sh[2][ti]) + sh[3][ti];
}

// Field weights of row (l, j) from its force weights: lane k of a wave holds
// W_k (zero for k > nmaxc) and forms the k-th weights, k < nmaxc + 2.  The
// radial weights come from the rounded force weights, in double precision.
// r0, r1: the lane's two factors (WeightTables.rtab).
template <typename R>
__device__ __forceinline__ void emit_row(const R wk, const double r0, const double r1,
                                         const int lj, const int k, const WeightTables& wt, R* FW) {
  const int nc = wt.nmaxc;
  if (k <= nc) FW[lj * (nc + 1) + k] = wk;
  if constexpr (sizeof(R) == 4) {
    if (!wt.image) return;
    const int l = (int)sqrtf((float)lj + 0.5f), j = lj - l * l, m = (j + 1) >> 1;
    double v;
    if (l == 0) {
      const double u = k <= nc ? (double)wk * r0 : 0.0;
      v = 0.0;
      for (int n = 1; n <= nc; ++n) {
        const double un = __shfl(u, n, 64);
        if (n > k && ((n - k) & 1)) v += un;
      }
      v *= r1;
    } else {
      const R wm = __shfl_up(wk, 1, 64), wp = __shfl_down(wk, 1, 64);
      v = -0.5 * (double)wk;
      if (k > 0) v += r0 * (double)wm;
      if (k < nc) v += r1 * (double)wp;
    }
    if (k < nc + 2) {
      // cosine part in lanes 0, 1 of the quadruple, sine part (even j > 0) in 2, 3
      const int q = m * (nc + 2) + k;
      R* d = FW + FwLayout::img0(nc, wt.lmax) + 64 * (FwLayout::off(l, nc) + (q >> 4)) +
             4 * (q & 15) + ((j > 0 && (j & 1) == 0) ? 2 : 0);
      d[0] = wk;
      d[1] = R(v);
    }
  }
}
// lane k's factors of row (l, j)
__device__ __forceinline__ void row_factors(const WeightTables& wt, const int lj, const int k,
                                            double& r0, double& r1) {
  const int l = (int)sqrtf((float)lj + 0.5f), NP = wt.nmaxc + 2;
  r0 = r1 = 0.0;
  if (wt.image && k < NP) {
    r0 = wt.rtab[(2 * l) * NP + k];
    r1 = wt.rtab[(2 * l + 1) * NP + k];
  }
}

// s + the next K rows of a column in order, every load issued before the first
// add.  In the batched step a thread has a few rows and the latency of its loads
// bounds the reduction: in a loop unrolled by eight the rows past a multiple of
// eight each take a latency of their own.  48 clusters of 1.5e5 particles, nmax
// 6, lmax 4, ten steps: 232 us against 238.  The single-cluster reduction, whose
// threads have 12 to 64 rows, keeps the loop (10 steps at 1e5 points 205.2 us,
// 206.4 with these batches, 207.2 with batches of up to 16).
template <int K, typename IN>
__device__ __forceinline__ double add_rows(const IN* __restrict__& p, const int64_t step,
                                           double s) {
  IN v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = p[k * step];
#pragma unroll
  for (int k = 0; k < K; ++k) s += double(v[k]);
  p += K * step;
  return s;
}

// Reduction and finalisation of the partial rows [r0, r1) for one row (l, j):
// a block of NT threads takes the row's NC = nmax + 1 <= CW coefficients
// (which lie next to each other in a partial row); thread (g, n) sums partial
// rows r0 + g, r0 + g + G, .. (G = NT / CW row groups) in double precision.
// The row groups of a wave are added by lane exchanges, those of the waves
// through LDS by wave 0 (a fixed order), which then holds the row in its lanes:
// a_t = cs_t * sum and the weights follow without another barrier.  One block
// per (l, j) rather than per 16 consecutive coefficients, so that it has the
// neighbours n - 1, n + 1 that the radial weights need.
// FEW: the batched step's few rows per thread (add_rows).  coef, W and FW are
// nullable.
template <int NT, int CW, bool FEW, typename IN, typename R>
__device__ __forceinline__ void reduce_final_row(const IN* __restrict__ partials, int r0, int r1,
                                                 const WeightTables& wt, double* coef, R* W,
                                                 R* FW, int lj) {
  constexpr int G = NT / CW, GW = 64 / CW;  // row groups of the block, of a wave
  __shared__ double sh[NT / 64][CW];
  const int L2 = (wt.lmax + 1) * (wt.lmax + 1), NC = wt.nmax + 1, T = NC * L2;
  const int tid = threadIdx.x, lane = tid & 63, g = tid / CW, c = tid % CW;
  // wave 0's factors, loaded before the sums
  double f0 = 0.0, f1 = 0.0, cs = 0.0, fw = 0.0;
  if (tid < 64) {
    row_factors(wt, lj, lane, f0, f1);
    if (c < NC) {
      cs = wt.cs[c * L2 + lj];
      fw = wt.fw[c * L2 + lj];
    }
  }
  double s = 0.0;
  if (c < NC) {
    if constexpr (FEW) {
      const int64_t step = (int64_t)G * T;
      const IN* __restrict__ p = partials + (int64_t)(r0 + g) * T + lj * NC + c;
      int left = (r1 - r0 - g + G - 1) / G;  // rows of this thread
      for (; left >= 8; left -= 8) s = add_rows<8>(p, step, s);
      if (left & 4) s = add_rows<4>(p, step, s);
      if (left & 2) s = add_rows<2>(p, step, s);
      if (left & 1) s = add_rows<1>(p, step, s);
    } else {
      const IN* __restrict__ col = partials + lj * NC + c;
#pragma unroll 8
      for (int b = r0 + g; b < r1; b += G) s += double(col[(int64_t)b * T]);
    }
  }
#pragma unroll
  for (int o = 32; o >= CW; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane < CW) sh[tid >> 6][lane] = s;
  __syncthreads();
  if (tid >= 64) return;
  s = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; w += GW) s += sh[w + lane / CW][c];
#pragma unroll
  for (int o = 32; o >= CW; o >>= 1) s += __shfl_xor(s, o, 64);
  R wk = R(0);
  if (lane < NC) {
    const double cv = cs * s;
    if (coef) coef[lane * L2 + lj] = cv;
    wk = R(fw * cv);
  }
  if (W && lane <= wt.nmaxc) W[lj * (wt.nmaxc + 1) + lane] = wk;
  if (FW) emit_row<R>(wk, f0, f1, lj, lane, wt, FW);
}

// Row (l, j) of a block: blocks are dealt to the 8 XCDs in turn (block b runs
// on XCD b mod 8), so row (b mod 8) per + b / 8 gives each XCD a contiguous
// range of rows, and the pieces of a 128-byte line of the partial rows are read
// through one L2 (the grid is a multiple of 8 blocks).
__device__ __forceinline__ int xcd_row() {
  const int per = gridDim.x >> 3;
  return (blockIdx.x & 7) * per + (blockIdx.x >> 3);
}
constexpr int grid_rows(int L2) { return (L2 + 7) / 8 * 8; }

template <int NT, typename IN, typename R>
__global__ void __launch_bounds__(NT) reduce_final_kernel(const IN* __restrict__ partials,
                                                            int nrows, WeightTables wt,
                                                            double* coef, R* W, R* FW) {
  const int lj = xcd_row();
  if (lj >= (wt.lmax + 1) * (wt.lmax + 1)) return;
  if (wt.nmax < 16)
    reduce_final_row<NT, 16, false, IN, R>(partials, 0, nrows, wt, coef, W, FW, lj);
  else
    reduce_final_row<NT, 32, false, IN, R>(partials, 0, nrows, wt, coef, W, FW, lj);
}

// one block (a wave) per row (l, j)
template <typename R>
__global__ void __launch_bounds__(64) make_w_kernel(const double* __restrict__ coef,
                                                    WeightTables wt,
                                                    const double* __restrict__ kd, R* FW) {
  const int lj = blockIdx.x, n = threadIdx.x, L2 = (wt.lmax + 1) * (wt.lmax + 1);
  double f0, f1;
  row_factors(wt, lj, n, f0, f1);
  R v = R(0);
  if (n <= wt.nmax) {
    const int t = n * L2 + lj;
    v = R(wt.fw[t] * coef[t]);
    if (kd) {
      const int l = (int)sqrtf((float)lj + 0.5f);
      v = R((double)v * kd[l * (wt.nmaxc + 1) + n]);
    }
  }
  emit_row<R>(v, f0, f1, lj, n, wt, FW);
}

template <typename R>
__global__ void __launch_bounds__(64) expand_w_kernel(const R* __restrict__ W, WeightTables wt,
                                                      R* FW, int64_t W_stride) {
  const int lj = blockIdx.x, n = threadIdx.x, NW = wt.nmaxc + 1;
  const int64_t k = blockIdx.y;
  double f0, f1;
  row_factors(wt, lj, n, f0, f1);
  const R v = n < NW ? W[(k * gridDim.x + lj) * NW + n] : R(0);
  emit_row<R>(v, f0, f1, lj, n, wt, FW + k * W_stride);
}

template <typename R>
__global__ void __launch_bounds__(256) kick_drift_kernel(int64_t n, R* x, R* y, R* z, R* vx, R* vy,
                                                         R* vz, const R* ax, const R* ay,
                                                         const R* az, R kick, R drift) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  R u = fma(kick, ax[i], vx[i]), v = fma(kick, ay[i], vy[i]), w = fma(kick, az[i], vz[i]);
  vx[i] = u;
  vy[i] = v;
  vz[i] = w;
  x[i] = fma(drift, u, x[i]);
  y[i] = fma(drift, v, y[i]);
  z[i] = fma(drift, w, z[i]);
}

// Batched reduction: cluster c owns partial rows [rows[c], rows[c+1]);
// red1[c][chunk][t] sums its rows of one chunk (double).
template <typename R>
__global__ void __launch_bounds__(256) reduce_batched_kernel(const R* __restrict__ partials,
                                                             const int32_t* __restrict__ rows,
                                                             int T, int nchunks, double* red1) {
  __shared__ double sh[4][64];
  const int ti = threadIdx.x & 63, kc = threadIdx.x >> 6;
  const int t = blockIdx.x * 64 + ti;
  const int c = blockIdx.z;
  const int r0 = rows[c], r1 = rows[c + 1];
  const int per_chunk = (r1 - r0 + nchunks - 1) / nchunks;
  const int b0 = r0 + blockIdx.y * per_chunk;
  int b1 = b0 + per_chunk;
  if (b1 > r1) b1 = r1;
  double s = 0.0;
  if (t < T)
    for (int b = b0 + kc; b < b1; b += 4) s += double(partials[(int64_t)b * T + t]);
  sh[kc][ti] = s;
  __syncthreads();
  if (kc == 0 && t < T)
    red1[((int64_t)c * nchunks + blockIdx.y) * T + t] =
        ((sh[0][ti] + sh[1][ti]) + sh[2][ti]) + sh[3][ti];
}

// Batched reduction and finalisation: block (lj, c) reduces cluster c's rows
// (rows[c] .. rows[c+1], or its nchunks chunk sums) as reduce_final_row does;
// block (0, 0) also copies row *step of the centre table into cur (the rows
// the field pass of this step reads) and then advances *step.
template <int NT, typename IN, typename R>
__global__ void __launch_bounds__(NT) reduce_final_batched_kernel(
    const IN* __restrict__ partials, const int32_t* __restrict__ rows, int nchunks,
    WeightTables wt, double* coef, R* FW, int64_t W_stride, const double* __restrict__ centre_tab,
    int ncl, double* cur, int* step) {
  const int c = blockIdx.y;
  if (blockIdx.x == 0 && c == 0 && step) {
    const int k = *step;
    for (int i = threadIdx.x; i < ncl * 9; i += blockDim.x)
      cur[i] = centre_tab[(int64_t)k * ncl * 9 + i];
    __syncthreads();
    if (threadIdx.x == 0) *step = k + 1;
  }
  const int lj = xcd_row(), L2 = (wt.lmax + 1) * (wt.lmax + 1);
  if (lj >= L2) return;
  const int r0 = nchunks ? c * nchunks : rows[c], r1 = nchunks ? r0 + nchunks : rows[c + 1];
  double* cf = coef ? coef + (int64_t)c * (wt.nmax + 1) * L2 : nullptr;
  R* fwc = FW + (int64_t)c * W_stride;
  if (wt.nmax < 16)
    reduce_final_row<NT, 16, true, IN, R>(partials, r0, r1, wt, cf, (R*)nullptr, fwc, lj);
  else
    reduce_final_row<NT, 32, true, IN, R>(partials, r0, r1, wt, cf, (R*)nullptr, fwc, lj);
}

__global__ void set_int_kernel(int* p, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

__global__ void fill_kernel(double* p, int64_t n, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_reduce(int dtype, const void* partials, int nblocks, int T, int nchunks,
                         double* red1, hipStream_t s) {
  if (nblocks <= 0 || T <= 0) return hipSuccess;
  const int per_chunk = (nblocks + nchunks - 1) / nchunks;
  dim3 grid((T + 63) / 64, nchunks);
  if (dtype == 0)
    reduce_kernel<float><<<grid, 256, 0, s>>>((const float*)partials, nblocks, T, per_chunk, red1);
  else
    reduce_kernel<double><<<grid, 256, 0, s>>>((const double*)partials, nblocks, T, per_chunk, red1);
  return hipGetLastError();
}

// Threads per block, input and real type of a reduction.  256 threads (16 row
// groups) up to 32 partial rows, where the rest of 1024 would have no row to
// add, and up to 128 rows when there are blocks enough to fill the chip several
// times (many clusters); with 90 rows and 25 blocks the larger block is already
// the faster one (coefficients and reduction of 1e4 points, nmax 6, lmax 4: 8.6
// against 9.6 us).
template <typename F>
static void with_reduce_types(int dtype, bool chunks_f64, int rows, int blocks, F f) {
  using T4 = std::integral_constant<int, 256>;
  using T16 = std::integral_constant<int, 1024>;
  const bool few = rows <= (blocks >= 1024 ? 128 : 32);
  if (dtype == 0 && !chunks_f64)
    few ? f(T4{}, float(0), float(0)) : f(T16{}, float(0), float(0));
  else if (dtype == 0)
    few ? f(T4{}, double(0), float(0)) : f(T16{}, double(0), float(0));
  else
    few ? f(T4{}, double(0), double(0)) : f(T16{}, double(0), double(0));
}

hipError_t launch_reduce_final(int dtype, bool chunks_f64, const void* partials, int nrows,
                               const WeightTables& wt, double* coef, void* W, void* FW,
                               hipStream_t s) {
  const int grid = grid_rows((wt.lmax + 1) * (wt.lmax + 1));
  with_reduce_types(dtype, chunks_f64, nrows, grid, [&](auto nt, auto in, auto r) {
    using IN = decltype(in);
    using R = decltype(r);
    constexpr int NT = decltype(nt)::value;
    reduce_final_kernel<NT, IN, R><<<grid, NT, 0, s>>>((const IN*)partials, nrows, wt, coef, (R*)W,
                                                       (R*)FW);
  });
  return hipGetLastError();
}

hipError_t launch_make_w(int dtype, const double* coef, const WeightTables& wt, const double* kd,
                         void* FW, hipStream_t s) {
  const int grid = (wt.lmax + 1) * (wt.lmax + 1);
  if (dtype == 0)
    make_w_kernel<float><<<grid, 64, 0, s>>>(coef, wt, kd, (float*)FW);
  else
    make_w_kernel<double><<<grid, 64, 0, s>>>(coef, wt, kd, (double*)FW);
  return hipGetLastError();
}

hipError_t launch_expand_w(int dtype, const void* W, int rows, const WeightTables& wt, void* FW,
                           hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int64_t stride = FwLayout::elems(wt.nmaxc, wt.lmax, dtype == 0);
  const int L2 = (wt.lmax + 1) * (wt.lmax + 1);
  // (at most 65535 rows per launch: the grid's y limit)
  for (int k0 = 0; k0 < rows; k0 += 65535) {
    const dim3 grid(L2, rows - k0 < 65535 ? rows - k0 : 65535);
    const int64_t wo = (int64_t)k0 * L2 * (wt.nmaxc + 1);
    if (dtype == 0)
      expand_w_kernel<float><<<grid, 64, 0, s>>>((const float*)W + wo, wt,
                                                 (float*)FW + k0 * stride, stride);
    else
      expand_w_kernel<double><<<grid, 64, 0, s>>>((const double*)W + wo, wt,
                                                  (double*)FW + k0 * stride, stride);
  }
  return hipGetLastError();
}

hipError_t launch_kick_drift(int dtype, int64_t n, void* x, void* y, void* z, void* vx, void* vy,
                             void* vz, const void* ax, const void* ay, const void* az, double kick,
                             double drift, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t grid = (n + 255) / 256;
  if (dtype == 0)
    kick_drift_kernel<float><<<dim3((unsigned)grid), 256, 0, s>>>(
        n, (float*)x, (float*)y, (float*)z, (float*)vx, (float*)vy, (float*)vz, (const float*)ax,
        (const float*)ay, (const float*)az, (float)kick, (float)drift);
  else
    kick_drift_kernel<double><<<dim3((unsigned)grid), 256, 0, s>>>(
        n, (double*)x, (double*)y, (double*)z, (double*)vx, (double*)vy, (double*)vz,
        (const double*)ax, (const double*)ay, (const double*)az, kick, drift);
  return hipGetLastError();
}

hipError_t launch_reduce_batched(int dtype, const void* partials, const int32_t* rows, int ncl,
                                 int T, int nchunks, double* red1, hipStream_t s) {
  if (ncl <= 0 || T <= 0) return hipSuccess;
  dim3 grid((T + 63) / 64, nchunks, ncl);
  if (dtype == 0)
    reduce_batched_kernel<float><<<grid, 256, 0, s>>>((const float*)partials, rows, T, nchunks, red1);
  else
    reduce_batched_kernel<double><<<grid, 256, 0, s>>>((const double*)partials, rows, T, nchunks,
                                                       red1);
  return hipGetLastError();
}

hipError_t launch_reduce_final_batched(int dtype, bool chunks_f64, const void* partials,
                                      const int32_t* rows, int nchunks, int max_rows, int ncl,
                                      const WeightTables& wt, double* coef, void* FW,
                                      int64_t W_stride, const double* centre_tab, double* cur,
                                      int* step, hipStream_t s) {
  if (ncl <= 0) return hipSuccess;
  const dim3 grid(grid_rows((wt.lmax + 1) * (wt.lmax + 1)), ncl);
  const int nch = chunks_f64 ? nchunks : 0;
  with_reduce_types(dtype, chunks_f64, max_rows, (int)(grid.x * grid.y), [&](auto nt, auto in, auto r) {
    using IN = decltype(in);
    using R = decltype(r);
    constexpr int NT = decltype(nt)::value;
    reduce_final_batched_kernel<NT, IN, R><<<grid, NT, 0, s>>>(
        (const IN*)partials, rows, nch, wt, coef, (R*)FW, W_stride, centre_tab, ncl, cur, step);
  });
  return hipGetLastError();
}

hipError_t launch_set_int(int* p, int v, hipStream_t s) {
  set_int_kernel<<<1, 64, 0, s>>>(p, v);
  return hipGetLastError();
}

hipError_t launch_fill(double* p, int64_t n, double v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  fill_kernel<<<dim3((unsigned)((n + 255) / 256)), 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// adjoint helpers
// ---------------------------------------------------------------------------
// out[k][q] = sum over blocks b of partials[k][b][q], q < 32, for every kick
// k (one block each), in double and in a fixed order (8 strided block
// subsets, then their sum)
template <typename R>
__global__ void __launch_bounds__(256) adj_reduce_kernel(const R* __restrict__ partials,
                                                         int64_t nblocks, double* out) {
  __shared__ double sh[8][32];
  const int q = threadIdx.x & 31, part = threadIdx.x >> 5;
  const R* pk = partials + (int64_t)blockIdx.x * nblocks * 32;
  double s = 0.0;
  for (int64_t b = part; b < nblocks; b += 8) s += double(pk[b * 32 + q]);
  sh[part][q] = s;
  __syncthreads();
  if (part == 0) {
    double t = 0.0;
    for (int k = 0; k < 8; ++k) t += sh[k][q];
    out[(int64_t)blockIdx.x * 32 + q] = t;
  }
}

hipError_t launch_adj_reduce(int dtype, const void* partials, int64_t nblocks, int nkicks,
                             double* out, hipStream_t s) {
  if (nkicks <= 0) return hipSuccess;
  if (dtype == 0)
    adj_reduce_kernel<float><<<nkicks, 256, 0, s>>>((const float*)partials, nblocks, out);
  else
    adj_reduce_kernel<double><<<nkicks, 256, 0, s>>>((const double*)partials, nblocks, out);
  return hipGetLastError();
}

// Power per degree: E_l = sum_n [a_nl0^2 + 2 sum_{m>=1} (Re^2 + Im^2)], one
// block per degree, a fixed-order tree over the block.
__global__ void __launch_bounds__(256) power_kernel(const double* __restrict__ coef, int nmax,
                                                    int lmax, double* El) {
  __shared__ double sh[256];
  const int l = blockIdx.x;
  const int L2 = (lmax + 1) * (lmax + 1);
  const int per = 2 * l + 1;
  double s = 0.0;
  for (int q = threadIdx.x; q < (nmax + 1) * per; q += blockDim.x) {
    const int n = q / per, j = q % per;
    const double a = coef[(int64_t)n * L2 + l * l + j];
    s += (j == 0 ? 1.0 : 2.0) * a * a;
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) El[l] = sh[0];
}

hipError_t launch_power(const double* coef, int nmax, int lmax, int ncl, double* El,
                        hipStream_t s) {
  const int64_t T = (int64_t)(nmax + 1) * (lmax + 1) * (lmax + 1);
  for (int c = 0; c < ncl; ++c) {
    power_kernel<<<lmax + 1, 256, 0, s>>>(coef + c * T, nmax, lmax, El + (int64_t)c * (lmax + 1));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

Engine* find_engine(int dtype, int nmax, int lmax) {
  if (nmax < 0 || lmax < 0) return nullptr;
  Engine* e = dtype == 0 ? find_engine_f32_exact(nmax, lmax) : find_engine_f64_exact(nmax, lmax);
  if (e) return e;
  return dtype == 0 ? find_engine_f32_generic(nmax, lmax) : find_engine_f64_generic(nmax, lmax);
}

}  // namespace scf
