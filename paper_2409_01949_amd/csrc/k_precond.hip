// Block-Jacobi preconditioning of the least-squares system from the diagonal Gram blocks.
//
// The random features of one subdomain are strongly redundant, which is the main source of
// the huge condition numbers of M (Sec. 5 "Conditioning and redundancy").  Right
// preconditioning with the block-diagonal R, R_j^T R_j = G_jj + lambda_j I (a Cholesky factor of
// each subdomain's Gram block, shifted by lambda_j = shift * trace(G_jj)/K), orthonormalises
// every subdomain's columns over its own support; LSQR then runs on M R^{-1} and the solution
// is x = R^{-1} y.  Factors are computed once in FP64 (k_factor.hip) and R^{-1} is stored
// explicitly together with its transpose, so both applications read memory contiguously.
#include "device.h"
#include "kernels.h"

namespace elmfb {

// The three applications below are batched upper-triangular matrix-vector products, one K x K
// factor per subdomain.  Work is split into tasks of 32 output coefficients of one block; a
// workgroup of 256 threads takes a task at a time (grid-stride), thread t owns output
// coefficient t % 32 and sums every 8th term of its dot product (split t / 32), and the 8
// partial sums are added in a fixed order through LDS.  Consecutive threads read consecutive
// factor entries.
constexpr int kBjRows = 32;
constexpr int kBjSplit = 8;

__device__ __forceinline__ int bj_tasks(const Geo& g) {
  return g.n_blocks * ((g.K + kBjRows - 1) / kBjRows);
}

// y = R^{-1} (v * scale):  y_i = sum_{k >= i} Ri[i][k] v_k = sum_k T[k][i] v_k; with red (may be
// NULL) also the partials of r . y.
__global__ void __launch_bounds__(256) k_bj_apply(Geo g, const double* __restrict__ rinvT,
                                                  const double* __restrict__ v,
                                                  const double* __restrict__ scale,
                                                  double* __restrict__ y,
                                                  const SolveState* __restrict__ st,
                                                  const double* __restrict__ r,
                                                  double* __restrict__ red) {
  __shared__ double part[kBjSplit][kBjRows];
  __shared__ double sh[4];
  if (st && st->done) return;
  double acc = 0.0;
  const int K = g.K;
  const int per = (K + kBjRows - 1) / kBjRows;
  const double sc = scale ? *scale : 1.0;
  const int ro = threadIdx.x % kBjRows, sp = threadIdx.x / kBjRows;
  for (int task = blockIdx.x; task < bj_tasks(g); task += gridDim.x) {
    const int b = task / per, i = (task - b * per) * kBjRows + ro;
    const int64_t q0 = (int64_t)b * K;
    const double* T = rinvT + (int64_t)b * K * K;
    double s = 0.0;
    if (i < K)
      for (int k = i + sp; k < K; k += kBjSplit) s += T[(int64_t)k * K + i] * v[q0 + k];
    part[sp][ro] = s;
    __syncthreads();
    if (sp == 0 && i < K) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < kBjSplit; ++q) t += part[q][ro];
      y[q0 + i] = t * sc;
      if (red) acc += r[q0 + i] * (t * sc);
    }
    __syncthreads();
  }
  if (red) {
    const double t = block_sum256(acc, sh);
    if (threadIdx.x == 0) red[blockIdx.x] = t;
  }
}

// z = R^{-T} x:  z_k = sum_{i <= k} Ri[i][k] x_i, then the LSQR epilogue on v
// (v = z - beta sv v, partial ||v||^2) or a plain store (COL_STORE / COL_STORE_SQ).
__global__ void __launch_bounds__(256) k_bj_apply_t(Geo g, const double* __restrict__ rinv,
                                                    const double* __restrict__ x, int mode,
                                                    double* __restrict__ out,
                                                    const SolveState* __restrict__ st,
                                                    double* __restrict__ red) {
  __shared__ double part[kBjSplit][kBjRows];
  __shared__ double sh[4];
  if (st && st->done) return;
  const int K = g.K;
  const int per = (K + kBjRows - 1) / kBjRows;
  double coef_v = 0.0;
  bool keep = false;
  if (mode == COL_LSQR_V) {
    coef_v = st->beta * st->sv;
    keep = !(st->beta > 0.0);
  }
  const int ro = threadIdx.x % kBjRows, sp = threadIdx.x / kBjRows;
  double acc = 0.0;
  for (int task = blockIdx.x; task < bj_tasks(g); task += gridDim.x) {
    const int b = task / per, k = (task - b * per) * kBjRows + ro;
    const int64_t q0 = (int64_t)b * K;
    const double* Ri = rinv + (int64_t)b * K * K;
    double s = 0.0;
    if (k < K)
      for (int i = sp; i <= k; i += kBjSplit) s += Ri[(int64_t)i * K + k] * x[q0 + i];
    part[sp][ro] = s;
    __syncthreads();
    if (sp == 0 && k < K) {
      double z = 0.0;
#pragma unroll
      for (int q = 0; q < kBjSplit; ++q) z += part[q][ro];
      if (mode == COL_STORE) {
        out[q0 + k] = z;
      } else if (mode == COL_LSQR_V) {
        double vv = out[q0 + k];
        if (!keep) { vv = z - coef_v * vv; out[q0 + k] = vv; }
        acc += vv * vv;
      } else {
        out[q0 + k] = z;
        acc += z * z;
      }
    }
    __syncthreads();
  }
  if (mode != COL_STORE) {
    const double t = block_sum256(acc, sh);
    if (threadIdx.x == 0) red[blockIdx.x] = t;
  }
}

// x = x0 + R^{-1} y  (x0 may be NULL).  x0 and x may be the same vector: each element is read
// and then written by one thread, after every read of y.
__global__ void __launch_bounds__(256) k_bj_recover(Geo g, const double* __restrict__ rinvT,
                                                    const double* __restrict__ yv,
                                                    const double* x0, double* x) {
  __shared__ double part[kBjSplit][kBjRows];
  const int K = g.K;
  const int per = (K + kBjRows - 1) / kBjRows;
  const int ro = threadIdx.x % kBjRows, sp = threadIdx.x / kBjRows;
  for (int task = blockIdx.x; task < bj_tasks(g); task += gridDim.x) {
    const int b = task / per, i = (task - b * per) * kBjRows + ro;
    const int64_t q0 = (int64_t)b * K;
    const double* T = rinvT + (int64_t)b * K * K;
    double s = 0.0;
    if (i < K)
      for (int k = i + sp; k < K; k += kBjSplit) s += T[(int64_t)k * K + i] * yv[q0 + k];
    part[sp][ro] = s;
    __syncthreads();
    if (sp == 0 && i < K) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < kBjSplit; ++q) t += part[q][ro];
      x[q0 + i] = (x0 ? x0[q0 + i] : 0.0) + t;
    }
    __syncthreads();
  }
}

int bj_wg(const Geo& g) {
  const int tasks = g.n_blocks * ((g.K + kBjRows - 1) / kBjRows);
  return tasks < kRedBlocks ? tasks : kRedBlocks;
}

hipError_t launch_bj_apply(const Geo& g, const double* rinvT, const double* v,
                           const double* scale, double* y, const SolveState* st, const double* r,
                           double* red, hipStream_t s) {
  hipLaunchKernelGGL(k_bj_apply, dim3(bj_wg(g)), dim3(256), 0, s, g, rinvT, v, scale, y, st, r, red);
  return hipGetLastError();
}
hipError_t launch_bj_apply_t(const Geo& g, const double* rinv, const double* x, int mode,
                             double* out, const SolveState* st, double* red, hipStream_t s) {
  hipLaunchKernelGGL(k_bj_apply_t, dim3(bj_wg(g)), dim3(256), 0, s, g, rinv, x, mode, out, st,
                     red);
  return hipGetLastError();
}
hipError_t launch_bj_recover(const Geo& g, const double* rinvT, const double* y, const double* x0,
                             double* x, hipStream_t s) {
  hipLaunchKernelGGL(k_bj_recover, dim3(bj_wg(g)), dim3(256), 0, s, g, rinvT, y, x0, x);
  return hipGetLastError();
}

}  // namespace elmfb
