// Block-Jacobi preconditioning of the least-squares system from the diagonal Gram blocks.
//
// The random features of one subdomain are strongly redundant, which is the main source of
// the huge condition numbers of M (Sec. 5 "Conditioning and redundancy").  Right
// preconditioning with the block-diagonal R, R_j^T R_j = G_jj + lambda_j I (a Cholesky factor of
// each subdomain's Gram block, shifted by lambda_j = shift * trace(G_jj)/K), orthonormalises
// every subdomain's columns over its own support; LSQR then runs on M R^{-1} and the solution
// is x = R^{-1} y.  Factors are computed once in FP64 (k_factor.hip) and R^{-1} is stored
// explicitly together with its transpose, so both applications read memory contiguously.
#include <algorithm>

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
static_assert(kGcgBlockK == 128, "row groups of k_gcg_block");

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

// The middle of a preconditioned CG step on the Gram blocks, one subdomain block per workgroup:
// al = gamma / (p . q) as in k_gcg_update, a += al p ; r -= al q, then, as r is the block's
// own, z = R^{-1} (R^{-T} r) through LDS and the partials of r . r and r . z.  The sums of z run as in
// k_bj_apply_t and k_bj_apply, whose launches this saves.  Bound by latency (launches, then the
// chain of sums); KB: K rounded up to 64 or 128; up to 64 both factors' entries are loaded before
// the step size is known, 8.5 -> 7.3 us.  A step in all, 6 -> 4 kernels: 81 blocks of K = 48 37 -> 32
// us, 4 of K = 128 30.1 -> 29.4, 273 of K = 128 204 -> 193.
template <int KB>
__global__ void __launch_bounds__(256) k_gcg_block(
    Geo g, double* __restrict__ a, double* __restrict__ r, const double* __restrict__ p,
    const double* __restrict__ q, const double* __restrict__ rinv,
    const double* __restrict__ rinvT, double* __restrict__ z, SolveState* st,
    const double* __restrict__ red_pq, int n, double* __restrict__ red_rr,
    double* __restrict__ red_rz) {
  constexpr int G = KB / kBjRows, L = KB / kBjSplit;   // row groups, terms of a split
  __shared__ double part[G][kBjSplit][kBjRows];
  __shared__ double rs[KB], ts[KB];
  __shared__ double sh[6];
  const int K = g.K;
  const int ro = threadIdx.x % kBjRows, sp = threadIdx.x / kBjRows;
  double ri[G][L], rt[G][L];
  // row o = kBjRows i + ro of R^{-T} (terms k <= o) or, upper, of R^{-1} (k >= o): term l of split sp
  auto load = [&](double (&x)[G][L], const double* F, bool upper) {
#pragma unroll
    for (int i = 0; i < G; ++i)
#pragma unroll
      for (int l = 0; l < L; ++l) {
        const int o = kBjRows * i + ro, k = upper ? o + sp + kBjSplit * l : sp + kBjSplit * l;
        x[i][l] = o < K && (upper ? k < K : k <= o) ? F[(int64_t)k * K + o] : 0.0;
      }
  };
  // its product with v: row kBjRows sp + ro in the threads with sp < G
  auto apply = [&](const double (&x)[G][L], const double* v, bool upper) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      double s = 0.0;
#pragma unroll
      for (int l = 0; l < L; ++l) {
        const int o = kBjRows * i + ro, k = upper ? o + sp + kBjSplit * l : sp + kBjSplit * l;
        if (o < K && (upper ? k < K : k <= o)) s += x[i][l] * v[k];
      }
      part[i][sp][ro] = s;
    }
    __syncthreads();
    double t = 0.0;
    if (sp < G) {
#pragma unroll
      for (int u = 0; u < kBjSplit; ++u) t += part[sp][u][ro];
    }
    return t;
  };
  int b = blockIdx.x;
  load(ri, rinv + (int64_t)b * K * K, false);
  if constexpr (KB <= 64) load(rt, rinvT + (int64_t)b * K * K, true);
  bool live;
  const double gamma = st->next_gamma;
  const double pq = reduce_partials_live(red_pq, n, &st->done, sh, &live);
  if (!live) return;
  const bool ok = pq > 0.0;
  const double al = ok ? gamma / pq : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->gamma = gamma;
    if (!ok) {
      st->istop = 3;
      st->done = 1;
    }
  }
  if (!ok) return;
  const int row = kBjRows * sp + ro;
  double rr = 0.0, rz = 0.0;
  while (true) {
    const int64_t q0 = (int64_t)b * K;
    if ((int)threadIdx.x < K) {
      const int64_t t = q0 + threadIdx.x;
      a[t] += al * p[t];
      const double x = r[t] - al * q[t];
      r[t] = x;
      rs[threadIdx.x] = x;
      rr += x * x;
    }
    __syncthreads();
    const double y = apply(ri, rs, false);
    if (sp < G && row < K) ts[row] = y;
    if constexpr (KB > 64) load(rt, rinvT + q0 * K, true);
    __syncthreads();
    const double x = apply(rt, ts, true);
    if (sp < G && row < K) {
      z[q0 + row] = x;
      rz += rs[row] * x;
    }
    b += gridDim.x;
    if (b >= g.n_blocks) break;
    load(ri, rinv + (int64_t)b * K * K, false);
    if constexpr (KB <= 64) load(rt, rinvT + (int64_t)b * K * K, true);
    __syncthreads();   // rs, ts and part are used again
  }
  rr = block_sum256(rr, sh);
  rz = block_sum256(rz, sh);
  if (threadIdx.x == 0) {
    red_rr[blockIdx.x] = rr;
    red_rz[blockIdx.x] = rz;
  }
}

int gcg_block_wg(const Geo& g) { return std::min(g.n_blocks, kRedBlocks); }

hipError_t launch_gcg_block(const Geo& g, double* a, double* r, const double* p, const double* q,
                            const double* rinv, const double* rinvT, double* z, SolveState* st,
                            const double* red_pq, int n_red, double* red_rr, double* red_rz,
                            hipStream_t s) {
  if (g.K > kGcgBlockK) return hipErrorInvalidValue;
#define GCG_BLOCK(KB)                                                                            \
  hipLaunchKernelGGL(k_gcg_block<KB>, dim3(gcg_block_wg(g)), dim3(256), 0, s, g, a, r, p, q, rinv, \
                     rinvT, z, st, red_pq, n_red, red_rr, red_rz)
  if (g.K <= 64) GCG_BLOCK(64); else GCG_BLOCK(128);
#undef GCG_BLOCK
  return hipGetLastError();
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
