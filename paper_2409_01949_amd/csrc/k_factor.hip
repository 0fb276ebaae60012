// Block-Jacobi factors: for every block b the upper Cholesky factor R of G_b + lambda I (lambda =
// shift trace(G_b)/K_b, G_b the diagonal Gram block) and X = R^{-1}, K_b <= 512 columns.
//
// Blocks of up to 16 columns (24 in some launches, factor_by_width) take one wavefront each, in
// registers: k_bj_factor_tile.  All others one workgroup per block (k_bj_factor), left-looking by
// panels of 32 rows on v_mfma_f64_16x16x4_f64, matrices K x K row-major in global memory (G read only, R into W, X apart), the 16 rows being finished in LDS:
//   R rows I:  S = G[I, J] - sum_{s < I} R[s, I]^T R[s, J]  (matrix cores, accumulators started at
//              G, s ascending), then the 16 x 16 diagonal block in the registers of one wavefront
//              (a column per lane, pivot rows by lane reads) and a column of S per thread by
//              substitution;
//   X rows I, from the bottom: S = E[I, J] - sum_{s > I} R[I, s] X[s, J], then back substitution.
// The second 16 rows of a panel take the first 16 from LDS.  Both operands of the first sum are
// rows of R, so every fragment load is four runs of 128 bytes and nothing is staged; 32-row
// panels because a B fragment then serves two products, which keeps the loads under what the
// caches deliver per CU.  Every entry's sum runs in the order of the unblocked elimination.
//
// Bound by the FP64 matrix rate, K^3/3 products a block, and by the 2 K/16 sequential 16-row steps,
// which workgroups on one CU overlap: at most 128 registers a lane (four wavefronts a SIMD; 124
// and no spills to 256 columns, 34 spilled above).  This file is compiled at -O1: from -O2 on,
// value numbering keeps the unrolled steps' operands in registers and the kernel takes 256 and
// spills.  Precondition calls, all kernels, -O3 at 256 registers / -O1 / -O1 at 128: 32 instances
// 8.0 / 6.5 / 6.0 ms, the same over 2 x 2 patches 40.9 / 39.2 / 36.8.
// Against one column per thread and scalar updates, this kernel alone: 16 instances over 2 x 2
// patches (K to 512) 28.1 -> 2.9 ms; 32 instances (blocks of K = 64 to 128, then in LDS with two
// barriers a row) 4.5 -> 1.3 ms; 273 blocks of K = 96 1,119 -> 125 us.
//
// A failed factorisation is retried with a 100x larger shift, 8 attempts in all; after that, or
// for an all-zero block, the block gets the identity.
#include "device.h"
#include "kernels.h"

namespace elmfb {

typedef double d4_t __attribute__((ext_vector_type(4)));

constexpr int kFacDiag = 17;   // row stride of the 16 x 16 diagonal block in LDS

// A value the optimiser takes as new: what is computed from it stays in its loop (hoisted out, the
// addresses of every unrolled tile together spill).
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The N x N diagonal block (N <= 32) in Pn[0..N)[c0..c0 + N) plus lam I by one wavefront: its Cholesky
// factor to D (zero below the diagonal) and the reciprocals of its diagonal to dinv; prow: LN doubles
// of LDS for the pivot row.  Rows and columns from nb on become the identity's first.  False on a
// pivot <= 0.
template <int N>
__device__ __forceinline__ bool factor_diag(double* Pn, const int pw, int c0, int nb, double lam,
                                            double* D, double* dinv, double* prow) {
  constexpr int LN = N > 16 ? 32 : 16, LD = LN + 1;   // lanes to a row, row stride of D
  const int li = threadIdx.x % LN;
  for (int i = (threadIdx.x & 63) / LN; nb < N && i < N; i += 64 / LN)
    if (i >= nb || li >= nb) Pn[i * pw + c0 + li] = i == li ? 1.0 : 0.0;
  __builtin_amdgcn_wave_barrier();       // LDS is in order within a wavefront
  double col[N];
#pragma unroll
  for (int i = 0; i < N; ++i) col[i] = Pn[i * pw + c0 + li] + (i == li ? lam : 0.0);
  bool ok = true;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double d = lane_value(col[k], k);
    ok = ok && d > 0.0;
    const double rk = sqrt(d > 0.0 ? d : 1.0);
    col[k] = li == k ? rk : col[k] / rk;
    if (li == k) dinv[k] = 1.0 / rk;
    prow[li] = col[k];                   // the lanes of a column write the same value; in order within a wave
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = k + 1; i < N; ++i) col[i] -= prow[i] * col[k];
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int i = 0; i < N; ++i) D[i * LD + li] = li >= i ? col[i] : 0.0;
  return ok;
}

// FULL: every block has the same K, X goes to rinv (K x K row-major, zero below the diagonal) and
// its transpose to rinvT (single problems).  Otherwise X is left in Xg (the Gram scratch itself)
// and goes out column-packed at foff[b] of rc (batches).  goff: element offset of block b in G, W
// and Xg.  nfail counts the identity fallbacks (single problems do not count all-zero blocks).
// NW wavefronts of NC 16-column tiles: K <= 16 NW NC.  The empty asm statements in the unrolled
// 16-row steps keep the compiler from loading a whole step's operands ahead (it spills then).
template <int NW, int NC, bool FULL>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4)))
k_bj_factor(const DevBlock* __restrict__ blocks,
                                                       int blk0, int Kall,
                                                       const double* G, double* W, double* Xg,
                                                       const int64_t* __restrict__ goff,
                                                       const int64_t* __restrict__ foff,
                                                       double shift, double* __restrict__ rc,
                                                       double* __restrict__ rinvT,
                                                       int32_t* __restrict__ nfail) {
  constexpr int NT = 64 * NW;
  constexpr int pw = 16 * NW * NC + 8;         // 8 past a multiple of 32: rows on other banks
  extern __shared__ double Pn[];               // 16 rows of pw columns
  __shared__ double D[16 * kFacDiag], dinv[16], prow[16], part[NW];
  __shared__ int bad_s;
  const int b = blk0 + (int)blockIdx.x;
  const int K = FULL ? Kall : blocks[b].nk;
  const int64_t o = FULL ? (int64_t)b * K * K : goff[b];
  const double* Gb = G + (FULL ? goff[b] : o);
  double* Wb = W + o;
  double* X = Xg + o;
  double* Pc = FULL ? nullptr : rc + foff[b];
  double* XT = FULL ? rinvT + o : nullptr;
  const int t = threadIdx.x, lane = t & 63;
  const int wid = __builtin_amdgcn_readfirstlane(t >> 6);   // scalar: tile tests are branches
  double tr = 0.0;
  for (int i = t; i < K; i += NT) tr += Gb[i * K + i];
  tr = wave_sum(tr);
  if (lane == 0) part[wid] = tr;
  __syncthreads();
  tr = 0.0;
  for (int w = 0; w < NW; ++w) tr += part[w];
  double lam = shift * tr / K;
  const bool zero = !(lam > 0.0);
  bool bad = true;
  // Tiles past column K repeat the last column: their results are never read, the diagonal blocks
  // being bordered with the identity there.
  for (int attempt = 0; attempt < 8 && bad && !zero; ++attempt) {
    if (attempt) lam *= 100.0;
    bad = false;
    for (int ib = 0; ib < K && !bad; ib += 32) {
      const int nct = (K - ib + 15) >> 4;      // column tiles from ib
      const int li = fresh(lane & 15), lq = fresh(lane >> 4);
      d4_t acc[2][NC];
      int col[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        col[c] = min(ib + 16 * (wid + NW * c) + li, K - 1);
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            acc[r][c][v] = Gb[(unsigned)(min(ib + 16 * r + lq + 4 * v, K - 1) * K + col[c])];
      }
      const unsigned a0 = min(ib + li, K - 1), a1 = min(ib + 16 + li, K - 1);
#pragma unroll 2
      for (int s = 0; s < ib; s += 4) {
        const unsigned row = (unsigned)((s + lq) * K);
        const double x0 = -Wb[row + a0], x1 = -Wb[row + a1];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if (wid + NW * c < nct) {
            const double y = Wb[row + col[c]];
            acc[0][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y, acc[0][c], 0, 0, 0);
            acc[1][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y, acc[1][c], 0, 0, 0);
          }
        }
      }
      // the first 16 rows go on to Pn; the second wait in W, where R will take their place
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int j = 16 * (wid + NW * c) + li;
        if (wid + NW * c < nct) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int i = lq + 4 * v;
            Pn[i * pw + j] = acc[0][c][v];
            if (ib + 16 + i < K && ib + j < K) Wb[(unsigned)((ib + 16 + i) * K + ib + j)] = acc[1][c][v];
          }
        }
      }
#pragma unroll 1
      for (int r = 0; r < 2 && ib + 16 * r < K; ++r) {
        const int i0 = ib + 16 * r;
        __syncthreads();
        if (r == 1) {
          const int li = fresh(lane & 15), lq = fresh(lane >> 4);
          // less the products with the first 16 rows of the panel, which are in Pn
          d4_t a1[NC];
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const int ct = wid + NW * c, j = min(ib + 16 * ct + li, K - 1);
            if (ct < nct) {
#pragma unroll
              for (int v = 0; v < 4; ++v)
                a1[c][v] = Wb[(unsigned)(min(i0 + lq + 4 * v, K - 1) * K + j)];
#pragma unroll
              for (int q = 0; q < 16; q += 4)
                a1[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(-Pn[(q + lq) * pw + 16 + li],
                                                             Pn[(q + lq) * pw + 16 * ct + li],
                                                             a1[c], 0, 0, 0);
            }
          }
          __syncthreads();
#pragma unroll
          for (int c = 0; c < NC; ++c)
            if (wid + NW * c < nct) {
#pragma unroll
              for (int v = 0; v < 4; ++v)
                Pn[(lq + 4 * v) * pw + 16 * (wid + NW * c) + li] = a1[c][v];
            }
          __syncthreads();
        }
        if (wid == 0) {
          const bool ok = factor_diag<16>(Pn, pw, 16 * r, K - i0, lam, D, dinv, prow);
          if (lane == 0) bad_s = !ok;
        }
        __syncthreads();
        bad = bad_s != 0;
        if (bad) break;
#pragma unroll 1
        for (int j = 16 * r + t; j < 16 * nct; j += NT) {
          asm volatile("" ::: "memory");       // D stays in LDS (else hoisted: 240 registers)
          double p[16];
          const int jr = j - 16 * r;           // below 16: the diagonal block itself
          if (jr < 16) {
#pragma unroll
            for (int i = 0; i < 16; ++i) p[i] = D[i * kFacDiag + jr];
          } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) p[i] = Pn[i * pw + j];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              asm volatile("" ::: "memory");
              p[i] *= dinv[i];
#pragma unroll
              for (int q = i + 1; q < 16; ++q) p[q] -= D[i * kFacDiag + q] * p[i];
            }
          }
          const unsigned out = (unsigned)(i0 * K + ib + j);
          const int rows = ib + j < K ? K - i0 : 0;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            Pn[i * pw + j] = p[i];
            if (i < rows) Wb[out + (unsigned)(i * K)] = p[i];
          }
        }
        __syncthreads();
      }
    }
    __syncthreads();
  }
  if (bad) {
    if (t == 0 && !(FULL && zero)) atomicAdd(nfail, 1);
    if constexpr (FULL) {
      for (int e = t; e < K * K; e += NT) {
        const double v = e / K == e - e / K * K ? 1.0 : 0.0;
        X[e] = v;
        XT[e] = v;
      }
    } else {
      for (int64_t e = t; e < (int64_t)K * (K + 1) / 2; e += NT) Pc[e] = 0.0;
      __syncthreads();
      for (int i = t; i < K; i += NT) Pc[(int64_t)i * (i + 1) / 2 + i] = 1.0;
    }
    return;
  }
  for (int ib = (K - 1) / 32 * 32; ib >= 0; ib -= 32) {
    const int nct = (K - ib + 15) >> 4;
    const int li = fresh(lane & 15), lq = fresh(lane >> 4);
    d4_t acc[2][NC];
    int col[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      col[c] = min(ib + 16 * (wid + NW * c) + li, K - 1);
      acc[0][c] = acc[1][c] = d4_t{0, 0, 0, 0};
    }
    // rows of R from ib, columns s; X[s][j] is zero for s > j
    const unsigned r0 = (unsigned)(min(ib + li, K - 1) * K);
    const unsigned r1 = (unsigned)(min(ib + 16 + li, K - 1) * K);
#pragma unroll 2
    for (int s = ib + 32; s < K; s += 4) {
      const int k = s + lq, kc = min(k, K - 1);
      const double x0 = k < K ? -Wb[r0 + kc] : 0.0, x1 = k < K ? -Wb[r1 + kc] : 0.0;
      const unsigned row = (unsigned)(kc * K);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int ct = wid + NW * c;
        if (ct < nct && s <= ib + 16 * ct + 15) {
          const double y = X[row + col[c]];
          acc[0][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y, acc[0][c], 0, 0, 0);
          acc[1][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y, acc[1][c], 0, 0, 0);
        }
      }
    }
    // the lower 16 rows go on to Pn; the upper wait in X, where their result will take their place
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = 16 * (wid + NW * c) + li;
      if (wid + NW * c < nct) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = lq + 4 * v;
          Pn[i * pw + j] = acc[1][c][v];
          if (ib + i < K && ib + j < K) X[(unsigned)((ib + i) * K + ib + j)] = acc[0][c][v];
        }
      }
    }
#pragma unroll 1
    for (int r = 1; r >= 0; --r) {
      const int i0 = ib + 16 * r;
      __syncthreads();
      if (i0 >= K) continue;
      if (r == 0) {
        const int li = fresh(lane & 15), lq = fresh(lane >> 4);
        const unsigned r0 = (unsigned)(min(ib + li, K - 1) * K);
        // less the products with the lower 16 rows of the panel, which are in Pn
        d4_t a0[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int ct = wid + NW * c, j = min(ib + 16 * ct + li, K - 1);
          if (ct < nct) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              a0[c][v] = X[(unsigned)(min(ib + lq + 4 * v, K - 1) * K + j)];
            if (ib + 16 < K) {
#pragma unroll
              for (int q = 0; q < 16; q += 4) {
                const int k = ib + 16 + q + lq;
                const double x0 = k < K ? -Wb[r0 + min(k, K - 1)] : 0.0;
                a0[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                    x0, Pn[(q + lq) * pw + 16 * ct + li], a0[c], 0, 0, 0);
              }
            }
          }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if (wid + NW * c < nct) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              Pn[(lq + 4 * v) * pw + 16 * (wid + NW * c) + li] = a0[c][v];
          }
      }
      for (int e = t; e < 256; e += NT) {
        const int i = e >> 4, j = e & 15;
        const double d = i0 + i < K && i0 + j < K ? Wb[(unsigned)((i0 + i) * K + i0 + j)]
                                                  : (i == j ? 1.0 : 0.0);
        D[i * kFacDiag + j] = d;
        if (i == j) dinv[i] = 1.0 / d;
      }
      __syncthreads();
#pragma unroll 1
      for (int j = t; j < 16 * nct; j += NT) {
        asm volatile("" ::: "memory");
        double p[16];
        const bool in = ib + j < K;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          p[i] = j >= 16 * r && i0 + i < K ? Pn[i * pw + j] : 0.0;
          p[i] += j - 16 * r == i ? 1.0 : 0.0;      // the right-hand side, E
        }
#pragma unroll
        for (int i = 15; i >= 0; --i) {
          asm volatile("" ::: "memory");
          p[i] *= dinv[i];
#pragma unroll
          for (int q = 0; q < i; ++q) p[q] -= D[q * kFacDiag + i] * p[i];
        }
        const int jc = ib + j, rows = in ? K - i0 : 0;
        const unsigned out = (unsigned)(i0 * K + jc);
        double* outT = FULL ? XT : Pc;
        const unsigned ot = (unsigned)((FULL ? jc * K : jc * (jc + 1) / 2) + i0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          Pn[i * pw + j] = p[i];
          if (i < rows) {
            X[out + (unsigned)(i * K)] = p[i];
            if (FULL || i0 + i <= jc) outT[ot + i] = p[i];
          }
        }
      }
      if constexpr (FULL) {
        for (int e = t; e < 16 * ib; e += NT) {   // left of the panel
          const int i = e / ib, j = e - e / ib * ib;
          if (i0 + i < K) {
            X[(unsigned)((i0 + i) * K + j)] = 0.0;
            XT[(unsigned)(j * K + i0 + i)] = 0.0;
          }
        }
      }
      __syncthreads();
    }
  }
}

// K <= N <= 32: one wavefront a block, the inverse a column per lane; arguments as above, without W.
// A chain of K pivots without the panels' barriers: 60 batched blocks of K = 4 / 7 / 16 / 20 take a
// precondition call of 41.7 / 47.6 / 47.7 / 60.0 us, 60.9 / 60.4 / 60.8 / 65.6 by panels.
template <bool FULL, int N>
__global__ void __launch_bounds__(64) k_bj_factor_tile(const DevBlock* __restrict__ blocks, int blk0,
                                                       int Kall, const double* __restrict__ G,
                                                       double* __restrict__ X,
                                                       const int64_t* __restrict__ goff,
                                                       const int64_t* __restrict__ foff, double shift,
                                                       double* __restrict__ rc,
                                                       double* __restrict__ rinvT,
                                                       int32_t* __restrict__ nfail) {
  constexpr int LN = N > 16 ? 32 : 16, LD = LN + 1;
  __shared__ double S[N * LD], D[N * LD], dinv[LN], prow[LN];
  const int b = blk0 + (int)blockIdx.x, K = FULL ? Kall : blocks[b].nk;
  const int li = threadIdx.x % LN;
  const double* Gb = G + goff[b];
  for (int i = threadIdx.x / LN; i < N; i += 64 / LN)
    S[i * LD + li] = i < K && li < K ? Gb[min(i, li) * K + max(i, li)] : 0.0;
  __builtin_amdgcn_wave_barrier();
  double tr = (int)threadIdx.x < K ? S[li * LD + li] : 0.0;
  tr = wave_sum(tr);
  double lam = shift * tr / K;
  const bool zero = !(lam > 0.0);
  bool bad = true;
  for (int attempt = 0; attempt < 8 && bad && !zero; ++attempt) {
    if (attempt) lam *= 100.0;
    bad = !factor_diag<N>(S, LD, 0, K, lam, D, dinv, prow);
  }
  if (bad && threadIdx.x == 0 && !(FULL && zero)) atomicAdd(nfail, 1);
  __builtin_amdgcn_wave_barrier();
  double p[N];
#pragma unroll
  for (int i = 0; i < N; ++i) p[i] = i == li ? 1.0 : 0.0;
  if (!bad) {
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
      p[i] *= dinv[i];
#pragma unroll
      for (int q = 0; q < i; ++q) p[q] -= D[q * LD + i] * p[i];
    }
  }
  if (threadIdx.x >= K) return;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i >= K) break;
    if constexpr (FULL) {
      X[(int64_t)b * K * K + i * K + li] = p[i];
      rinvT[(int64_t)b * K * K + li * K + i] = p[i];
    } else if (i <= li) {
      rc[foff[b] + li * (li + 1) / 2 + i] = p[i];
    }
  }
}

template <int NW, int NC, bool FULL>
static hipError_t factor_launch(const DevBlock* blocks, int blk0, int64_t n_blocks, int kmax,
                                const double* G, double* W, double* X, const int64_t* goff,
                                const int64_t* foff, double shift, double* rc, double* rinvT,
                                int32_t* nfail, hipStream_t s) {
  constexpr int pw = 16 * NW * NC + 8;
  const size_t lds = (size_t)16 * pw * sizeof(double);
  if (lds > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)k_bj_factor<NW, NC, FULL>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_bj_factor<NW, NC, FULL>), dim3((unsigned)n_blocks), dim3(64 * NW), lds, s,
                     blocks, blk0, kmax, G, W, X, goff, foff, shift, rc, rinvT, nfail);
  return hipGetLastError();
}

// One wavefront to 16 columns, and to 24 where that gives no more than one to a SIMD (it takes all
// registers: 256 blocks of K = 20 66 against 72 us, 4,096 313 against 295); four of two tiles to 128
// columns (several workgroups a CU overlap the sequential steps), eight of two to 256 and of four to
// 512.
template <bool FULL>
static hipError_t factor_by_width(const DevBlock* blocks, int blk0, int64_t n_blocks, int kmax,
                                  const double* G, double* W, double* X, const int64_t* goff,
                                  const int64_t* foff, double shift, double* rc, double* rinvT,
                                  int32_t* nfail, hipStream_t s) {
  if (kmax < 1 || kmax > kPatchMaxK) return hipErrorInvalidValue;
  if (n_blocks == 0) return hipSuccess;
  if (kmax <= 16 || (kmax <= 24 && n_blocks <= 1024)) {
    const auto tile = kmax <= 4    ? k_bj_factor_tile<FULL, 4>
                      : kmax <= 16 ? k_bj_factor_tile<FULL, 16>
                                   : k_bj_factor_tile<FULL, 24>;
    hipLaunchKernelGGL(tile, dim3((unsigned)n_blocks), dim3(64), 0, s, blocks, blk0, kmax, G, X, goff,
                       foff, shift, rc, rinvT, nfail);
    return hipGetLastError();
  }
  const auto launch = kmax <= 128   ? factor_launch<4, 2, FULL>
                      : kmax <= 256 ? factor_launch<8, 2, FULL>
                                    : factor_launch<8, 4, FULL>;
  return launch(blocks, blk0, n_blocks, kmax, G, W, X, goff, foff, shift, rc, rinvT, nfail, s);
}

hipError_t launch_bj_factor(const Geo& g, const double* G, const int64_t* diag_off, double shift,
                            double* work, double* rinv, double* rinvT, int32_t* nfail,
                            hipStream_t s) {
  return factor_by_width<true>(nullptr, 0, g.n_blocks, g.K, G, work, rinv, diag_off, nullptr,
                               shift, nullptr, rinvT, nfail, s);
}

hipError_t launch_bt_bj_factor(const DevBlock* blocks, int blk0, int64_t n_blocks, int kmax,
                               double* G, double* W, const int64_t* goff, const int64_t* foff,
                               double shift, double* rc, int32_t* nfail, hipStream_t s) {
  return factor_by_width<false>(blocks, blk0, n_blocks, kmax, G, W, G, goff, foff, shift, rc,
                                nullptr, nfail, s);
}

}  // namespace elmfb
