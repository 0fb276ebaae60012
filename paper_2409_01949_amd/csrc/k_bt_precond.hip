// Block-Jacobi preconditioning for batches: per subdomain block b (K_b <= 128 features) the
// diagonal Gram block G_b = M_b^T M_b on the matrix cores, the upper Cholesky factor R_b of
// G_b + lambda_b I (lambda_b = shift trace(G_b)/K_b) and its inverse (column-packed; k_factor.hip),
// then the preconditioned matrix M_b R_b^{-1} formed once on the matrix cores, so that preconditioned
// Krylov steps cost the same as plain ones.  Same preconditioner as for single problems (the
// random features of one subdomain are the main source of the condition numbers of M, Sec. 5),
// with the ragged K of the instances.
#include "device.h"
#include "gram_core.h"
#include "kernels.h"

namespace elmfb {

typedef double d4_t __attribute__((ext_vector_type(4)));

// One square of G_b (a GramTask: rows i0.., columns j0.., at most 128 each; on the diagonal the
// tiles I <= J), FP64, over all points of the block (gram_product).  8,192 blocks of K = 64 to 128
// 1,944 -> 955 us, patches of up to 512 columns (16 instances) 1,741 -> 958 us, against tiles dealt
// with a search per product and stages of 32 points without prefetch.
__global__ void __launch_bounds__(256) k_bt_gram_diag(const DevBlock* __restrict__ blocks,
                                                      const GramTask* __restrict__ tasks,
                                                      const double* __restrict__ A,
                                                      const int64_t* __restrict__ goff,
                                                      double* __restrict__ G) {
  extern __shared__ gr_vec gd_lds[];
  const GramTask T = tasks[blockIdx.x];
  const DevBlock B = blocks[T.blk];
  const int K = B.nk;
  GramRun R;
  R.ldx = R.ldy = (int64_t)B.ld * 8;
  R.x = reinterpret_cast<const char*>(A + B.a_off) + T.i0 * R.ldx;
  R.y = reinterpret_cast<const char*>(A + B.a_off) + T.j0 * R.ldy;
  R.stepx = R.stepy = 0;
  R.nx = min(kBatchMaxK, K - T.i0);
  R.ny = min(kBatchMaxK, K - T.j0);
  R.len = B.n;
  R.v0 = 0;
  R.v1 = B.n;
  double* out = G + goff[T.blk] + (int64_t)T.i0 * K + T.j0;
  auto put = [&](int r, int c, double v) { out[r * K + c] = v; };
  if (T.i0 == T.j0) gram_product<ELMFB_FP64, 4, GRAM_UPPER>(R, gd_lds, put);
  else gram_product<ELMFB_FP64, 4, GRAM_SQUARE>(R, gd_lds, put);
}

// Fold the preconditioner into the matrix: Mhat_b = M_b R_b^{-1}, i.e. in the feature-major
// block layout Mhat_b[k'][p] = sum_{k <= k'} Ri[k][k'] M_b[k][p] (R^{-T} times the block), on
// v_mfma_f64_16x16x4_f64 (K <= 512).  One workgroup per run of 16 NB points of a block: the four
// waves own output row tiles (16 features each) w, w + 4, ... and the NB 16-point column tiles;
// the contraction over k runs in LDS stages of 16 (R^{-T} columns from the factor, M_b rows), and
// tiles entirely above the diagonal are skipped.  The FP64 result goes to Mhat (if not NULL) and,
// rounded to nearest even, to the low-precision copy.  Each workgroup reads all K rows of its
// points before it writes any, so Mhat may be A itself (the patch blocks fold in place).
constexpr int kFoldK = 16;

template <int LO, bool FULL, int TPW, int NB>
__global__ void __launch_bounds__(256) k_bt_fold(const DevBlock* __restrict__ blocks,
                                                 const Tile* __restrict__ ftiles,
                                                 const double* A,
                                                 const double* __restrict__ rc,
                                                 const int64_t* __restrict__ foff,
                                                 double* Ahat,
                                                 void* __restrict__ Ahat_lo) {
  constexpr int KMAX = 64 * TPW;                  // TPW row tiles of 16 features per wave
  constexpr int NP = 16 * NB;                     // points per run
  __shared__ double Rt[KMAX][kFoldK + 1];         // Rt[k'][kk] = Ri[k0 + kk][k']
  __shared__ double At[kFoldK][NP + 1];           // At[kk][c] = M_b[k0 + kk][p0 + c]
  const Tile t = ftiles[blockIdx.x];
  if (t.blk < 0) return;                          // an empty run (launch order padding)
  const DevBlock B = blocks[t.blk];
  const int K = B.nk;
  const int n = B.n, p0 = t.p0;
  const double* Ab = A + B.a_off;
  // FULL: R^{-1} stored K x K row-major per block (single problems); else column-packed
  const double* Rb = FULL ? rc + (int64_t)t.blk * K * K : rc + foff[t.blk];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int li = lane & 15, lq = lane >> 4;
  const int nT = (K + 15) >> 4;
  d4_t acc[TPW][NB];
#pragma unroll
  for (int a = 0; a < TPW; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = d4_t{0, 0, 0, 0};
  for (int k0 = 0; k0 < K; k0 += kFoldK) {
    for (int e = threadIdx.x; e < KMAX * kFoldK; e += 256) {
      const int kp = e / kFoldK, kk = e - (e / kFoldK) * kFoldK;
      const int k = k0 + kk;
      const int64_t ri = FULL ? (int64_t)k * K + kp : (int64_t)kp * (kp + 1) / 2 + k;
      Rt[kp][kk] = (kp < K && k <= kp) ? Rb[ri] : 0.0;
    }
    for (int e = threadIdx.x; e < kFoldK * NP; e += 256) {
      const int kk = e / NP, c = e - (e / NP) * NP;
      const int k = k0 + kk, p = p0 + c;
      At[kk][c] = (k < K && p < n) ? Ab[(int64_t)k * B.ld + p] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < TPW; ++a) {
      const int I = wid + 4 * a;
      if (I < nT && 16 * I + 15 >= k0) {     // rows k' < k0 of R^{-T} vanish on this stage
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
          for (int q = 0; q < kFoldK; q += 4)
            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(Rt[16 * I + li][q + lq],
                                                             At[q + lq][16 * b + li], acc[a][b],
                                                             0, 0, 0);
        }
      }
    }
    __syncthreads();
  }
  // accumulator of v_mfma_f64_16x16x4_f64: lane holds column li, rows lq + 4 v
#pragma unroll
  for (int a = 0; a < TPW; ++a) {
    const int I = wid + 4 * a;
    if (I >= nT) continue;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int p = p0 + 16 * b + li;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int kp = 16 * I + lq + 4 * v;
        if (kp < K && p < n) {
          const int64_t o = B.a_off + (int64_t)kp * B.ld + p;
          const double val = acc[a][b][v];
          if (Ahat) Ahat[o] = val;
          if constexpr (LO == ELMFB_FP32) static_cast<float*>(Ahat_lo)[o] = (float)val;
          if constexpr (LO == ELMFB_BF16) static_cast<uint16_t*>(Ahat_lo)[o] = f64_to_bf16_rne(val);
          if constexpr (LO == ELMFB_FP16) static_cast<uint16_t*>(Ahat_lo)[o] = f64_to_fp16_rne(val);
        }
      }
    }
  }
}

// Points per run of the fold for blocks of up to kmax columns: 64, or 32 above 256 columns.
int fold_run_points(int kmax) { return kmax > 256 ? 32 : 64; }

hipError_t launch_bt_fold(int lo_prec, bool full, int kmax, const DevBlock* blocks,
                          const Tile* ftiles, int64_t n_ftiles, const double* A, const double* rc,
                          const int64_t* foff, double* Ahat, void* Ahat_lo, hipStream_t s) {
  if (n_ftiles == 0) return hipSuccess;
  if (kmax > kPatchMaxK || (full && kmax > 256)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)n_ftiles), blk(256);
#define FOLD(L, F, T, N)                                                                         \
  hipLaunchKernelGGL((k_bt_fold<L, F, T, N>), grid, blk, 0, s, blocks, ftiles, A, rc, foff, Ahat, \
                     Ahat_lo)
#define FOLD_T(L, F)                                                                             \
  do {                                                                                           \
    if (kmax > 256) FOLD(L, F, 8, 2);                                                            \
    else if (kmax > 128) FOLD(L, F, 4, 4);                                                       \
    else FOLD(L, F, 2, 4);                                                                       \
  } while (0)
  if (lo_prec == ELMFB_FP32) { if (full) FOLD_T(ELMFB_FP32, true); else FOLD_T(ELMFB_FP32, false); }
  else if (lo_prec == ELMFB_BF16) { if (full) FOLD_T(ELMFB_BF16, true); else FOLD_T(ELMFB_BF16, false); }
  else if (lo_prec == ELMFB_FP16) { if (full) FOLD_T(ELMFB_FP16, true); else FOLD_T(ELMFB_FP16, false); }
  else { if (full) FOLD_T(-1, true); else FOLD_T(-1, false); }
#undef FOLD_T
#undef FOLD
  return hipGetLastError();
}

// Patch blocks from the assembled subdomain blocks: column c of patch b is feature c mod K of its
// member c / K (members[moff[b]..], lexicographic in the per-axis indices), on the patch's box,
// zero where the point lies outside the member's box and in the row padding.  One workgroup per
// run of 256 stored points of a patch (runs[].p0 < ld).
__global__ void __launch_bounds__(256) k_bt_expand(const Geo* __restrict__ geos,
                                                   const DevBlock* __restrict__ pblocks,
                                                   const Tile* __restrict__ runs,
                                                   const DevBlock* __restrict__ blocks,
                                                   const int32_t* __restrict__ members,
                                                   const int32_t* __restrict__ moff,
                                                   const double* __restrict__ A,
                                                   double* __restrict__ Ap) {
  const Tile r = runs[blockIdx.x];
  const DevBlock P = pblocks[r.blk];
  const int K = geos[P.inst].K;
  const int p = r.p0 + (int)threadIdx.x;
  if (p >= P.ld) return;
  const bool in = p < P.n;
  const int lx = in ? p / P.ny : 0;
  const int ix = P.ix0 + lx, iy = P.iy0 + (in ? p - lx * P.ny : 0);
  const int nm = P.nk / K;
  for (int m = 0; m < nm; ++m) {
    const DevBlock S = blocks[members[moff[r.blk] + m]];
    const bool inside = in && ix >= S.ix0 && ix < S.ix0 + S.nx && iy >= S.iy0 && iy < S.iy0 + S.ny;
    const int64_t src = inside ? S.a_off + (int64_t)(ix - S.ix0) * S.ny + (iy - S.iy0) : 0;
    double* dst = Ap + P.a_off + (int64_t)m * K * P.ld + p;
    for (int k = 0; k < K; ++k) dst[(int64_t)k * P.ld] = inside ? A[src + (int64_t)k * S.ld] : 0.0;
  }
}

hipError_t launch_bt_gram_diag(const DevBlock* blocks, const GramTask* tasks, int64_t n_tasks,
                               bool two_panels, const double* A, const int64_t* goff, double* G,
                               hipStream_t s) {
  if (n_tasks == 0) return hipSuccess;
  const size_t lds = (size_t)(two_panels ? 2 : 1) * kBatchMaxK * kGrStride * sizeof(gr_vec);
  if (two_panels) {   // 68 KB
    const hipError_t e = hipFuncSetAttribute((const void*)k_bt_gram_diag,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_bt_gram_diag, dim3((unsigned)n_tasks), dim3(256), lds, s, blocks, tasks, A,
                     goff, G);
  return hipGetLastError();
}

hipError_t launch_bt_expand(const Geo* geos, const DevBlock* pblocks, const Tile* runs,
                            int64_t n_runs, const DevBlock* blocks, const int32_t* members,
                            const int32_t* moff, const double* A, double* Ap, hipStream_t s) {
  if (n_runs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bt_expand, dim3((unsigned)n_runs), dim3(256), 0, s, geos, pblocks, runs,
                     blocks, members, moff, A, Ap);
  return hipGetLastError();
}

}  // namespace elmfb
