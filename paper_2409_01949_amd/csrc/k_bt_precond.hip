// Block-Jacobi preconditioning for batches: per subdomain block b (K_b <= 128 features) the
// diagonal Gram block G_b = M_b^T M_b on the matrix cores, the upper Cholesky factor R_b of
// G_b + lambda_b I (lambda_b = shift trace(G_b)/K_b) and its inverse (column-packed; k_factor.hip),
// then the preconditioned matrix M_b R_b^{-1} formed once on the matrix cores, so that preconditioned
// Krylov steps cost the same as plain ones.  Same preconditioner as for single problems (the
// random features of one subdomain are the main source of the condition numbers of M, Sec. 5),
// with the ragged K of the instances.
#include "device.h"
#include "envelope.h"
#include "gram_core.h"
#include "kernels.h"

namespace elmfb {

typedef double d4_t __attribute__((ext_vector_type(4)));

// One square of G_b (a GramTask: rows i0.., columns j0.., at most 128 each; on the diagonal the
// tiles I <= J), FP64, over all points of the block (gram_product).  8,192 blocks of K = 64 to 128
// 1,944 -> 955 us, patches of up to 512 columns (16 instances) 1,741 -> 958 us, against tiles dealt
// with a search per product and stages of 32 points without prefetch.  On the diagonal a block
// takes the square of 32, 64 or 128 columns that holds it, WT being that of the batch's widest (the
// staging of 128 rows was the time of narrow blocks: 16 of K = 33 and one of K = 4 on 1,600 points 205
// us a precondition call, 120 so).
template <int WT>
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
  R.len = max(1, B.n);   // a block without points: one load, masked by v1 = 0
  R.v0 = 0;
  R.v1 = B.n;
  double* out = G + goff[T.blk] + (int64_t)T.i0 * K + T.j0;
  auto put = [&](int r, int c, double v) { out[r * K + c] = v; };
  if (T.i0 == T.j0) {
    if (WT == 1 || R.nx <= 32) gram_product<ELMFB_FP64, 1, GRAM_UPPER>(R, gd_lds, put);
    else if (WT == 2 || R.nx <= 64) gram_product<ELMFB_FP64, 2, GRAM_UPPER>(R, gd_lds, put);
    else if constexpr (WT == 4) gram_product<ELMFB_FP64, 4, GRAM_UPPER>(R, gd_lds, put);
  } else if constexpr (WT == 4) {
    gram_product<ELMFB_FP64, 4, GRAM_SQUARE>(R, gd_lds, put);
  }
}

// Fold the preconditioner into the matrix: Mhat_b = M_b R_b^{-1}, i.e. in the feature-major
// block layout Mhat_b[k'][p] = sum_{k <= k'} Ri[k][k'] M_b[k][p] (R^{-T} times the block), on
// v_mfma_f64_16x16x4_f64 (K <= 512), in tiles of 16 features k' x 16 points; tiles entirely above
// the diagonal are skipped.  The FP64 result goes to Mhat (if not NULL) and, rounded to nearest
// even, to the low-precision copy.  Every wavefront (k_bt_fold) or workgroup (k_bt_fold_wide) reads
// all K rows of its points before it writes any, so Mhat may be A itself (the patch blocks).
//
// Two 16-point tiles share a load: tile 2h + e has the points 32h + 2i + e (i = 0..15), so lanes
// load and store pairs of points, 16 bytes in FP64 and 256 contiguous bytes over 16 lanes.
constexpr int kFoldTile = 16 * 17;   // a staged 16 x 16 tile of R^{-1}, rows padded

typedef double d2_t __attribute__((ext_vector_type(2)));

// Element (k, kp) of R_b^{-1}, zero below the diagonal and outside: FULL, stored K x K row-major
// per block (single problems), else column-packed.
template <bool FULL>
__device__ __forceinline__ double fold_r(const double* __restrict__ Rb, int K, int k, int kp) {
  const int i = FULL ? k * K + kp : kp * (kp + 1) / 2 + k;
  return kp < K && k <= kp ? Rb[i] : 0.0;
}

// The 16-feature tile I (rows 16 I + lq + 4 v of lane column li) of the points p + 32h + 2 li + e.
template <int LO, int NB>
__device__ __forceinline__ void fold_store(const DevBlock& B, int p, int I, int li, int lq,
                                           const d4_t (&acc)[NB], double* Ahat, void* Ahat_lo) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int kp = 16 * I + lq + 4 * v;
    if (kp >= B.nk) continue;
#pragma unroll
    for (int h = 0; h < NB / 2; ++h) {
      const int q = p + 32 * h + 2 * li;
      if (q >= B.n) continue;
      const int64_t o = B.a_off + (int64_t)kp * B.ld + q;
      const double x = acc[2 * h][v], y = acc[2 * h + 1][v];
      if (q + 1 < B.n) {
        if (Ahat) __builtin_nontemporal_store(d2_t{x, y}, reinterpret_cast<d2_t*>(Ahat + o));
        if constexpr (LO == ELMFB_FP32)
          *reinterpret_cast<float2*>(static_cast<float*>(Ahat_lo) + o) =
              make_float2((float)x, (float)y);
        if constexpr (LO == ELMFB_BF16 || LO == ELMFB_FP16)
          *reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(Ahat_lo) + o) =
              entry16<LO>(x) | (uint32_t)entry16<LO>(y) << 16;
      } else {
        if (Ahat) Ahat[o] = x;
        if constexpr (LO > ELMFB_FP64) store_entry<LO>(Ahat_lo, o, x);
      }
    }
  }
}

// Up to 16 NT <= 128 columns.  R_b^{-1} (its upper tiles) is staged in LDS once per run of points;
// each wavefront then takes 16 NB points at a time with all their features, loading the rows of M
// straight into the matrix cores' operand layout, one tile of 16 rows ahead.  Bound by HBM (M read,
// FP64 and rounded copy written): the 3-level problem (K = 96, FP16 copy) 2,400 -> 1,090 us, 4.2
// TB/s; 8,192 blocks of 64 to 128 columns (FP32 copy; 250 points each, so that staging R^{-1} and
// the first loads weigh) 2,190 -> 1,700 us, 2.8 TB/s, against features split over the wavefronts
// (K = 96 keeps half of them idle), both operands through one LDS buffer, and the 16-bit rounding
// by integers.  J stays a loop: unrolled, the addresses of all tiles take 400 registers.
template <int LO, bool FULL, int NT>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(2))) k_bt_fold(const DevBlock* __restrict__ blocks,
                                                 const Tile* __restrict__ ftiles, int run,
                                                 const double* A, const double* __restrict__ rc,
                                                 const int64_t* __restrict__ foff, double* Ahat,
                                                 void* __restrict__ Ahat_lo) {
  constexpr int NB = NT > 4 ? 2 : 4;
  extern __shared__ double fold_lds[];
  const Tile t = ftiles[blockIdx.x];
  if (t.blk < 0) return;                          // an empty run (launch order padding)
  const DevBlock B = blocks[t.blk];
  const int K = B.nk, nT = (K + 15) >> 4;
  const double* Rb = FULL ? rc + (int64_t)t.blk * K * K : rc + foff[t.blk];
  {
    // element (r, c) of each tile: the factor's fast direction across the threads
    const int r = FULL ? threadIdx.x >> 4 : threadIdx.x & 15;
    const int c = FULL ? threadIdx.x & 15 : threadIdx.x >> 4;
    int I = 0, J = 0;                             // tile (J, I), J <= I, number I (I + 1) / 2 + J
    for (int s = 0; s < nT * (nT + 1) / 2; s += 12) {
      double x[12];
#pragma unroll
      for (int u = 0; u < 12; ++u) {
        x[u] = fold_r<FULL>(Rb, K, 16 * J + r, 16 * I + c);   // zero past the last tile
        if (++J > I) { ++I; J = 0; }
      }
#pragma unroll
      for (int u = 0; u < 12; ++u)
        if (s + u < nT * (nT + 1) / 2) fold_lds[(s + u) * kFoldTile + r * 17 + c] = x[u];
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lq = lane >> 4;
  const double* Ab = A + B.a_off;
  const int end = min(t.p0 + run, B.n);
  auto load = [&](int p, int J, d2_t (&m)[4][NB / 2]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = 16 * J + 4 * q + lq;
      const double* row = Ab + (int64_t)min(k, K - 1) * B.ld;
#pragma unroll
      for (int h = 0; h < NB / 2; ++h) {
        const int c = p + 32 * h + 2 * li;        // pairs past the row: its first (not stored)
        m[q][h] = *reinterpret_cast<const d2_t*>(row + (c < B.ld ? c : 0));
        if (k >= K) m[q][h] = d2_t{0.0, 0.0};
      }
    }
  };
  int p = t.p0 + wid * 16 * NB;
  if (p >= end) return;                           // no barrier follows
  d2_t cur[4][NB / 2];
  load(p, 0, cur);
  while (true) {
    const int pn = p + 64 * NB;
    d4_t acc[NT][NB];
#pragma unroll
    for (int I = 0; I < NT; ++I)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[I][b] = d4_t{0, 0, 0, 0};
#pragma unroll 1
    for (int J = 0; J < nT; ++J) {
      d2_t nxt[4][NB / 2];
      if (J + 1 < nT) load(p, J + 1, nxt);
      else if (pn < end) load(pn, 0, nxt);
#pragma unroll
      for (int I = 0; I < NT; ++I) {
        if (I >= J && I < nT) {
          const double* R = fold_lds + (I * (I + 1) / 2 + J) * kFoldTile + lq * 17 + li;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const double r = R[4 * q * 17];
#pragma unroll
            for (int b = 0; b < NB; ++b)
              acc[I][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(r, cur[q][b >> 1][b & 1], acc[I][b], 0,
                                                               0, 0);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int h = 0; h < NB / 2; ++h) cur[q][h] = nxt[q][h];
    }
#pragma unroll
    for (int I = 0; I < NT; ++I)
      if (I < nT) fold_store<LO, NB>(B, p, I, li, lq, acc[I], Ahat, Ahat_lo);
    if (pn >= end) return;
    p = pn;
  }
}

// Up to 128 TPW columns (a patch's, or a single problem's wide block): 64 points per workgroup of 8
// wavefronts, which own the feature tiles w, w + 8, ...; the contraction runs in stages of 16 rows
// of M and of R^{-1} in two LDS buffers, the next stage's loads in flight during the products.  At
// 512 columns the stages' products and the latency of their loads are the bound (16 instances,
// patches of 2 x 2 subdomains of 64 to 128 columns, about 30 GFLOP): 3,110 -> 1,440 us.
template <int LO, bool FULL, int TPW>
__global__ void __launch_bounds__(512) k_bt_fold_wide(const DevBlock* __restrict__ blocks,
                                                      const Tile* __restrict__ ftiles,
                                                      const double* A,
                                                      const double* __restrict__ rc,
                                                      const int64_t* __restrict__ foff,
                                                      double* Ahat, void* __restrict__ Ahat_lo) {
  constexpr int KMAX = 128 * TPW, NR = KMAX * 16 / 512;
  constexpr int kRows = KMAX / 16 * kFoldTile;    // one stage of R^{-1}
  extern __shared__ double fold_lds[];
  double* const Rt = fold_lds;                    // [2][KMAX / 16 tiles]
  double* const At = fold_lds + 2 * kRows;        // [2][16][64]
  const Tile t = ftiles[blockIdx.x];
  if (t.blk < 0) return;
  const DevBlock B = blocks[t.blk];
  const int K = B.nk, nT = (K + 15) >> 4, p = t.p0;
  const double* Ab = A + B.a_off;
  const double* Rb = FULL ? rc + (int64_t)t.blk * K * K : rc + foff[t.blk];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lq = lane >> 4;
  // this thread's elements of a stage
  const int ar = tid >> 5, ac = 2 * (tid & 31);
  const int acl = p + ac < B.ld ? p + ac : 0;     // pairs past the row: its first (not stored)
  double rr[NR];
  d2_t mm;
  auto load = [&](int J) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int e = tid + 512 * i;
      const int kk = FULL ? e / KMAX : e & 15, kp = FULL ? e % KMAX : e >> 4;
      rr[i] = fold_r<FULL>(Rb, K, 16 * J + kk, kp);
    }
    const int k = 16 * J + ar;
    mm = *reinterpret_cast<const d2_t*>(Ab + (int64_t)min(k, K - 1) * B.ld + acl);
    if (k >= K) mm = d2_t{0.0, 0.0};
  };
  auto put = [&](int s) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int e = tid + 512 * i;
      const int kk = FULL ? e / KMAX : e & 15, kp = FULL ? e % KMAX : e >> 4;
      Rt[s * kRows + (kp >> 4) * kFoldTile + kk * 17 + (kp & 15)] = rr[i];
    }
    *reinterpret_cast<d2_t*>(At + s * 1024 + ar * 64 + ac) = mm;
  };
  d4_t acc[TPW][4];
#pragma unroll
  for (int a = 0; a < TPW; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = d4_t{0, 0, 0, 0};
  load(0);
  put(0);
  __syncthreads();
  for (int J = 0; J < nT; ++J) {
    const int s = J & 1;
    if (J + 1 < nT) load(J + 1);
    d2_t m[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        m[q][h] = *reinterpret_cast<const d2_t*>(At + s * 1024 + (4 * q + lq) * 64 + 32 * h + 2 * li);
#pragma unroll
    for (int a = 0; a < TPW; ++a) {
      const int I = wid + 8 * a;
      if (I >= J && I < nT) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double r = Rt[s * kRows + I * kFoldTile + (4 * q + lq) * 17 + li];
#pragma unroll
          for (int b = 0; b < 4; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(r, m[q][b >> 1][b & 1], acc[a][b], 0, 0,
                                                             0);
        }
      }
    }
    if (J + 1 < nT) put(s ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < TPW; ++a)
    if (wid + 8 * a < nT) fold_store<LO, 4>(B, p, wid + 8 * a, li, lq, acc[a], Ahat, Ahat_lo);
}

// Points per run of the fold for blocks of up to kmax columns: one pass of the wide kernel; else
// four wavefronts' passes of 64 points, or two of 32 above 64 columns.  512 points, which stage
// R^{-1} half as often, measured the same on large problems (1,074 against 1,090 us) and worse on
// 81 blocks of K = 48 (69 against 63 us), whose workgroups then leave CUs idle.
int fold_run_points(int kmax) { return kmax > 128 ? 64 : 256; }

template <typename F, typename... Args>
static hipError_t fold_launch(F kernel, size_t lds, int threads, int64_t n, hipStream_t s,
                              Args... args) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(threads), lds, s, args...);
  return hipGetLastError();
}

template <int LO, bool FULL>
static hipError_t fold_columns(int kmax, const DevBlock* blocks, const Tile* ftiles,
                               int64_t n_ftiles, const double* A, const double* rc,
                               const int64_t* foff, double* Ahat, void* Ahat_lo, hipStream_t s) {
  const int nT = (kmax + 15) / 16, run = fold_run_points(kmax);
  const size_t lds = (size_t)nT * (nT + 1) / 2 * kFoldTile * 8;
  const auto wide = [](int tpw) { return (size_t)(2 * 8 * tpw * kFoldTile + 2 * 1024) * 8; };
  if (kmax > 256)
    return fold_launch(k_bt_fold_wide<LO, FULL, 4>, wide(4), 512, n_ftiles, s, blocks, ftiles, A, rc,
                       foff, Ahat, Ahat_lo);
  if (kmax > 128)
    return fold_launch(k_bt_fold_wide<LO, FULL, 2>, wide(2), 512, n_ftiles, s, blocks, ftiles, A, rc,
                       foff, Ahat, Ahat_lo);
  if (kmax > 64)
    return fold_launch(k_bt_fold<LO, FULL, 8>, lds, 256, n_ftiles, s, blocks, ftiles, run, A, rc,
                       foff, Ahat, Ahat_lo);
  if (kmax > 32)
    return fold_launch(k_bt_fold<LO, FULL, 4>, lds, 256, n_ftiles, s, blocks, ftiles, run, A, rc,
                       foff, Ahat, Ahat_lo);
  return fold_launch(k_bt_fold<LO, FULL, 2>, lds, 256, n_ftiles, s, blocks, ftiles, run, A, rc, foff,
                     Ahat, Ahat_lo);
}

hipError_t launch_bt_fold(int lo_prec, bool full, int kmax, const DevBlock* blocks,
                          const Tile* ftiles, int64_t n_ftiles, const double* A, const double* rc,
                          const int64_t* foff, double* Ahat, void* Ahat_lo, hipStream_t s) {
  if (n_ftiles == 0) return hipSuccess;
  if (kmax > kPatchMaxK || (full && kmax > 256)) return hipErrorInvalidValue;
#define FOLD(L)                                                                                   \
  return full ? fold_columns<L, true>(kmax, blocks, ftiles, n_ftiles, A, rc, foff, Ahat, Ahat_lo,  \
                                      s)                                                          \
              : fold_columns<L, false>(kmax, blocks, ftiles, n_ftiles, A, rc, foff, Ahat, Ahat_lo, \
                                       s)
  if (lo_prec == ELMFB_FP32) FOLD(ELMFB_FP32);
  if (lo_prec == ELMFB_BF16) FOLD(ELMFB_BF16);
  if (lo_prec == ELMFB_FP16) FOLD(ELMFB_FP16);
  FOLD(-1);
#undef FOLD
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
                               int kmax, const double* A, const int64_t* goff, double* G,
                               hipStream_t s) {
  if (n_tasks == 0) return hipSuccess;
  const int wt = kmax > 64 ? 4 : kmax > 32 ? 2 : 1;
  // above 128 columns also squares off the diagonal, which stage two operands
  const size_t lds = (size_t)(kmax > kBatchMaxK ? 2 : 1) * 32 * wt * kGrStride * sizeof(gr_vec);
#define GRAM_DIAG(W)                                                                              \
  hipLaunchKernelGGL(k_bt_gram_diag<W>, dim3((unsigned)n_tasks), dim3(256), lds, s, blocks, tasks, \
                     A, goff, G)
  if (wt == 4) GRAM_DIAG(4); else if (wt == 2) GRAM_DIAG(2); else GRAM_DIAG(1);
#undef GRAM_DIAG
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
