// Gram blocks of the normal equations, G_ij = M_i^T M_j summed over the grid points the two
// supports share (the block decomposition of Sec. 3, eq. multilevel_domain_decomp, gives
// M^T M = sum_ij W_i^T M_i^T V_i V_j^T M_j W_j, nonzero only where I_i and I_j intersect).
//
// Each overlapping pair (i <= j) has a rectangular shared box, whose grid rows are runs of
// consecutive points of both blocks; its loads are split into chunks.  One workgroup per
// (chunk, square of 32 WT x 32 WT outputs) runs gram_product on the stored precision: FP64
// v_mfma_f64_16x16x4_f64, FP32 v_mfma_f32_16x16x4_f32, 16-bit v_mfma_f32_16x16x32 with FP32
// accumulation.  A diagonal block computes the upper tiles and writes their mirror images (the
// same products in the same order).  A pair with one chunk writes its block directly; a pair with
// several chunks writes chunk partials that a second kernel sums in chunk order (deterministic,
// no atomics).
#include "device.h"
#include "gram_core.h"
#include "kernels.h"

namespace elmfb {

// Bound: FP64 by the matrix cores, 16-bit by the caches (a pair reads 2 K S entries for 2 K^2 S
// flops): the host orders the chunks so that the pairs of one second block, the finer of two
// levels, follow each other on one XCD's L2 (by first block FP16 took 1.88 ms: 13 GB past the L2s
// instead of 10.6; 8 or 40 groups an XCD instead of 16 1.62 and 1.61).  Staged before with one entry
// per load, every feature row by every group of output tiles, chunks of 4,096 points whatever their
// number; computations with their chunk sums, before -> now:
//   3-level problem, 5,361 pairs of K = 96: FP64 9.6 -> 8.8 ms (46 TFLOP/s), FP32 5.9 -> 4.6,
//     FP16 3.3 -> 1.57 ms (255 TFLOP/s); its diagonal blocks 1,522 -> 725, 964 -> 424, 557 -> 201 us
//   11 blocks of K = 256: 1,957 -> 440, 1,642 -> 254, 1,167 -> 82 us
//   256 blocks of K = 16: 50 -> 18, 34 -> 13, 31 -> 10 us
// (16 loads a row and stage instead of 8 take the registers of a wavefront a SIMD: FP64 8.7 -> 14 ms;
// one contiguous range of chunks per XCD instead of dealt groups leaves the one with the coarse
// blocks behind: FP16 2.3 -> 3.0 ms.)
template <int PREC, int WT>
__global__ void __launch_bounds__(256) k_gram(Geo g, const DevBlock* __restrict__ blocks,
                                              const GramPair* __restrict__ pairs,
                                              const GramChunk* __restrict__ chunks, int chunk_vecs,
                                              const void* __restrict__ A,
                                              typename GramT<PREC>::out* __restrict__ G,
                                              typename GramT<PREC>::out* __restrict__ part) {
  constexpr int ES = GramT<PREC>::es, VE = sizeof(typename GramLoad<PREC, WT>::t) / ES, M = 32 * WT;
  extern __shared__ gr_vec lds[];              // 2 x M rows
  const int K = g.K;
  const int nsq = (K + M - 1) / M;
  const int i0 = (int)blockIdx.y / nsq * M, j0 = (int)blockIdx.y % nsq * M;
  const GramChunk ck = chunks[blockIdx.x];
  if (ck.pair < 0) return;
  const GramPair pr = pairs[ck.pair];
  const bool diag = pr.bi == pr.bj;
  if (diag && i0 > j0) return;                 // the mirror image of square (j0, i0)
  const DevBlock Bi = blocks[pr.bi], Bj = blocks[pr.bj];
  GramRun R;
  const int64_t pi = (int64_t)(pr.ix0 - Bi.ix0) * Bi.ny + (pr.iy0 - Bi.iy0);
  const int64_t pj = (int64_t)(pr.ix0 - Bj.ix0) * Bj.ny + (pr.iy0 - Bj.iy0);
  R.ldx = (int64_t)Bi.ld * ES;
  R.ldy = (int64_t)Bj.ld * ES;
  R.x = static_cast<const char*>(A) + (Bi.a_off + pi) * ES + i0 * R.ldx;
  R.y = static_cast<const char*>(A) + (Bj.a_off + pj) * ES + j0 * R.ldy;
  R.stepx = (int64_t)Bi.ny * ES;
  R.stepy = (int64_t)Bj.ny * ES;
  R.nx = min(M, K - i0);
  R.ny = min(M, K - j0);
  int rows;
  gram_runs(pr, Bi, Bj, &rows, &R.len);
  R.v0 = ck.s0;
  R.v1 = min(ck.s0 + chunk_vecs, rows * ((R.len + VE - 1) / VE));
  typename GramT<PREC>::out* out =
      (pr.nchunks == 1) ? G + pr.g_off : part + (pr.p_off + ck.slot) * K * K;
  if (!diag) {
    auto put = [&](int r, int c, typename GramT<PREC>::out v) { out[(i0 + r) * K + j0 + c] = v; };
    // An odd number of tiles a side (K = 48): the squares of four wavefronts hold 4, 2, 2 and 1 of
    // 9 tiles, dealt they hold 3, 2, 2, 2.  16-bit entries deal up to 64 columns only: beyond, they
    // need the squares' reuse of fragments (a product takes as long as its two LDS reads).
    if ((PREC == ELMFB_FP64 || PREC == ELMFB_FP32 || WT <= 2) && ((K + 15) / 16) % 2 != 0)
      gram_product<PREC, WT, GRAM_DEALT>(R, lds, put);
    else
      gram_product<PREC, WT, GRAM_SQUARE>(R, lds, put);
  } else if (i0 == j0) {
    gram_product<PREC, WT, GRAM_UPPER>(R, lds, [&](int r, int c, typename GramT<PREC>::out v) {
      out[(i0 + r) * K + i0 + c] = v;
      if ((r >> 4) != (c >> 4)) out[(i0 + c) * K + i0 + r] = v;
    });
  } else {
    gram_product<PREC, WT, GRAM_SQUARE>(R, lds, [&](int r, int c, typename GramT<PREC>::out v) {
      out[(i0 + r) * K + j0 + c] = v;
      out[(j0 + c) * K + i0 + r] = v;
    });
  }
}

// Sum the chunk partials of every multi-chunk pair in chunk order.
template <typename acc_t>
__global__ void __launch_bounds__(256) k_gram_reduce(Geo g, const GramPair* __restrict__ pairs,
                                                     const int32_t* __restrict__ multi,
                                                     const acc_t* __restrict__ part,
                                                     acc_t* __restrict__ G) {
  const GramPair pr = pairs[multi[blockIdx.x]];
  const int KK = g.K * g.K;
  for (int e = blockIdx.y * 256 + threadIdx.x; e < KK; e += 256 * gridDim.y) {
    acc_t s = 0;
    for (int c = 0; c < pr.nchunks; ++c) s += part[(int64_t)(pr.p_off + c) * KK + e];
    G[pr.g_off + e] = s;
  }
}

template <int PREC>
static int load_points(int K) {
  const int side = gram_square(K);
  const size_t b = side == 64   ? sizeof(typename GramLoad<PREC, 2>::t)
                   : side == 96 ? sizeof(typename GramLoad<PREC, 3>::t)
                                : sizeof(typename GramLoad<PREC, 1>::t);
  return (int)b / GramT<PREC>::es;
}

int gram_load_points(int prec, int K) {
  return prec == ELMFB_FP64   ? load_points<ELMFB_FP64>(K)
         : prec == ELMFB_FP32 ? load_points<ELMFB_FP32>(K)
         : prec == ELMFB_BF16 ? load_points<ELMFB_BF16>(K)
                              : load_points<ELMFB_FP16>(K);
}

template <int PREC>
static hipError_t gram_launch(const Geo& g, const DevBlock* blocks, const GramPair* pairs,
                              const GramChunk* chunks, int64_t n_chunks, int chunk_vecs,
                              const void* A, void* G, void* part, hipStream_t s) {
  typedef typename GramT<PREC>::out out_t;
  const int wt = gram_square(g.K) / 32, nsq = (g.K + 32 * wt - 1) / (32 * wt);
  const dim3 grid((unsigned)n_chunks, (unsigned)(nsq * nsq));
  const size_t sm = (size_t)2 * 32 * wt * kGrStride * sizeof(gr_vec);
#define GRAM(W)                                                                                  \
  hipLaunchKernelGGL((k_gram<PREC, W>), grid, dim3(256), sm, s, g, blocks, pairs, chunks,        \
                     chunk_vecs, A, (out_t*)G, (out_t*)part)
  if (wt == 1) GRAM(1); else if (wt == 2) GRAM(2); else if (wt == 3) GRAM(3); else GRAM(4);
#undef GRAM
  return hipGetLastError();
}

hipError_t launch_gram(const Geo& g, int prec, const DevBlock* blocks, const GramPair* pairs,
                       const GramChunk* chunks, int64_t n_chunks, int chunk_vecs,
                       const int32_t* multi, int64_t n_multi, const void* A, void* G, void* part,
                       hipStream_t s) {
  if (n_chunks == 0) return hipSuccess;
  hipError_t e;
  if (prec == ELMFB_FP64)
    e = gram_launch<ELMFB_FP64>(g, blocks, pairs, chunks, n_chunks, chunk_vecs, A, G, part, s);
  else if (prec == ELMFB_FP32)
    e = gram_launch<ELMFB_FP32>(g, blocks, pairs, chunks, n_chunks, chunk_vecs, A, G, part, s);
  else if (prec == ELMFB_BF16)
    e = gram_launch<ELMFB_BF16>(g, blocks, pairs, chunks, n_chunks, chunk_vecs, A, G, part, s);
  else
    e = gram_launch<ELMFB_FP16>(g, blocks, pairs, chunks, n_chunks, chunk_vecs, A, G, part, s);
  if (e != hipSuccess || n_multi == 0) return e;
  const dim3 rgrid((unsigned)n_multi, (unsigned)((g.K * g.K + 255) / 256 < 64 ? (g.K * g.K + 255) / 256 : 64));
  if (prec == ELMFB_FP64)
    hipLaunchKernelGGL(k_gram_reduce<double>, rgrid, dim3(256), 0, s, g, pairs, multi,
                       (const double*)part, (double*)G);
  else
    hipLaunchKernelGGL(k_gram_reduce<float>, rgrid, dim3(256), 0, s, g, pairs, multi,
                       (const float*)part, (float*)G);
  return hipGetLastError();
}

// ---- y = G p from the stored upper Gram blocks (the normal-equation operator of CG on G)
//
// G = M^T M is symmetric; only the blocks G_ij (i <= j) are stored.  Pass 1, one workgroup per
// stored block: the row products G_ij p_j (for block-row i) and, off the diagonal, the column
// products G_ij^T p_i (for block-row j), each written as a K-vector of partials.  A group of 16
// lanes owns one row at a time and reads it in 128-byte segments (lane s takes columns
// s, s + 16, ...), so G_ij is read from memory exactly once: each loaded entry feeds the row
// sum (a 16-lane butterfly) and the lane's running column sums, which are added over the 16
// row groups through LDS at the end.  Pass 2 (k_gmv_rows): every output coefficient sums the
// partials that belong to its block-row in a fixed order (a table built on the host), 4 lanes
// per coefficient, and the workgroup adds its share of p . y.  Deterministic; no atomics.
constexpr int kGmvMaxK = 256;
constexpr int kGmvCols = kGmvMaxK / 16;   // columns per lane

template <typename GT>
__global__ void __launch_bounds__(256) k_gmv_pairs(int K, const GramPair* __restrict__ pairs,
                                                   const GT* __restrict__ G,
                                                   const double* __restrict__ p,
                                                   const SolveState* __restrict__ st,
                                                   double* __restrict__ part) {
  __shared__ double pi_s[kGmvMaxK], pj_s[kGmvMaxK];
  __shared__ double csum[16][kGmvMaxK];
  if (st && st->done) return;
  const int pr = blockIdx.x;
  const GramPair P = pairs[pr];
  const int64_t qi = (int64_t)P.bi * K, qj = (int64_t)P.bj * K;
  for (int t = threadIdx.x; t < K; t += 256) {
    pi_s[t] = p[qi + t];
    pj_s[t] = p[qj + t];
  }
  __syncthreads();
  const GT* Gb = G + P.g_off;
  const bool offd = P.bi != P.bj;
  const int r = threadIdx.x >> 4, s = threadIdx.x & 15;
  const int nc = (K - s + 15) >> 4;          // columns s + 16 j < K of this lane
  double pjr[kGmvCols], cs[kGmvCols];
#pragma unroll
  for (int j = 0; j < kGmvCols; ++j) {
    pjr[j] = j < nc ? pj_s[s + 16 * j] : 0.0;
    cs[j] = 0.0;
  }
  for (int k = r; k < K; k += 16) {
    const GT* row = Gb + (int64_t)k * K + s;
    double gv[kGmvCols];
#pragma unroll
    for (int j = 0; j < kGmvCols; ++j) gv[j] = j < nc ? (double)row[16 * j] : 0.0;
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < kGmvCols; ++j) v += gv[j] * pjr[j];
    v += __shfl_xor(v, 8, 16);
    v += __shfl_xor(v, 4, 16);
    v += __shfl_xor(v, 2, 16);
    v += __shfl_xor(v, 1, 16);
    if (s == 0) part[(int64_t)(2 * pr) * K + k] = v;
    const double pk = pi_s[k];
#pragma unroll
    for (int j = 0; j < kGmvCols; ++j) cs[j] += gv[j] * pk;
  }
  if (!offd) return;
#pragma unroll
  for (int j = 0; j < kGmvCols; ++j)
    if (j < nc) csum[r][s + 16 * j] = cs[j];
  __syncthreads();
  for (int t = threadIdx.x; t < K; t += 256) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) v += csum[q][t];
    part[(int64_t)(2 * pr + 1) * K + t] = v;
  }
}

// y[b K + k] = sum over the partials listed for block-row b (row_ptr / idx, in table order),
// 4 lanes per coefficient taking every 4th partial, combined by a fixed butterfly;
// red[workgroup] = its share of p . y.
__global__ void __launch_bounds__(256) k_gmv_rows(int K, int64_t n_phi,
                                                  const int32_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ idx,
                                                  const double* __restrict__ part,
                                                  const double* __restrict__ p,
                                                  double* __restrict__ y,
                                                  const SolveState* __restrict__ st,
                                                  double* __restrict__ red) {
  __shared__ double sh[4];
  if (st && st->done) return;
  const int sub = threadIdx.x & 3;
  double acc = 0.0;
  const int64_t n4 = n_phi * 4;
  for (int64_t t4 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t4 < n4;
       t4 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = t4 >> 2;
    const int b = (int)(t / K), k = (int)(t - (int64_t)b * K);
    const int e1 = row_ptr[b + 1];
    double v = 0.0;
    int e = row_ptr[b] + sub;
    for (; e + 12 < e1; e += 16) {   // 4 partials of this lane in flight
      double tv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) tv[q] = part[(int64_t)idx[e + 4 * q] * K + k];
#pragma unroll
      for (int q = 0; q < 4; ++q) v += tv[q];
    }
    for (; e < e1; e += 4) v += part[(int64_t)idx[e] * K + k];
    v += __shfl_xor(v, 1, 4);
    v += __shfl_xor(v, 2, 4);
    if (sub == 0) {
      y[t] = v;
      acc += p[t] * v;
    }
  }
  const double sum = block_sum256(acc, sh);
  if (threadIdx.x == 0) red[blockIdx.x] = sum;
}

hipError_t launch_gram_mv_pairs_only(const Geo& g, int gram_prec, const GramPair* pairs,
                                     int64_t n_pairs, const void* G, const double* p, double* part,
                                     hipStream_t s) {
  if (g.K > kGmvMaxK) return hipErrorInvalidValue;
  if (n_pairs == 0) return hipSuccess;
  if (gram_prec == ELMFB_FP64)
    hipLaunchKernelGGL(k_gmv_pairs<double>, dim3((unsigned)n_pairs), dim3(256), 0, s, g.K, pairs,
                       (const double*)G, p, nullptr, part);
  else
    hipLaunchKernelGGL(k_gmv_pairs<float>, dim3((unsigned)n_pairs), dim3(256), 0, s, g.K, pairs,
                       (const float*)G, p, nullptr, part);
  return hipGetLastError();
}

hipError_t launch_gram_mv(const Geo& g, int gram_prec, const GramPair* pairs, int64_t n_pairs,
                          const void* G, const int32_t* row_ptr, const int32_t* idx,
                          const double* p, double* part, double* y, const SolveState* st,
                          double* red, int n_wg, hipStream_t s) {
  if (g.K > kGmvMaxK) return hipErrorInvalidValue;
  if (n_pairs > 0) {
    if (gram_prec == ELMFB_FP64)
      hipLaunchKernelGGL(k_gmv_pairs<double>, dim3((unsigned)n_pairs), dim3(256), 0, s, g.K,
                         pairs, (const double*)G, p, st, part);
    else
      hipLaunchKernelGGL(k_gmv_pairs<float>, dim3((unsigned)n_pairs), dim3(256), 0, s, g.K,
                         pairs, (const float*)G, p, st, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_gmv_rows, dim3(n_wg), dim3(256), 0, s, g.K, g.n_phi, row_ptr, idx, part,
                     p, y, st, red);   // n_wg <= kRedBlocks partials
  return hipGetLastError();
}

}  // namespace elmfb
