// Block-sparse products with the assembled matrix M = sum_j V_j^T M_j W_j (Sec. 3
// eq. multilevel_domain_decomp), each block M_j stored feature-major [K][ld_j] (rows padded with
// zeros to a multiple of 8 entries, so vector loads stay aligned).
//
// y = M v runs in two passes that stream the matrix exactly once:
//   1. per block point (consecutive points on consecutive lanes; 16-bit copies take two points
//      per lane in one 4-byte load): t_j[p] = sum_k M_j[k][p] v[q0_j + k] -- the K coefficients
//      of the block are wavefront-uniform, so they come from the scalar cache;
//   2. per row (grid point): y_r = sum over the blocks covering it of t_j[p_j(r)], the covering
//      blocks found arithmetically from per-axis index ranges; no atomics, fixed order.
// x = M^T u also streams the matrix once:
//   1. per chunk of <= 2048 consecutive points of one block (its features split over several
//      workgroups when the chunks are few): each thread holds up to 8 gathered
//      u values (in vector-load groups of 2 or 4 consecutive points for FP32 and 16-bit
//      copies); for every group of 8 features the 256 lanes form their dot products, a
//      transposing butterfly across the wavefront reduces the 8 features at once (10 cross-lane
//      shuffles) and a 4-wave LDS sum gives the chunk partials;
//   2. per column: sum of the chunk partials of its block in chunk order.
// All reductions are deterministic (fixed order, no floating-point atomics).
#include <algorithm>

#include "device.h"
#include "kernels.h"

namespace elmfb {

// PTS consecutive points per thread (one vector load per feature row); a tile of 256 points
// runs on 256 / PTS threads.  Per point the sum order does not depend on PTS.
template <int PREC, int PTS, int AHEAD>
__global__ void __launch_bounds__(256) k_mv_blocks(Geo g, const DevBlock* __restrict__ blocks,
                                                   const Tile* __restrict__ tiles,
                                                   const void* __restrict__ A,
                                                   const double* __restrict__ v,
                                                   const double* __restrict__ vscale,
                                                   double* __restrict__ tpart,
                                                   const SolveState* __restrict__ st) {
  if (st && st->done) return;
  const Tile t = tiles[xcd_tile(blockIdx.x, gridDim.x)];
  const DevBlock B = blocks[t.blk];
  const int p = t.p0 + threadIdx.x * PTS;
  if (p >= B.n) return;
  const double* vb = v + B.q0;
  const int K = g.K;
  const int ld = B.ld;
  const int64_t base = B.a_off + p;
  double acc[4][PTS];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int q = 0; q < PTS; ++q) acc[u][q] = 0.0;
  int k = 0;
  for (; k + AHEAD <= K; k += AHEAD) {
    double a[AHEAD][PTS];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) load_vec<PREC, PTS>(A, base + (int64_t)(k + u) * ld, a[u]);
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
#pragma unroll
      for (int q = 0; q < PTS; ++q) acc[u & 3][q] += a[u][q] * vb[k + u];
  }
  if constexpr (AHEAD > 4) {
    for (; k + 4 <= K; k += 4) {
      double a[4][PTS];
#pragma unroll
      for (int u = 0; u < 4; ++u) load_vec<PREC, PTS>(A, base + (int64_t)(k + u) * ld, a[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < PTS; ++q) acc[u][q] += a[u][q] * vb[k + u];
    }
  }
  for (; k < K; ++k) {
    double a[PTS];
    load_vec<PREC, PTS>(A, base + (int64_t)k * ld, a);
#pragma unroll
    for (int q = 0; q < PTS; ++q) acc[0][q] += a[q] * vb[k];
  }
  const double sc = vscale ? *vscale : 1.0;
#pragma unroll
  for (int q = 0; q < PTS; ++q)
    if (p + q < B.n)
      tpart[B.p_off + p + q] = ((acc[0][q] + acc[1][q]) + (acc[2][q] + acc[3][q])) * sc;
}

// y_b = sum_q bc[b][q] v_q (v scaled by *vscale when given) for the soft-constraint rows, one
// wavefront per row and 4 rows per workgroup, then the row mode at row n_rows + b as
// k_gather_rows applies it; workgroup `wg` writes one partial squared norm to *red (its rows' in
// order).  A wavefront keeps 8 of its n_phi / 64 loads in flight (one at a time, the chain of
// loads was the pass: 320 rows of 3,072 columns 12.7 us).
__device__ __forceinline__ void bc_rows(const Geo& g, int wg, const double* __restrict__ bc,
                                        const double* __restrict__ v,
                                        const double* __restrict__ vscale, int mode,
                                        double* __restrict__ out, const double* __restrict__ bvec,
                                        const SolveState* __restrict__ st,
                                        double* __restrict__ red, double* sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int b = wg * 4 + wid;
  const double sc = vscale ? *vscale : 1.0;
  double acc = 0.0;
  if (b < g.n_bc) {
    const double* row = bc + (int64_t)b * g.n_phi;
    double d = 0.0;
    int64_t q = lane;
    for (; q + 64 * 7 < g.n_phi; q += 64 * 8) {
      double a[8], x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        a[i] = row[q + 64 * i];
        x[i] = v[q + 64 * i];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) d += a[i] * x[i];
    }
    for (; q < g.n_phi; q += 64) d += row[q] * v[q];
    const double y = wave_sum(d) * sc;
    if (lane == 0) {
      const int64_t r = g.n_rows + b;
      if (mode == ROW_STORE) {
        out[r] = y;
      } else if (mode == ROW_LSQR_U) {
        const double u = y - st->alpha * st->su * out[r];
        out[r] = u;
        acc = u * u;
      } else if (mode == ROW_RESID) {
        const double u = bvec[r] - y;
        out[r] = u;
        acc = u * u;
      } else {
        out[r] = y;
        acc = y * y;
      }
    }
  }
  if (lane == 0) sh[wid] = acc;
  __syncthreads();
  if (mode != ROW_STORE && threadIdx.x == 0) *red = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// With BC the workgroups from n_row_wgs on take the soft-constraint rows (bc, vb, vscale); MAPPED:
// an L-shaped domain, which discards subdomains (covering blocks through the block map).
template <bool BC, bool MAPPED>
__global__ void __launch_bounds__(256) k_gather_rows(Geo g, const DevBlock* __restrict__ blocks,
                                                     const int32_t* __restrict__ cov,
                                                     const double* __restrict__ tpart, int mode,
                                                     double* __restrict__ out,
                                                     const double* __restrict__ bvec,
                                                     const SolveState* __restrict__ st,
                                                     double* __restrict__ red, int n_row_wgs,
                                                     const double* __restrict__ bc,
                                                     const double* __restrict__ vb,
                                                     const double* __restrict__ vscale) {
  __shared__ double sh[4];
  if (st && st->done) return;
  if constexpr (BC) {
    if ((int)blockIdx.x >= n_row_wgs) {
      bc_rows(g, (int)blockIdx.x - n_row_wgs, bc, vb, vscale, mode, out, bvec, st,
              red + blockIdx.x, sh);
      return;
    }
  }
  double coef_u = 0.0;
  if (mode == ROW_LSQR_U) coef_u = st->alpha * st->su;
  double acc = 0.0;
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < g.n_rows;
       r += (int64_t)n_row_wgs * blockDim.x) {
    const int ix = (int)(r / g.ny), iy = (int)(r - (int64_t)ix * g.ny);
    double y = 0.0;
    for (int l = 0; l < g.n_levels; ++l) {
      const int jx0 = cov[g.cov_off[l][0] + 2 * ix], jx1 = cov[g.cov_off[l][0] + 2 * ix + 1];
      const int jy0 = cov[g.cov_off[l][1] + 2 * iy], jy1 = cov[g.cov_off[l][1] + 2 * iy + 1];
      const int Jy = g.J[l][1];
      const int ncx = jx1 - jx0 + 1, ncy = jy1 - jy0 + 1;
      if (ncx <= 3 && ncy <= 3) {
        // up to 3 x 3 covering blocks (width ratio < 3): every load issued before the sums,
        // which keep the order jx-major, jy-minor; absent slots read the first block (a
        // discarded one: block 0's first point) and add 0
        int at[9];
        if constexpr (MAPPED) {
#pragma unroll
          for (int q = 0; q < 9; ++q)
            at[q] = g.bmap[g.bmap_off[l] + (jx0 + (q / 3 < ncx ? q / 3 : 0)) * Jy + jy0 +
                           (q % 3 < ncy ? q % 3 : 0)];
        }
        double tv[9];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            bool ok = a < ncx && c < ncy;
            double t;
            if constexpr (MAPPED) {
              const int bi = at[a * 3 + c];
              ok = ok && bi >= 0;
              const DevBlock& B = blocks[ok ? bi : 0];
              t = tpart[B.p_off + (ok ? (ix - B.ix0) * B.ny + (iy - B.iy0) : 0)];
            } else {
              const DevBlock& B = blocks[g.bbase[l] + (jx0 + (ok ? a : 0)) * Jy + jy0 + (ok ? c : 0)];
              t = tpart[B.p_off + (ix - B.ix0) * B.ny + (iy - B.iy0)];
            }
            tv[a * 3 + c] = ok ? t : 0.0;
          }
        }
#pragma unroll
        for (int q = 0; q < 9; ++q) y += tv[q];
      } else {
        for (int jx = jx0; jx <= jx1; ++jx) {
          for (int jy = jy0; jy <= jy1; ++jy) {
            const int bi = MAPPED ? g.bmap[g.bmap_off[l] + jx * Jy + jy] : g.bbase[l] + jx * Jy + jy;
            if (MAPPED && bi < 0) continue;
            const DevBlock& B = blocks[bi];
            const int p = (ix - B.ix0) * B.ny + (iy - B.iy0);
            y += tpart[B.p_off + p];
          }
        }
      }
    }
    if (mode == ROW_STORE) {
      out[r] = y;
    } else if (mode == ROW_LSQR_U) {
      const double u = y - coef_u * out[r];
      out[r] = u;
      acc += u * u;
    } else if (mode == ROW_RESID) {
      const double u = bvec[r] - y;
      out[r] = u;
      acc += u * u;
    } else {
      out[r] = y;
      acc += y * y;
    }
  }
  if (mode != ROW_STORE) {
    const double s = block_sum256(acc, sh);
    if (threadIdx.x == 0) red[blockIdx.x] = s;
  }
}

// The features [k0, k1) of one chunk against the NL live groups of points of each thread (group i
// of thread t: VEC consecutive points from i*256*VEC + t*VEC; the groups past the block's end carry
// zero weights and are left out, which changes no sum).
template <int PREC, int VEC, int NL, int NG>
__device__ __forceinline__ void rmv_features(const void* __restrict__ A, const int64_t (&idx)[NG],
                                             const double (&uv)[NG][VEC], int ld, int K, int k0,
                                             int k1, double (*sred)[264]) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int kb = k0; kb < k1; kb += 8) {
    double acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      acc[j] = 0.0;
      const int k = kb + j < K ? kb + j : K - 1;     // padded features reread the last one
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        double a[VEC];
        load_vec<PREC, VEC>(A, idx[i] + (int64_t)k * ld, a);
#pragma unroll
        for (int q = 0; q < VEC; ++q) acc[j] += a[q] * uv[i][q];
      }
    }
    int f;
    const double v = butterfly8(acc, lane, &f);
    if ((lane & 7) == 0) sred[wid][kb - k0 + f] = v;
  }
}

// VEC consecutive points per vector load; each thread holds NG groups of them, the groups of a
// chunk interleaved across the workgroup.  blockIdx.y takes `kper` features (a multiple of 8) of
// the chunk.  FEW: also loops over only the live groups (blocks that fill part of their chunk);
// their extra copies of the loop take 96 instead of 60 registers in FP64, which a grid that fills
// the chip pays for (345 against 341 us on the 3-level problem), so it keeps the one loop.
// With red, u is LSQR's new u = A v - alpha u, of which red holds the n_red partial squared norms:
// every workgroup sums them (in one order) to beta = ||u|| and scales u by 1/beta as it reads, and
// the first one records beta, su = 1/beta, anorm = sqrt(anorm^2 + alpha^2 + beta^2) and hist (may
// be NULL: beta_{i+1} of step i = itn + 1).  The sums' latency is hidden behind the loads of u;
// a kernel of its own for beta was about 4.7 us of every step, whatever the problem's size.
template <int PREC, int VEC, bool FEW>
__global__ void __launch_bounds__(256) k_rmv_chunks(Geo g, const DevBlock* __restrict__ blocks,
                                                    const Tile* __restrict__ chunks,
                                                    const void* __restrict__ A,
                                                    const double* __restrict__ u,
                                                    const double* __restrict__ uscale,
                                                    double* __restrict__ part, int kper,
                                                    SolveState* st,
                                                    const double* __restrict__ red, int n_red,
                                                    double* hist) {
  constexpr int NG = kChunkPts / (256 * VEC);
  static_assert(NG * 256 * VEC == kChunkPts, "chunk size");
  __shared__ double sred[4][264];
  if (st && st->done) return;
  const int ci = xcd_tile(blockIdx.x, gridDim.x);
  const Tile c = chunks[ci];
  const DevBlock B = blocks[c.blk];
  const int K = g.K;
  const int live = (min(B.n - c.p0, kChunkPts) + 256 * VEC - 1) / (256 * VEC);
  double uv[NG][VEC];
  int64_t idx[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int p0 = c.p0 + i * 256 * VEC + threadIdx.x * VEC;
    // a group past the block reads the block's first entries with zero weights (in bounds);
    // a group that straddles the end reads padding (zeros, p0 + VEC <= ld) with zero weights
    idx[i] = B.a_off + (p0 < B.n ? p0 : 0);
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
      const int p = p0 + q;
      if (p < B.n) {
        const int lx = p / B.ny, ly = p - lx * B.ny;
        const int64_t r = (int64_t)(B.ix0 + lx) * g.ny + (B.iy0 + ly);
        uv[i][q] = u[r];
      } else {
        uv[i][q] = 0.0;
      }
    }
  }
  double sc = uscale ? *uscale : 1.0;
  if (red) {
    const double beta = sqrt(reduce_partials_all(red, n_red, &sred[0][0]));
    sc = beta > 0.0 ? 1.0 / beta : st->su;   // beta = 0: su and anorm stay as they are
    __syncthreads();                         // sred is used again below
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
      const int step = st->itn + 1;
      if (hist && step < kHistCap) hist[2 * step + 1] = beta;
      st->beta = beta;
      if (beta > 0.0) {
        st->su = sc;
        const double a = st->alpha;
        st->anorm = sqrt(st->anorm * st->anorm + a * a + beta * beta);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NG; ++i)
#pragma unroll
    for (int q = 0; q < VEC; ++q) uv[i][q] *= sc;
  const int k0 = blockIdx.y * kper, k1 = min(k0 + kper, K);
  if constexpr (!FEW) rmv_features<PREC, VEC, NG>(A, idx, uv, B.ld, K, k0, k1, sred);
  else if (live <= NG / 8) rmv_features<PREC, VEC, (NG + 7) / 8>(A, idx, uv, B.ld, K, k0, k1, sred);
  else if (live <= NG / 4) rmv_features<PREC, VEC, (NG + 3) / 4>(A, idx, uv, B.ld, K, k0, k1, sred);
  else if (live <= NG / 2) rmv_features<PREC, VEC, NG / 2>(A, idx, uv, B.ld, K, k0, k1, sred);
  else rmv_features<PREC, VEC, NG>(A, idx, uv, B.ld, K, k0, k1, sred);
  __syncthreads();
  for (int k = k0 + threadIdx.x; k < k1; k += 256) {
    const int f = k - k0;
    part[(int64_t)ci * K + k] = (sred[0][f] + sred[1][f]) + (sred[2][f] + sred[3][f]);
  }
}

// bc (may be NULL): the dense soft-constraint rows [n_bc][n_phi]; their part of column q,
// sum_b bc[b][q] u[n_rows + b] (u scaled by *uscale when given), is added after the chunk
// partials.
__global__ void __launch_bounds__(256) k_rmv_finish(Geo g, const int32_t* __restrict__ cstart,
                                                    const double* __restrict__ part, int mode,
                                                    double* __restrict__ out,
                                                    const SolveState* __restrict__ st,
                                                    double* __restrict__ red,
                                                    const double* __restrict__ bc,
                                                    const double* __restrict__ u,
                                                    const double* __restrict__ uscale) {
  __shared__ double sh[4];
  if (st && st->done) return;
  const int K = g.K;
  double coef_v = 0.0;
  bool keep = false;
  if (mode == COL_LSQR_V) {
    coef_v = st->beta * st->sv;
    keep = !(st->beta > 0.0);   // beta == 0: v and alpha stay as they are
  }
  double acc = 0.0;
  for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < g.n_phi;
       q += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(q / K), k = (int)(q - (int64_t)b * K);
    double x = 0.0;
    int c = cstart[b];
    const int ce = cstart[b + 1];
    for (; c + 8 <= ce; c += 8) {   // 8 partials in flight, summed in chunk order
      double t[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) t[q] = part[(int64_t)(c + q) * K + k];
#pragma unroll
      for (int q = 0; q < 8; ++q) x += t[q];
    }
    for (; c < ce; ++c) x += part[(int64_t)c * K + k];
    if (bc) {   // fewer than kSplitBc rows
      const double usc = uscale ? *uscale : 1.0;
      for (int r = 0; r < g.n_bc; ++r) x += bc[(int64_t)r * g.n_phi + q] * (u[g.n_rows + r] * usc);
    }
    if (mode == COL_STORE) {
      out[q] = x;
    } else if (mode == COL_LSQR_V) {
      double v = out[q];
      if (!keep) {
        v = x - coef_v * v;
        out[q] = v;
      }
      acc += v * v;
    } else {
      out[q] = x;
      acc += x * x;
    }
  }
  if (mode != COL_STORE) {
    const double s = block_sum256(acc, sh);
    if (threadIdx.x == 0) red[blockIdx.x] = s;
  }
}

// The same with many soft-constraint rows: a workgroup of 16 wavefronts takes 64 columns, each
// wavefront every 16th row with up to 8 loads in flight, and the first one adds the 16 sums to
// the chunk partials.  n_wg workgroups stride over the columns.  One thread per column summing
// the rows in turn was a chain of n_bc loads: 320 rows of 3,072 columns 41.6 us a
// pass, now 6.9 (the row pass with them in it 21.4 -> 7.8 us, one launch less).
constexpr int kBcSlices = 16;
__global__ void __launch_bounds__(64 * kBcSlices) k_rmv_finish_bc(
    Geo g, const int32_t* __restrict__ cstart, const double* __restrict__ part, int mode,
    double* __restrict__ out, const SolveState* __restrict__ st, double* __restrict__ red,
    const double* __restrict__ bc, const double* __restrict__ u,
    const double* __restrict__ uscale) {
  __shared__ double sums[kBcSlices][64];
  if (st && st->done) return;
  const int K = g.K;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double usc = uscale ? *uscale : 1.0;
  const double* ub = u + g.n_rows;
  double coef_v = 0.0;
  bool keep = false;
  if (mode == COL_LSQR_V) {
    coef_v = st->beta * st->sv;
    keep = !(st->beta > 0.0);
  }
  double acc = 0.0;
  for (int64_t q0 = (int64_t)blockIdx.x * 64; q0 < g.n_phi; q0 += (int64_t)gridDim.x * 64) {
    const int64_t q = q0 + lane;
    const bool live = q < g.n_phi;
    const double* col = bc + (live ? q : q0);
    double d = 0.0;
    int r = wid;
    for (; r + 7 * kBcSlices < g.n_bc; r += 8 * kBcSlices) {
      double t[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) t[i] = col[(int64_t)(r + i * kBcSlices) * g.n_phi];
#pragma unroll
      for (int i = 0; i < 8; ++i) d += t[i] * (ub[r + i * kBcSlices] * usc);
    }
    for (; r < g.n_bc; r += kBcSlices) d += col[(int64_t)r * g.n_phi] * (ub[r] * usc);
    sums[wid][lane] = d;
    __syncthreads();
    if (wid == 0 && live) {
      const int b = (int)(q / K), k = (int)(q - (int64_t)b * K);
      double x = 0.0;
      for (int c = cstart[b]; c < cstart[b + 1]; ++c) x += part[(int64_t)c * K + k];
      double y = 0.0;
#pragma unroll
      for (int i = 0; i < kBcSlices; ++i) y += sums[i][lane];
      x += y;
      if (mode == COL_STORE) {
        out[q] = x;
      } else if (mode == COL_LSQR_V) {
        double v = out[q];
        if (!keep) {
          v = x - coef_v * v;
          out[q] = v;
        }
        acc += v * v;
      } else {
        out[q] = x;
        acc += x * x;
      }
    }
    __syncthreads();
  }
  if (mode != COL_STORE && wid == 0) {
    const double s = wave_sum(acc);
    if (lane == 0) red[blockIdx.x] = s;
  }
}

// Soft-constraint rows from which their sums are split over wavefronts: below, one thread per
// column adds them in turn (a boundary value problem's one or two rows; every sum as before).
constexpr int kSplitBc = 16;

int rows_wg(const Geo& g) {
  int64_t nb = (g.n_rows + 255) / 256;
  return (int)(nb < kRedBlocks ? nb : kRedBlocks);
}
int bc_row_wgs(const Geo& g) { return (g.n_bc + 3) / 4; }
int cols_wg(const Geo& g) {
  const int per = g.n_bc >= kSplitBc ? 64 : 256;
  int64_t nb = (g.n_phi + per - 1) / per;
  return (int)(nb < kRedBlocks ? nb : kRedBlocks);
}

// Points per thread of the y = M v pass and points per vector load of the M^T u pass, per
// stored precision (16-bit rows are read 4 or 8 bytes per lane).
template <int PREC> struct MvShape { static constexpr int pts = 1, vec = 1; };
template <> struct MvShape<ELMFB_FP32> { static constexpr int pts = 1, vec = 2; };
template <> struct MvShape<ELMFB_BF16> { static constexpr int pts = 2, vec = 4; };
template <> struct MvShape<ELMFB_FP16> { static constexpr int pts = 2, vec = 4; };

// Feature rows loaded ahead in M v: up to 2,048 tiles (8 workgroups per CU) the pass has too few
// wavefronts in flight to hide the load latency and takes 16 rows ahead; above, 4 (8 or 16 rows
// cost occupancy there: 95 against 104 us on the 3-level problem's FP16 copy).  Measured, FP64,
// 4 -> 16 rows: 11 blocks of K = 256 23.9 -> 13.1 us, 20 blocks of K = 64 4.3 -> 3.9, 81 blocks
// of K = 48 (1,398 tiles) 21.9 -> 20.5; the sum order, and so every bit, is the same.
constexpr int kFewTiles = 2048;
// Workgroups M^T u aims at: a problem of a few blocks has a few chunks, each of which would
// stream all K features through one workgroup (the serial chain of K/8 feature groups is then
// the time), so the features of a chunk are split over workgroups until about 4 per CU are in
// flight.  Measured, FP64, with the live-group loops: 11 blocks of K = 256 266.6 -> 12.5 us,
// 20 blocks of K = 64 25.5 -> 3.2 us, 81 blocks of K = 48 55.8 -> 24.2 us; the 1,322 chunks of
// the 3-level problem keep one workgroup per chunk (341 us, 5.7 TB/s).  Every bit is the same.
constexpr int kChunkWgs = 1024;

template <int PREC>
static void mv_launch(const Geo& g, const DevBlock* blocks, const Tile* tiles, int64_t n_tiles,
                      const void* A, const double* v, const double* vscale, double* tpart,
                      const SolveState* st, hipStream_t s) {
  constexpr int P = MvShape<PREC>::pts;
  if (n_tiles <= kFewTiles)
    hipLaunchKernelGGL((k_mv_blocks<PREC, P, 16>), dim3((unsigned)n_tiles), dim3(kTile / P), 0, s,
                       g, blocks, tiles, A, v, vscale, tpart, st);
  else
    hipLaunchKernelGGL((k_mv_blocks<PREC, P, 4>), dim3((unsigned)n_tiles), dim3(kTile / P), 0, s,
                       g, blocks, tiles, A, v, vscale, tpart, st);
}

hipError_t launch_mv_blocks(const Geo& g, int prec, const DevBlock* blocks, const Tile* tiles,
                            int64_t n_tiles, const void* A, const double* v, const double* vscale,
                            double* tpart, const SolveState* st, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  if (prec == ELMFB_FP32) mv_launch<ELMFB_FP32>(g, blocks, tiles, n_tiles, A, v, vscale, tpart, st, s);
  else if (prec == ELMFB_BF16) mv_launch<ELMFB_BF16>(g, blocks, tiles, n_tiles, A, v, vscale, tpart, st, s);
  else if (prec == ELMFB_FP16) mv_launch<ELMFB_FP16>(g, blocks, tiles, n_tiles, A, v, vscale, tpart, st, s);
  else mv_launch<ELMFB_FP64>(g, blocks, tiles, n_tiles, A, v, vscale, tpart, st, s);
  return hipGetLastError();
}

hipError_t launch_gather_rows(const Geo& g, const DevBlock* blocks, const int32_t* cov,
                              const double* tpart, int mode, double* out, const double* bvec,
                              const SolveState* st, double* red, int n_wg, const double* bc,
                              const double* v, const double* vscale, hipStream_t s) {
  const int n_bc_wg = bc ? bc_row_wgs(g) : 0;
  const bool mapped = g.domain == ELMFB_DOMAIN_L;
#define GATHER(BC, M)                                                                            \
  hipLaunchKernelGGL((k_gather_rows<BC, M>), dim3(n_wg + n_bc_wg), dim3(256), 0, s, g, blocks,   \
                     cov, tpart, mode, out, bvec, st, red, n_wg, bc, v, vscale)
  if (n_bc_wg) { if (mapped) GATHER(true, true); else GATHER(true, false); }
  else { if (mapped) GATHER(false, true); else GATHER(false, false); }
#undef GATHER
  return hipGetLastError();
}
hipError_t launch_gather_rows(const Geo& g, const DevBlock* blocks, const int32_t* cov,
                              const double* tpart, int mode, double* out, const double* bvec,
                              const SolveState* st, double* red, int n_wg, hipStream_t s) {
  return launch_gather_rows(g, blocks, cov, tpart, mode, out, bvec, st, red, n_wg, nullptr, nullptr,
                            nullptr, s);
}

template <int PREC>
static void rmv_launch(const Geo& g, const DevBlock* blocks, const Tile* chunks, int64_t n_chunks,
                       const void* A, const double* u, const double* uscale, double* part,
                       SolveState* st, const double* red, int n_red, double* hist,
                       hipStream_t s) {
  const int k8 = (g.K + 7) / 8;
  const int split = (int)std::max<int64_t>(1, std::min<int64_t>(k8, kChunkWgs / n_chunks));
  const int kper = 8 * ((k8 + split - 1) / split);
  const dim3 grid((unsigned)n_chunks, (unsigned)((g.K + kper - 1) / kper));
  if (n_chunks < kChunkWgs)
    hipLaunchKernelGGL((k_rmv_chunks<PREC, MvShape<PREC>::vec, true>), grid, dim3(256), 0, s, g,
                       blocks, chunks, A, u, uscale, part, kper, st, red, n_red, hist);
  else
    hipLaunchKernelGGL((k_rmv_chunks<PREC, MvShape<PREC>::vec, false>), grid, dim3(256), 0, s, g,
                       blocks, chunks, A, u, uscale, part, kper, st, red, n_red, hist);
}

hipError_t launch_rmv_chunks(const Geo& g, int prec, const DevBlock* blocks, const Tile* chunks,
                             int64_t n_chunks, const void* A, const double* u,
                             const double* uscale, double* part, SolveState* st,
                             const double* red, int n_red, double* hist, hipStream_t s) {
  if (n_chunks == 0) return hipSuccess;
  if (prec == ELMFB_FP32) rmv_launch<ELMFB_FP32>(g, blocks, chunks, n_chunks, A, u, uscale, part, st, red, n_red, hist, s);
  else if (prec == ELMFB_BF16) rmv_launch<ELMFB_BF16>(g, blocks, chunks, n_chunks, A, u, uscale, part, st, red, n_red, hist, s);
  else if (prec == ELMFB_FP16) rmv_launch<ELMFB_FP16>(g, blocks, chunks, n_chunks, A, u, uscale, part, st, red, n_red, hist, s);
  else rmv_launch<ELMFB_FP64>(g, blocks, chunks, n_chunks, A, u, uscale, part, st, red, n_red, hist, s);
  return hipGetLastError();
}
hipError_t launch_rmv_chunks(const Geo& g, int prec, const DevBlock* blocks, const Tile* chunks,
                             int64_t n_chunks, const void* A, const double* u,
                             const double* uscale, double* part, SolveState* st, hipStream_t s) {
  return launch_rmv_chunks(g, prec, blocks, chunks, n_chunks, A, u, uscale, part, st, nullptr, 0,
                           nullptr, s);
}

hipError_t launch_rmv_finish(const Geo& g, const int32_t* chunk_start, const double* part,
                             int mode, double* out, const SolveState* st, double* red, int n_wg,
                             const double* bc, const double* u, const double* uscale,
                             hipStream_t s) {
  if (bc && g.n_bc >= kSplitBc) {
    hipLaunchKernelGGL(k_rmv_finish_bc, dim3(n_wg), dim3(64 * kBcSlices), 0, s, g, chunk_start, part,
                       mode, out, st, red, bc, u, uscale);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_rmv_finish, dim3(n_wg), dim3(256), 0, s, g, chunk_start, part, mode, out,
                     st, red, g.n_bc > 0 ? bc : nullptr, u, uscale);
  return hipGetLastError();
}
hipError_t launch_rmv_finish(const Geo& g, const int32_t* chunk_start, const double* part,
                             int mode, double* out, const SolveState* st, double* red, int n_wg,
                             hipStream_t s) {
  return launch_rmv_finish(g, chunk_start, part, mode, out, st, red, n_wg, nullptr, nullptr,
                           nullptr, s);
}

}  // namespace elmfb
