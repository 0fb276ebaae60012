// Evaluation of the fitted solution at arbitrary points (Sec. 3 eq. multilevel_solution, times
// the hard-constraint factor of Sec. 4.3):
//   u(x) = C(x) (1/L) sum_l sum_{j : x in supp omega_j} omega_j(x) sum_k a_q tanh(W_q xbar + b_q).
// One wavefront per point.  Two levels at a time, 16 lanes per (level, axis) test the candidate
// subdomains of that axis together (centre spacing, then the support test |x - mu| < sigma) and
// sum their windows for the partition of unity; the covering blocks of a level are then listed in
// LDS and the lanes take their (block, feature) pairs 64 at a time, so no lane idles on a feature
// count that is no multiple of 64.  The point's sum is reduced across the wavefront at the end in
// a fixed order.  Bound by instruction issue: a tanh (the LDS table) and its loads per pair.
// Calls on 230,400 points of the 3-level problem (16 blocks of K = 96 a point): 4.30 ms with a
// serial covering search in every lane and the device library's tanh, 0.99 ms so; 9,216 points of
// the L-shaped baseline (K = 16, where 48 of 64 lanes idled) 69 -> 16 us.  Held to 80 registers (6
// wavefronts a SIMD for 4) it spills and takes 15% longer.
#include "device.h"
#include "fast_tanh.h"
#include "kernels.h"

namespace elmfb {

constexpr int kMaxCover = 8;   // covering subdomains per axis and level (width ratio < 7)
constexpr int kEvWaves = 4;

// One covering block of a point: its weight omega_j, the feature inputs and its first column.
struct EvBlock {
  double w, xb, yb;
  int64_t q0;      // -1: a subdomain discarded from an L-shaped domain
};

// Value of the hard-constraint factor along one axis.
__device__ __forceinline__ double ansatz_value(const Geo& g, int a, double x, const double2* tt) {
  const double w = g.ansatz_omega;
  if (g.ansatz == ELMFB_ANSATZ_TANH_BOX && a < g.dim)
    return table_tanh(w * (x - g.lo[a]), tt) * table_tanh(w * (g.hi[a] - x), tt);
  if (g.ansatz == ELMFB_ANSATZ_TANH_ORIGIN && a == 0) return table_tanh(w * x, tt);
  return 1.0;
}

__global__ void __launch_bounds__(64 * kEvWaves) k_evaluate(Geo g, const double* __restrict__ W,
                                                            const double* __restrict__ bias,
                                                            const double* __restrict__ coef,
                                                            const double* __restrict__ pts,
                                                            int64_t n_pts,
                                                            double* __restrict__ u) {
  __shared__ double2 tt[kTanhN];
  // per wavefront: (window, feature input) of the covering subdomains, [level pair][axis][slot]
  __shared__ double2 axis_s[kEvWaves][2][2][kMaxCover];
  __shared__ EvBlock list_s[kEvWaves][kMaxCover * kMaxCover];
  stage_tanh(tt);
  __syncthreads();
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  double2(*ax)[2][kMaxCover] = axis_s[wid];
  EvBlock* list = list_s[wid];
  const int K = g.K;
  const int dq = 64 / K, dr = 64 - dq * K;          // (block, feature) 64 pairs on
  const int c0 = lane / K, k0 = lane - c0 * K;
  const bool lshape = g.domain == ELMFB_DOMAIN_L;
  const int half = lane >> 5, axl = (lane >> 4) & 1, cand = lane & 15;
  const int64_t nwaves = (int64_t)gridDim.x * kEvWaves;
  for (int64_t i = (int64_t)blockIdx.x * kEvWaves + wid; i < n_pts; i += nwaves) {
    const double px = pts[i * g.dim];
    const double py = (g.dim == 2) ? pts[i * g.dim + 1] : 0.0;
    double total = 0.0;
    for (int l0 = 0; l0 < g.n_levels; l0 += 2) {
      // this lane's candidate: level l0 + half, axis axl, subdomain j
      const int l = l0 + half;
      bool in = false;
      double w = 0.0, xb = 0.0, d = 0.0;
      int j = 0;
      if (l < g.n_levels) {
        const double x = axl ? py : px;
        const int J = g.J[l][axl];
        if (J == 1 || axl >= g.dim) {
          in = cand == 0;
          w = in ? 1.0 : 0.0;
          xb = axl < g.dim ? feat_in(g, l, axl, 0, x) : 0.0;
        } else {
          const double h = g.cen_h[l][axl], sigma = g.sigma[l][axl];
          int j0 = (int)floor((x - g.lo[axl] - sigma) / h) - 1;
          int j1 = (int)ceil((x - g.lo[axl] + sigma) / h) + 1;
          if (j0 < 0) j0 = 0;
          if (j1 > J - 1) j1 = J - 1;
          j = j0 + cand;
          if (j <= j1) {
            const double mu = centre(g, l, axl, j);
            if (fabs(x - mu) < sigma) {
              in = true;
              double w1, w2;
              raw_window(x, mu, sigma, w, w1, w2);
              xb = feat_in(g, l, axl, j, x);
              // L domain: the sum over the centres above the midpoint (the discarded subdomains
              // are the products of such centres on both axes)
              if (lshape && mu > g.lmid[axl]) d = w;
            }
          }
        }
      }
      double S = w, D = d;
#pragma unroll
      for (int o = 8; o >= 1; o >>= 1) {
        S += __shfl_xor(S, o, 64);
        D += __shfl_xor(D, o, 64);
      }
      const unsigned m = (unsigned)(__ballot(in) >> (lane & 48)) & 0xffffu;
      const int first = m ? __builtin_ctz(m) : 0;   // the support is a run of subdomains
      const int n = min((int)__popc(m), kMaxCover);
      if (in && cand - first < kMaxCover) ax[half][axl][cand - first] = double2{lshape ? w : w / S, xb};
      const int jf = j - cand + first;
      __builtin_amdgcn_wave_barrier();   // LDS is in order within a wavefront
      for (int h = 0; h < 2 && l0 + h < g.n_levels; ++h) {
        const int lv = l0 + h, bx = 32 * h, by = 32 * h + 16;
        const int nx = __shfl(n, bx, 64), ny = __shfl(n, by, 64);
        const int jx0 = __shfl(jf, bx, 64), jy0 = __shfl(jf, by, 64);
        double inv_s = 1.0;
        if (lshape) {
          // windows normalised over the kept subdomains: S = Sx Sy - Dx Dy
          inv_s = 1.0 / (__shfl(S, bx, 64) * __shfl(S, by, 64) -
                         __shfl(D, bx, 64) * __shfl(D, by, 64));
        }
        const int nc = nx * ny;
        // off every support of an L-shaped domain's level the windows are 0/0: NaN (a box: 0)
        if (nc == 0) total += 0.0 * inv_s;
        if (lane < nc) {
          const int a = lane / ny, c = lane - a * ny;
          int bi = (jx0 + a) * g.J[lv][1] + jy0 + c;
          bi = lshape ? g.bmap[g.bmap_off[lv] + bi] : g.bbase[lv] + bi;
          const double2 X = ax[h][0][a], Y = ax[h][1][c];
          list[lane] = EvBlock{X.x * Y.x * inv_s, X.y, Y.y, bi < 0 ? -1 : (int64_t)bi * K};
        }
        __builtin_amdgcn_wave_barrier();
        int c = c0, k = k0;
        double lev = 0.0;                // a level at a time: fewer terms to a running sum
        while (c < nc) {
          const EvBlock B = list[c];
          if (B.q0 >= 0) {
            const int64_t q = B.q0 + k;
            const double2 wq = reinterpret_cast<const double2*>(W)[q];
            const double z = wq.x * B.xb + wq.y * B.yb + bias[q];
            lev += B.w * (coef[q] * table_tanh(z, tt));
          }
          c += dq;
          k += dr;
          if (k >= K) {
            k -= K;
            ++c;
          }
        }
        total += lev;
        __builtin_amdgcn_wave_barrier();
      }
    }
    total = wave_sum(total);
    const double cx = ansatz_value(g, 0, px, tt), cy = ansatz_value(g, 1, py, tt);
    if (lane == 0) u[i] = total * (cx * cy) * g.inv_levels;
  }
}

__global__ void __launch_bounds__(256) k_rel_l2_partials(const double* __restrict__ u,
                                                         const double* __restrict__ ref,
                                                         int64_t n, double* __restrict__ red) {
  __shared__ double sh[4];
  double a = 0.0, b = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double d = u[i] - ref[i];
    a += d * d;
    b += ref[i] * ref[i];
  }
  const double sa = block_sum256(a, sh);
  const double sb = block_sum256(b, sh);
  if (threadIdx.x == 0) {
    red[2 * blockIdx.x] = sa;
    red[2 * blockIdx.x + 1] = sb;
  }
}

__global__ void __launch_bounds__(256) k_rel_l2_final(const double* __restrict__ red, int n,
                                                      SolveState* st) {
  __shared__ double sh[4];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    a += red[2 * i];
    b += red[2 * i + 1];
  }
  const double sa = block_sum256(a, sh);
  const double sb = block_sum256(b, sh);
  if (threadIdx.x == 0) {
    const double r = sqrt(sa) / sqrt(sb);
    st->rel_l2 = r;
    if (st->target > 0.0 && r <= st->target) {
      st->target_hit = 1;
      st->istop = 8;
      st->done = 1;
    }
  }
}

hipError_t launch_evaluate(const Geo& g, const double* W, const double* b, const double* coef,
                           const double* pts, int64_t n_pts, double* u, hipStream_t s) {
  if (n_pts == 0) return hipSuccess;
  // a wavefront per point, up to 8 workgroups per CU (each stages the 10 KB tanh table once)
  int64_t nb = (n_pts + kEvWaves - 1) / kEvWaves;
  if (nb > 2048) nb = 2048;
  hipLaunchKernelGGL(k_evaluate, dim3((unsigned)nb), dim3(64 * kEvWaves), 0, s, g, W, b, coef, pts, n_pts, u);
  return hipGetLastError();
}

hipError_t launch_check_rel_l2(const double* u, const double* ref, int64_t n, SolveState* st,
                               double* red, int n_wg, hipStream_t s) {
  hipLaunchKernelGGL(k_rel_l2_partials, dim3(n_wg), dim3(256), 0, s, u, ref, n, red);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_rel_l2_final, dim3(1), dim3(256), 0, s, red, n_wg, st);
  return hipGetLastError();
}

}  // namespace elmfb
