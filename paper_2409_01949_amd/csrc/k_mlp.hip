// Kernels of the warm-start MLP: a tanh network from problem parameters to a subdomain's
// coefficient block, trained with mean-squared error and Adam (the method's optimiser and
// learning rate, Sec. 4.1).  Products take bfloat16 operands on the matrix cores
// (v_mfma_f32_16x16x32_bf16) with FP32 accumulation; master weights, biases, moments and
// pre-activations are FP32.  Rounding to bfloat16 is round-to-nearest-even.
#include <algorithm>

#include "device.h"
#include "kernels.h"

namespace elmfb {

typedef __bf16 bf8v_t __attribute__((ext_vector_type(8)));
typedef float f4v_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);   // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Workgroup tile 64 x 64, k in stages of KT = 128 or, for short products, 32; LDS rows padded by 16
// bytes (the operand reads of a wavefront then spread evenly over the banks).
constexpr int kMT = 64, kNT = 64, kKT = 128, kShortK = 32;

typedef uint16_t u16x4_t __attribute__((ext_vector_type(4)));
typedef uint16_t u16x8_t __attribute__((ext_vector_type(8)));

// How a 64 x KT (rows x k) operand tile X(row, k) = P[row sr + k sk] is staged into rows of
// consecutive k: each thread takes KT / 32 groups of 8 elements, consecutive k of a row (OP_K) or
// consecutive rows at each of as many consecutive k (OP_M: rows contiguous in memory), a 16-byte load
// each where `vec` says that the groups are aligned and the group lies within the operand.
enum { OP_K = 0, OP_M = 1 };

template <int MODE, int KT>
__device__ __forceinline__ void tile_place(int v, int* row, int* k) {
  const int t = threadIdx.x;
  if constexpr (KT == kShortK) {
    *row = MODE == OP_K ? t >> 2 : 8 * (t & 7);
    *k = MODE == OP_K ? 8 * (t & 3) : t >> 3;
  } else if constexpr (MODE == OP_K) {
    *row = (t >> 4) + 16 * v;
    *k = 8 * (t & 15);
  } else {   // per wavefront 4 groups of rows (64 contiguous bytes) x 64 k (two-way LDS banks)
    *row = 8 * ((t & 3) + 4 * ((t >> 6) & 1));
    *k = 4 * (((t >> 2) & 15) + 16 * (t >> 7)) + v;
  }
}

template <int MODE, int KT>
__device__ __forceinline__ void tile_load(const uint16_t* __restrict__ P, int64_t sr, int64_t sk,
                                          bool vec, int rows, int K, int r0, int k0,
                                          u16x8_t (&r)[KT / 32]) {
#pragma unroll
  for (int v = 0; v < KT / 32; ++v) {
    int row, k;
    tile_place<MODE, KT>(v, &row, &k);
    row += r0;
    k += k0;
    const uint16_t* q = P + (int64_t)row * sr + (int64_t)k * sk;
    const bool in = MODE == OP_K ? row < rows && k + 8 <= K : k < K && row + 8 <= rows;
    if (vec && in) {
      r[v] = *reinterpret_cast<const u16x8_t*>(q);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        r[v][e] = MODE == OP_K ? (row < rows && k + e < K ? q[e * sk] : (uint16_t)0)
                               : (k < K && row + e < rows ? q[e * sr] : (uint16_t)0);
    }
  }
}

template <int MODE, int KT>
__device__ __forceinline__ void tile_store(uint16_t (*S)[KT + 8], const u16x8_t (&r)[KT / 32]) {
  int row, k;
  if constexpr (MODE == OP_K) {
#pragma unroll
    for (int v = 0; v < KT / 32; ++v) {
      tile_place<MODE, KT>(v, &row, &k);
      *reinterpret_cast<u16x8_t*>(&S[row][k]) = r[v];
    }
  } else {
    tile_place<MODE, KT>(0, &row, &k);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (KT == kShortK) S[row + e][k] = r[0][e];
      else *reinterpret_cast<u16x4_t*>(&S[row + e][k]) = u16x4_t{r[0][e], r[1][e], r[2][e], r[3][e]};
    }
  }
}

// Partial column sums of a bfloat16 matrix g[M][N] over chunks of kColRows rows, each in the order
// of its rows (part[c][n], FP32): 64 columns of a chunk through LDS, then one wavefront.
constexpr int kColRows = 256;

__host__ __device__ inline int colsum_tasks(int M, int N) {
  return (N + 63) / 64 * ((M + kColRows - 1) / kColRows);
}

__device__ __forceinline__ void column_sums(const uint16_t* __restrict__ g, int M, int N, bool vec,
                                            int task, float* __restrict__ part, uint16_t* lds) {
  const int tiles = (N + 63) / 64, c = task / tiles, n0 = (task - c * tiles) * 64;
  const int t = threadIdx.x, m0 = c * kColRows, rows = min(M - m0, kColRows);
  u16x8_t r[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    const int row = (t >> 3) + 32 * v, n = n0 + 8 * (t & 7);
    const uint16_t* q = g + (int64_t)(m0 + row) * N + n;
    if (vec && row < rows && n + 8 <= N) {
      r[v] = *reinterpret_cast<const u16x8_t*>(q);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) r[v][e] = row < rows && n + e < N ? q[e] : (uint16_t)0;
    }
  }
#pragma unroll
  for (int v = 0; v < 8; ++v)
    *reinterpret_cast<u16x8_t*>(lds + ((t >> 3) + 32 * v) * 64 + 8 * (t & 7)) = r[v];
  __syncthreads();
  if (t < 64 && n0 + t < N) {
    float s = 0.0f;
    int m = 0;
    for (; m + 16 <= rows; m += 16) {
      float x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = bf16_to_f32(lds[(m + i) * 64 + t]);
#pragma unroll
      for (int i = 0; i < 16; ++i) s += x[i];
    }
    for (; m < rows; ++m) s += bf16_to_f32(lds[m * 64 + t]);
    part[(int64_t)c * N + n0 + t] = s;
  }
}

// The first w of 16 consecutive elements, in 16-byte accesses where all 16 are wanted and aligned.
template <typename T>
__device__ __forceinline__ bool whole_row(const T* p, int w) {
  return w == 16 && ((uintptr_t)p & 15) == 0;
}
template <typename T>
__device__ __forceinline__ void put_row(T* __restrict__ p, const T (&x)[16], int w) {
  constexpr int V = 16 / sizeof(T);
  typedef T vec_t __attribute__((ext_vector_type(V)));
  if (whole_row(p, w)) {
#pragma unroll
    for (int q = 0; q < 16; q += V) {
      vec_t v;
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = x[q + e];
      *reinterpret_cast<vec_t*>(p + q) = v;
    }
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (q < w) p[q] = x[q];
  }
}
__device__ __forceinline__ void get_row(uint16_t (&x)[16], const uint16_t* __restrict__ p, int w) {
  if (whole_row(p, w)) {
#pragma unroll
    for (int q = 0; q < 16; q += 8) {
      const u16x8_t v = *reinterpret_cast<const u16x8_t*>(p + q);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[q + e] = v[e];
    }
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = q < w ? p[q] : (uint16_t)0;
  }
}

// The epilogue of one element.
__device__ __forceinline__ void put_one(const MlpGemm& p, int S, float* __restrict__ ws, int m, int n,
                                        float c) {
  const int64_t o = (int64_t)m * p.ldo + n;
  if (S > 1) ws[((int64_t)blockIdx.z * p.M + m) * p.N + n] = c;
  else if (p.epi == MLP_EPI_F32) p.out_f32[o] = c;
  else if (p.epi == MLP_EPI_BIAS) p.out_f32[o] = c + p.bias[n];
  else if (p.epi == MLP_EPI_BIAS_TANH) p.out_bf16[o] = f32_to_bf16(tanhf(c + p.bias[n]));
  else {   // MLP_EPI_DTANH
    const float a = bf16_to_f32(p.act[o]);
    p.out_bf16[o] = f32_to_bf16(c * (1.0f - a * a));
  }
}

// C[M][N] = sum_k A(m, k) B(k, n), A(m, k) = A[m sam + k sak], B(k, n) = B[k sbk + n sbn]
// (bfloat16), then the epilogue.  Four waves of 32 x 32 (2 x 2 tiles of v_mfma_f32_16x16x32_bf16),
// k through two LDS buffers (rows of A and columns of B with k contiguous, each lane's operand one
// 16-byte read).  At these sizes (some ten microseconds of work for the whole chip) the latency of
// the stages' loads is the time, so stages are long and the loads of three are in flight:
// 4096 x 512 x 512 15.1 -> 11.6 us per layer forward, 18.8 -> 11.2 with a transposed operand, dW
// 25.7 -> 12.9 with the column sums (51 us more by themselves), against stages of 32, one ahead,
// and 2-byte stores.  (A launch is 3 to 4 us of each, tanhf 1.3, writing the result 3.)  Workgroups go to the 8 XCDs in turn: each takes consecutive rows of tiles, so
// that its L2 reads a share of A and all of the (small) B.  With S > 1 workgroup z covers k in
// [z kc, (z + 1) kc) and writes its FP32 partial tile to ws[z][M][N]; k_mlp_gemm_reduce sums them
// in order and applies the epilogue.  The workgroups of z >= S, if any, form the column sums of A^T
// (p.colsum), one task each.
template <int MA, int MB, int KT>
__global__ void __launch_bounds__(256) k_mlp_gemm(MlpGemm p, bool va, bool vb, int kc, int S,
                                                  float* __restrict__ ws) {
  extern __shared__ __align__(16) uint16_t mlp_lds[];
  const int nx = gridDim.x, tiles = nx * gridDim.y;
  int id = blockIdx.y * nx + blockIdx.x;
  if ((int)blockIdx.z >= S) {
    id += ((int)blockIdx.z - S) * tiles;
    if (id < colsum_tasks(p.K, p.M)) column_sums(p.A, p.K, p.M, va, id, p.colpart, mlp_lds);
    return;
  }
  typedef uint16_t Buf[kMT + kNT][KT + 8];
  Buf* const T = reinterpret_cast<Buf*>(mlp_lds);   // [2]: rows of A, then columns of B
  id = xcd_tile(id, tiles);
  const int m0 = id / nx * kMT, n0 = id % nx * kNT;
  const int kb = blockIdx.z * kc, ke = min(p.K, kb + kc);
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wid >> 1, wn = wid & 1;
  const int li = lane & 15, lq = lane >> 4;
  f4v_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f4v_t{0.f, 0.f, 0.f, 0.f};
  u16x8_t ra[4][KT / 32], rb[4][KT / 32];
  // operand B is staged as its transpose: rows n, X(n, k) = B[k sbk + n sbn]
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (kb + u * KT < ke) {
      tile_load<MA, KT>(p.A, p.sam, p.sak, va, p.M, ke, m0, kb + u * KT, ra[u]);
      tile_load<MB, KT>(p.B, p.sbn, p.sbk, vb, p.N, ke, n0, kb + u * KT, rb[u]);
    }
  for (int k4 = kb; k4 < ke; k4 += 4 * KT) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k0 = k4 + u * KT;
      if (k0 < ke) {
        // the buffer's last readers passed the barrier of the stage between
        Buf& Sb = T[u & 1];
        tile_store<MA, KT>(Sb, ra[u]);
        tile_store<MB, KT>(Sb + kMT, rb[u]);
        if (k0 + 3 * KT < ke) {
          tile_load<MA, KT>(p.A, p.sam, p.sak, va, p.M, ke, m0, k0 + 3 * KT, ra[(u + 3) & 3]);
          tile_load<MB, KT>(p.B, p.sbn, p.sbk, vb, p.N, ke, n0, k0 + 3 * KT, rb[(u + 3) & 3]);
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < KT; ks += 32) {
          if (k0 + ks >= ke) break;
          bf8v_t a[2], b[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            a[i] = *reinterpret_cast<const bf8v_t*>(&Sb[wm * 32 + i * 16 + li][ks + 8 * lq]);
            b[i] = *reinterpret_cast<const bf8v_t*>(&Sb[kMT + wn * 32 + i * 16 + li][ks + 8 * lq]);
          }
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
      }
    }
  }
  if constexpr (KT == kShortK) {
    if (p.M < kMT) {   // few rows: their elements one by one, over all lanes that hold any
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int m = wm * 32 + i * 16 + 4 * lq + v, n = n0 + wn * 32 + j * 16 + li;
            if (m < p.M && n < p.N) put_one(p, S, ws, m, n, acc[i][j][v]);
          }
      return;
    }
  }
  // the tile through LDS (lane holds column li, rows 4 lq + v of an accumulator), so that a thread
  // has 16 consecutive columns of a row: results go out in whole 16-byte stores
  __syncthreads();
  float (*const C)[kNT + 4] = reinterpret_cast<float (*)[kNT + 4]>(mlp_lds);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        C[wm * 32 + i * 16 + 4 * lq + v][wn * 32 + j * 16 + li] = acc[i][j][v];
  __syncthreads();
  const int row = threadIdx.x >> 2, col = 16 * (threadIdx.x & 3);
  const int m = m0 + row, n = n0 + col;
  if (m >= p.M || n >= p.N) return;
  const int w = min(16, p.N - n);
  float c[16];
#pragma unroll
  for (int q = 0; q < 16; q += 4)
    *reinterpret_cast<f4v_t*>(c + q) = *reinterpret_cast<const f4v_t*>(&C[row][col + q]);
  if (S > 1) {
    put_row(ws + ((int64_t)blockIdx.z * p.M + m) * p.N + n, c, w);
    return;
  }
  const int64_t o = (int64_t)m * p.ldo + n;
  if (p.epi == MLP_EPI_F32) {
    put_row(p.out_f32 + o, c, w);
  } else if (p.epi == MLP_EPI_BIAS) {
#pragma unroll
    for (int q = 0; q < 16; ++q) c[q] += p.bias[n + min(q, w - 1)];
    put_row(p.out_f32 + o, c, w);
  } else if (p.epi == MLP_EPI_BIAS_TANH) {
    uint16_t r[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) r[q] = f32_to_bf16(tanhf(c[q] + p.bias[n + min(q, w - 1)]));
    put_row(p.out_bf16 + o, r, w);
  } else {   // MLP_EPI_DTANH
    uint16_t r[16];
    get_row(r, p.act + o, w);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const float a = bf16_to_f32(r[q]);
      r[q] = f32_to_bf16(c[q] * (1.0f - a * a));
    }
    put_row(p.out_bf16 + o, r, w);
  }
}

// Sum of the S partial tiles of a split-k product, in order of z (F32 epilogue; S = 1: none), and
// of the partial column sums, in order of their chunks.
__global__ void k_mlp_gemm_reduce(MlpGemm p, int S, const float* __restrict__ ws) {
  const int64_t MN = S > 1 ? (int64_t)p.M * p.N : p.M;
  const int nc = (p.K + kColRows - 1) / kColRows;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < MN;
       e += (int64_t)gridDim.x * blockDim.x) {
    if (S > 1) {
      float c = 0.0f;
      for (int z = 0; z < S; ++z) c += ws[z * MN + e];
      const int64_t m = e / p.N, n = e - m * p.N;
      p.out_f32[m * p.ldo + n] = c;
    }
    if (p.colsum && e < p.M) {   // M <= M N
      float r = 0.0f;
      for (int c = 0; c < nc; ++c) r += p.colpart[(int64_t)c * p.M + e];
      p.colsum[e] = r;
    }
  }
}

// y [rows][ld] = bf16(x [rows][cols]).
__global__ void k_mlp_rows_to_bf16(int64_t rows, int cols, int ld, const float* __restrict__ x,
                                   uint16_t* __restrict__ y) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < rows * cols;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / cols;
    y[r * ld + (i - r * cols)] = f32_to_bf16(x[i]);
  }
}

__global__ void k_mlp_to_bf16(int64_t n, const float* __restrict__ x, uint16_t* __restrict__ y) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    y[i] = f32_to_bf16(x[i]);
}

// g = bf16(2 (y - t) / n); per-workgroup partial sums of (y - t)^2 in FP64.
__global__ void __launch_bounds__(256) k_mlp_loss(int64_t n, const float* __restrict__ y,
                                                  const float* __restrict__ t,
                                                  uint16_t* __restrict__ g,
                                                  double* __restrict__ part) {
  __shared__ double sh[4];
  double acc = 0.0;
  const float sc = 2.0f / (float)n;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float d = y[i] - t[i];
    g[i] = f32_to_bf16(sc * d);
    acc += (double)d * (double)d;
  }
  const double s = block_sum256(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Modulated output y[b][k] = sum_i f[b][i] z[b][i K + k] (FP32).
__global__ void k_mlp_modulate(int64_t n, int K, int n_mod, const float* __restrict__ z,
                               const float* __restrict__ f, float* __restrict__ y) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = e / K;
    const int k = (int)(e - b * K);
    float s = 0.0f;
    for (int i = 0; i < n_mod; ++i) s += f[b * n_mod + i] * z[(b * n_mod + i) * K + k];
    y[e] = s;
  }
}

// Loss of the modulated output: d = y - t, g = 2 d / n, gz[b][i K + k] = bf16(f[b][i] g);
// per-workgroup partial sums of d^2 in FP64.
__global__ void __launch_bounds__(256) k_mlp_mod_loss(int64_t n, int K, int n_mod,
                                                      const float* __restrict__ z,
                                                      const float* __restrict__ f,
                                                      const float* __restrict__ t,
                                                      uint16_t* __restrict__ gz,
                                                      double* __restrict__ part) {
  __shared__ double sh[4];
  double acc = 0.0;
  const float sc = 2.0f / (float)n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = e / K;
    const int k = (int)(e - b * K);
    float y = 0.0f;
    for (int i = 0; i < n_mod; ++i) y += f[b * n_mod + i] * z[(b * n_mod + i) * K + k];
    const float d = y - t[e];
    const float g = sc * d;
    for (int i = 0; i < n_mod; ++i) gz[(b * n_mod + i) * K + k] = f32_to_bf16(f[b * n_mod + i] * g);
    acc += (double)d * (double)d;
  }
  const double s = block_sum256(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(256) k_mlp_sum(int n, const double* __restrict__ part,
                                                 double scale, double* __restrict__ out) {
  __shared__ double sh[4];
  const double s = reduce_partials(part, n, sh);
  if (threadIdx.x == 0) *out = s * scale;
}

// Adam on the flat FP32 parameters; refreshes their bfloat16 copy.
__global__ void k_mlp_adam(int64_t n, float* __restrict__ prm, const float* __restrict__ grad,
                           float* __restrict__ m1, float* __restrict__ m2,
                           uint16_t* __restrict__ pb, float lr, float b1, float b2, float eps,
                           float c1, float c2) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float g = grad[i];
    const float a = b1 * m1[i] + (1.0f - b1) * g;
    const float b = b2 * m2[i] + (1.0f - b2) * g * g;
    m1[i] = a;
    m2[i] = b;
    const float p = prm[i] - lr * (a / c1) / (sqrtf(b / c2) + eps);
    prm[i] = p;
    pb[i] = f32_to_bf16(p);
  }
}

static unsigned flat_grid(int64_t n) {
  int64_t g = (n + 255) / 256;
  return (unsigned)(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

static bool aligned16(const void* q) { return ((uintptr_t)q & 15) == 0; }

int mlp_colsum_chunks(int K) { return std::max(1, (K + kColRows - 1) / kColRows); }

int64_t mlp_gemm_ws_floats(int M, int N, int K) {
  const int S = mlp_gemm_splits(M, N, K);
  return S > 1 ? (int64_t)S * M * N : 0;
}

// Split k when the output has too few tiles to fill the chip and k is long (the weight
// gradients: k = batch): about 256 workgroups, at least 256 k per split.
int mlp_gemm_splits(int M, int N, int K) {
  const int64_t tiles = (int64_t)((N + kNT - 1) / kNT) * ((M + kMT - 1) / kMT);
  if (tiles >= 256) return 1;
  int S = (int)std::min<int64_t>(256 / tiles, K / 256);
  return std::max(1, std::min(S, 64));
}

hipError_t launch_mlp_gemm(const MlpGemm& p, float* ws, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0) return hipSuccess;
  int S = p.epi == MLP_EPI_F32 && ws ? mlp_gemm_splits(p.M, p.N, p.K) : 1;
  int kc = p.K;
  if (S > 1) {
    kc = ((p.K + S - 1) / S + 31) / 32 * 32;
    S = (p.K + kc - 1) / kc;
  }
  const int nx = (p.N + kNT - 1) / kNT, ny = (p.M + kMT - 1) / kMT;
  const int64_t tiles = (int64_t)nx * ny;
  const int nz = p.colsum ? (int)((colsum_tasks(p.K, p.M) + tiles - 1) / tiles) : 0;
  const dim3 grid((unsigned)nx, (unsigned)ny, (unsigned)(S + nz));
  // up to 64 k in stages of 32: a stage of 128 of which half is there takes longer to load and store
  // (predictions of one row through widths 4, 16, 16, 8 26.1 against 35.8 us, of 4,096 rows through 4,
  // 48, 16 28.7 against 31.4; a layer of 64 rows, 64 by 64, 4.2 against 5.2)
  const bool sh = kc <= 2 * kShortK;
  // two stages (68 KB), in short ones at least a task of the column sums
  const size_t lds = sh ? (size_t)kColRows * 64 * sizeof(uint16_t)
                        : 2 * (kMT + kNT) * (kKT + 8) * sizeof(uint16_t);
  const bool am = p.sak != 1 && p.sam == 1, bm = p.sbk != 1 && p.sbn == 1;
  const bool va = aligned16(p.A) && (am ? p.sak % 8 == 0 : p.sak == 1 && p.sam % 8 == 0);
  const bool vb = aligned16(p.B) && (bm ? p.sbk % 8 == 0 : p.sbk == 1 && p.sbn % 8 == 0);
  float* w = S > 1 ? ws : nullptr;
  hipError_t e = hipSuccess;
#define GEMM(A_, B_)                                                                             \
  do {                                                                                           \
    if (sh) {                                                                                    \
      hipLaunchKernelGGL((k_mlp_gemm<A_, B_, kShortK>), grid, dim3(256), lds, s, p, va, vb, kc, S, w); \
      break;                                                                                     \
    }                                                                                            \
    e = hipFuncSetAttribute((const void*)k_mlp_gemm<A_, B_, kKT>,                                \
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);               \
    if (e != hipSuccess) return e;                                                               \
    hipLaunchKernelGGL((k_mlp_gemm<A_, B_, kKT>), grid, dim3(256), lds, s, p, va, vb, kc, S, w);  \
  } while (0)
  if (am) { if (bm) GEMM(OP_M, OP_M); else GEMM(OP_M, OP_K); }
  else { if (bm) GEMM(OP_K, OP_M); else GEMM(OP_K, OP_K); }
#undef GEMM
  if (S > 1 || p.colsum) {
    const int64_t MN = S > 1 ? (int64_t)p.M * p.N : p.M;
    hipLaunchKernelGGL(k_mlp_gemm_reduce, dim3(flat_grid(MN)), dim3(256), 0, s, p, S, ws);
  }
  return hipGetLastError();
}
hipError_t launch_mlp_to_bf16(int64_t n, const float* x, uint16_t* y, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_to_bf16, dim3(flat_grid(n)), dim3(256), 0, s, n, x, y);
  return hipGetLastError();
}
hipError_t launch_mlp_rows_to_bf16(int64_t rows, int cols, int ld, const float* x, uint16_t* y,
                                   hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_rows_to_bf16, dim3(flat_grid(rows * cols)), dim3(256), 0, s, rows, cols,
                     ld, x, y);
  return hipGetLastError();
}
hipError_t launch_mlp_loss(int64_t n, const float* y, const float* t, uint16_t* g, double* part,
                           int n_part, double* loss, hipStream_t s) {
  const unsigned nb = (unsigned)std::min<int64_t>(n_part, std::max<int64_t>(1, (n + 255) / 256));
  hipLaunchKernelGGL(k_mlp_loss, dim3(nb), dim3(256), 0, s, n, y, t, g, part);
  hipLaunchKernelGGL(k_mlp_sum, dim3(1), dim3(256), 0, s, (int)nb, part, 1.0 / (double)n, loss);
  return hipGetLastError();
}
hipError_t launch_mlp_modulate(int64_t n, int K, int n_mod, const float* z, const float* f,
                               float* y, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_modulate, dim3(flat_grid(n)), dim3(256), 0, s, n, K, n_mod, z, f, y);
  return hipGetLastError();
}
hipError_t launch_mlp_mod_loss(int64_t n, int K, int n_mod, const float* z, const float* f,
                               const float* t, uint16_t* gz, double* part, int n_part,
                               double* loss, hipStream_t s) {
  const unsigned nb = (unsigned)std::min<int64_t>(n_part, std::max<int64_t>(1, (n + 255) / 256));
  hipLaunchKernelGGL(k_mlp_mod_loss, dim3(nb), dim3(256), 0, s, n, K, n_mod, z, f, t, gz, part);
  hipLaunchKernelGGL(k_mlp_sum, dim3(1), dim3(256), 0, s, (int)nb, part, 1.0 / (double)n, loss);
  return hipGetLastError();
}
hipError_t launch_mlp_adam(int64_t n, float* prm, const float* grad, float* m1, float* m2,
                           uint16_t* pb, float lr, float b1, float b2, float eps, float c1,
                           float c2, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_adam, dim3(flat_grid(n)), dim3(256), 0, s, n, prm, grad, m1, m2, pb, lr,
                     b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace elmfb
