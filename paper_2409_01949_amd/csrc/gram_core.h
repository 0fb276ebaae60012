// C = X Y^T on the matrix cores for two groups of up to 32 WT feature rows over a set of points,
// shared by the Gram blocks of single problems and of batches.
//
// The points are `rows` runs of `len` consecutive points of both operands (one run where the
// shared box is a whole block).  A run is read in loads of 8 or 16 bytes (GramLoad) whatever its
// alignment, the last one masked; a stage is 128 bytes of every feature row in LDS, the next
// stage's loads in registers meanwhile.  Row stride 144 bytes: the 16 rows x 4 vectors of a fragment
// read fall on every bank equally.  A lane's fragment is one 16-byte LDS read, which feeds one 16-bit MFMA or several of the FP32
// and FP64 forms (k-slot lane/16 takes the lane's own points in turn: the same for X and Y).
//
// Four wavefronts: 2 x 2 squares of WT x WT tiles of 16 x 16, so a fragment serves WT products
// (GRAM_SQUARE), or the tiles dealt to them in turn: all of them (GRAM_DEALT) or, for X = Y, those
// on and above the diagonal (GRAM_UPPER).
#pragma once

#include "device.h"

namespace elmfb {

typedef uint32_t gr_vec __attribute__((ext_vector_type(4)));
typedef double gr_d4 __attribute__((ext_vector_type(4)));
typedef double gr_d2 __attribute__((ext_vector_type(2)));
typedef float gr_f4 __attribute__((ext_vector_type(4)));
typedef __bf16 gr_b8 __attribute__((ext_vector_type(8)));
typedef _Float16 gr_h8 __attribute__((ext_vector_type(8)));

template <int PREC> struct GramT { typedef gr_f4 acc; typedef float out; static constexpr int es = 2; };
template <> struct GramT<ELMFB_FP64> { typedef gr_d4 acc; typedef double out; static constexpr int es = 8; };
template <> struct GramT<ELMFB_FP32> { typedef gr_f4 acc; typedef float out; static constexpr int es = 4; };

constexpr int kGrVecs = 8;             // 16-byte vectors of a feature row in a stage
constexpr int kGrStride = kGrVecs + 1; // and of an LDS row: one of padding

// One load: 16 bytes, but 8 where that measured faster.  The runs start at any entry, and a load off
// its own size is split on the way: FP64 entries are loaded singly (all pairs of K = 96 8.7 against
// 11.3 ms, K = 48 0.54 against 0.72), FP32 entries by 4 (4.5 against 4.9 by 2 and 4.5 singly).
// 16-bit entries on squares of 64 and 96 are loaded by 4 from the three dwords around them and cut
// out: whole dwords are never split (K = 96 1.60 -> 1.54 ms, K = 48 120 -> 107 us, against 8-byte
// and 16-byte loads where they lie).  The other squares read 16 bytes: those of 128 lose by the cuts
// (273 blocks of K = 100 / 128 / 160 / 256, all pairs: 247 / 325 / 808 / 1,213 us against 265 / 323 /
// 895 / 1,234; only 11 blocks of K = 100 to 128 gain, 33 to 31), those of 32 are within 5% either way
// (K = 8 39 against 42, K = 32 57 against 56).
typedef uint32_t gr_half __attribute__((ext_vector_type(2)));
template <int PREC, int WT> struct GramLoad { typedef gr_vec t; };
template <int WT> struct GramLoad<ELMFB_FP64, WT> { typedef double t; };
template <> struct GramLoad<ELMFB_FP16, 2> { typedef gr_half t; };
template <> struct GramLoad<ELMFB_FP16, 3> { typedef gr_half t; };
template <> struct GramLoad<ELMFB_BF16, 2> { typedef gr_half t; };
template <> struct GramLoad<ELMFB_BF16, 3> { typedef gr_half t; };

// Points and operands of one product.
struct GramRun {
  const char* x;                      // feature row 0 of X at the first point, and of Y
  const char* y;
  int64_t ldx, ldy;                   // bytes from one feature row to the next
  int64_t stepx, stepy;               // bytes from one run of points to the next
  int nx, ny;                         // feature rows (<= 32 WT)
  int len;                            // points of a run
  int v0, v1;                         // loads (GramLoad), run by run
};

// Product e of a fragment pair (PREC's MFMA takes 2, 4 or all 8 of a fragment's points in turn): the
// callers run e outermost over several tiles, so that no product waits for its own accumulator.
template <int PREC>
constexpr int kGramSteps = PREC == ELMFB_FP64 ? 2 : (PREC == ELMFB_FP32 ? 4 : 1);

template <int PREC>
__device__ __forceinline__ void gram_mma(gr_vec a, gr_vec b, int e, typename GramT<PREC>::acc& c) {
  if constexpr (PREC == ELMFB_FP64) {
    const gr_d2 x = __builtin_bit_cast(gr_d2, a), y = __builtin_bit_cast(gr_d2, b);
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(x[e], y[e], c, 0, 0, 0);
  } else if constexpr (PREC == ELMFB_FP32) {
    const gr_f4 x = __builtin_bit_cast(gr_f4, a), y = __builtin_bit_cast(gr_f4, b);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], c, 0, 0, 0);
  } else if constexpr (PREC == ELMFB_BF16) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(gr_b8, a),
                                                __builtin_bit_cast(gr_b8, b), c, 0, 0, 0);
  } else {
    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(gr_h8, a),
                                               __builtin_bit_cast(gr_h8, b), c, 0, 0, 0);
  }
}

// Tile (I, J), I <= J, number t of the upper tiles of an n x n array, row by row.
__device__ __forceinline__ void gram_upper(int t, int n, int& I, int& J) {
  I = 0;
  while (t >= n - I) {
    t -= n - I;
    ++I;
  }
  J = I + t;
}

// lds: 2 x 32 WT x kGrStride vectors (the second half unused for GRAM_UPPER).  put(row, column, value)
// receives every product of the tiles computed (rows and columns past nx, ny are dropped).
enum { GRAM_SQUARE = 0, GRAM_DEALT = 1, GRAM_UPPER = 2 };

template <int PREC, int WT, int MODE, typename PUT>
__device__ __forceinline__ void gram_product(const GramRun& R, gr_vec* lds, PUT put) {
  typedef typename GramT<PREC>::acc acc_t;
  typedef typename GramLoad<PREC, WT>::t vec_t;
  constexpr int ES = GramT<PREC>::es, VB = sizeof(vec_t), VE = VB / ES, NS = 128 / VB;
  constexpr int TD = 2 * WT;                                   // tiles per dimension
  constexpr bool SAME = MODE == GRAM_UPPER, DEAL = MODE != GRAM_SQUARE;
  constexpr int NT = SAME ? (TD * (TD + 1) / 2 + 3) / 4 : WT * WT;
  gr_vec* X = lds;
  gr_vec* Y = SAME ? lds : lds + 32 * WT * kGrStride;
  const int t = threadIdx.x, lane = t & 63;
  const int wid = __builtin_amdgcn_readfirstlane(t >> 6);
  const int li = lane & 15, lq = lane >> 4;
  constexpr int NR = 256 / NS, NL = 32 * WT / NR;              // rows a pass, passes
  const int slot = t % NS, f0 = t / NS;                        // staging: load, first feature row
  const int nv = (R.len + VE - 1) / VE;                        // loads of a run, at least 1
  const int ntx = (R.nx + 15) >> 4, nty = (R.ny + 15) >> 4;
  acc_t acc[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) acc[i] = acc_t{0, 0, 0, 0};
  // dealt tiles: LDS offsets of this wavefront's
  const int nt = SAME ? ntx * (ntx + 1) / 2 : ntx * nty;
  int tI[DEAL ? NT : 1], tJ[DEAL ? NT : 1];
  const gr_vec* xl = X + li * kGrStride + lq;
  const gr_vec* yl = Y + li * kGrStride + lq;
  if constexpr (DEAL) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      int I = 0, J = 0;
      if (wid + 4 * i < nt) {
        if constexpr (SAME) gram_upper(wid + 4 * i, ntx, I, J);
        else I = (wid + 4 * i) / nty, J = (wid + 4 * i) % nty;
      }
      tI[i] = 16 * I * kGrStride;
      tJ[i] = 16 * J * kGrStride;
    }
  }
  // HALF: the dwords around each load, and the bits to its first point
  constexpr bool HALF = ES == 2 && VB == 8;
  struct wide_t { uint32_t d[3]; };
  wide_t wx[HALF ? NL : 1], wy[HALF ? NL : 1];
  uint32_t hx = 0, hy = 0;
  vec_t rx[NL], ry[NL], mask{};
  int v = R.v0 + slot, run = v / nv, c = v - run * nv;
  auto fetch = [&]() {
    const int left = v < R.v1 ? R.len - c * VE : 0;            // points from this load on
    const int64_t ox = run * R.stepx + (int64_t)c * VB, oy = run * R.stepy + (int64_t)c * VB;
    vec_t m{};
    if constexpr (VE > 1) m = ~m;
    if (VE > 1 && left < VE) {
#pragma unroll
      for (int d = 0; d < VB / 4; ++d) {
        const int b = min(max(left * ES - 4 * d, 0), 4);
        if constexpr (VE > 1) m[d] = b == 4 ? ~0u : (1u << (8 * b)) - 1;
      }
    }
    const char* px = R.x + ox;
    const char* py = R.y + oy;
    if constexpr (HALF) {
      hx = 8 * ((uintptr_t)px & 2), hy = 8 * ((uintptr_t)py & 2);
      px -= (uintptr_t)px & 2, py -= (uintptr_t)py & 2;
      mask = m;
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int f = f0 + NR * i;
      if constexpr (HALF) {
        wx[i] = wy[i] = wide_t{};
        if (left > 0 && f < R.nx) wx[i] = *reinterpret_cast<const wide_t*>(px + f * R.ldx);
        if (!SAME && left > 0 && f < R.ny) wy[i] = *reinterpret_cast<const wide_t*>(py + f * R.ldy);
        continue;
      }
      rx[i] = ry[i] = vec_t{};
      if (left > 0 && f < R.nx) __builtin_memcpy(&rx[i], R.x + f * R.ldx + ox, VB);
      if (!SAME && left > 0 && f < R.ny) __builtin_memcpy(&ry[i], R.y + f * R.ldy + oy, VB);
      if constexpr (VE > 1) {
        rx[i] &= m;
        if (!SAME) ry[i] &= m;
      }
    }
    v += NS;
    c += NS;
    while (c >= nv) {
      c -= nv;
      ++run;
    }
  };
  fetch();
  vec_t* Xs = reinterpret_cast<vec_t*>(X);
  vec_t* Ys = reinterpret_cast<vec_t*>(Y);
  constexpr int LS = kGrStride * 16 / VB;                      // LDS row in loads
  for (int s = R.v0; s < R.v1; s += NS) {
    __syncthreads();   // the previous stage's fragments are read
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      if constexpr (HALF) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          rx[i][e] = __builtin_amdgcn_alignbit(wx[i].d[e + 1], wx[i].d[e], hx) & mask[e];
          ry[i][e] = __builtin_amdgcn_alignbit(wy[i].d[e + 1], wy[i].d[e], hy) & mask[e];
        }
      }
      Xs[(f0 + NR * i) * LS + slot] = rx[i];
      if (!SAME) Ys[(f0 + NR * i) * LS + slot] = ry[i];
    }
    __syncthreads();
    if (s + NS < R.v1) fetch();
#pragma unroll 1
    for (int g = 0; g < kGrVecs; g += 4) {
      if constexpr (DEAL) {
#pragma unroll
        for (int i0 = 0; i0 < NT; i0 += 3) {
          gr_vec a[3], b[3];
#pragma unroll
          for (int i = 0; i < 3; ++i)
            if (i0 + i < NT) {
              a[i] = xl[tI[i0 + i] + g];       // a wavefront's missing tiles read tile (0, 0)
              b[i] = yl[tJ[i0 + i] + g];
            }
#pragma unroll
          for (int e = 0; e < kGramSteps<PREC>; ++e)
#pragma unroll
            for (int i = 0; i < 3; ++i)
              if (i0 + i < NT && wid + 4 * (i0 + i) < nt) gram_mma<PREC>(a[i], b[i], e, acc[i0 + i]);
        }
      } else {
        const int I0 = (wid >> 1) * WT, J0 = (wid & 1) * WT;
        gr_vec a[WT], b[WT];
#pragma unroll
        for (int i = 0; i < WT; ++i) {
          a[i] = X[(16 * (I0 + i) + li) * kGrStride + g + lq];
          b[i] = Y[(16 * (J0 + i) + li) * kGrStride + g + lq];
        }
#pragma unroll
        for (int e = 0; e < kGramSteps<PREC>; ++e)
#pragma unroll
          for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j)
              if (I0 + i < ntx && J0 + j < nty) gram_mma<PREC>(a[i], b[j], e, acc[i * WT + j]);
      }
    }
  }
  // accumulator of a 16 x 16 tile: lane holds column li; rows 4 lq + e for the FP32 forms,
  // lq + 4 e for v_mfma_f64_16x16x4_f64
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    int I, J;
    if constexpr (DEAL) {
      if (wid + 4 * i >= nt) break;
      I = tI[i] / (16 * kGrStride);
      J = tJ[i] / (16 * kGrStride);
    } else {
      I = (wid >> 1) * WT + i / WT;
      J = (wid & 1) * WT + i % WT;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = 16 * I + (PREC == ELMFB_FP64 ? lq + 4 * e : 4 * lq + e), col = 16 * J + li;
      if (row < R.nx && col < R.ny) put(row, col, acc[i][e]);
    }
  }
}

}  // namespace elmfb
