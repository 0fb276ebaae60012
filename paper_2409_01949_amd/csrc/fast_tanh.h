// FP64 tanh for the feature kernels: a table of tanh(i/32) and the addition theorem.
//
// With a = |x|, i = round(32 a), b = a - i/32 (exact, |b| <= 1/64), T = tanh(i/32), t = tanh(b):
//   tanh(a) = (T + t) / (1 + T t) = T + t - T t (T + t) / (1 + T t),
// the last form because all but T and b in it is small: T + b is added without error, so one
// rounding of size remains; t from its odd series up to b^7 (the next term is below 1e-16 of t and is folded into the last
// coefficient), 1/(1 + q) = (1 - q + q^2)(1 - q^3 + q^6) up to q^9 < 2^-54 of a term that is
// itself at most 2^-6.  T is held as a sum of two doubles; |x| < 1/64 has T = 0 and returns the series.
// Above 19.0625 tanh rounds to 1.  Error against 80-bit tanh over 2e6 values in each of (-0.02,
// 0.02) to (-25, 25): at most 0.60 ulp, 0.289 rms (a correct rounding's rms is 0.2887); the device
// library's tanh has up to 0.86 and 0.29 to 0.31.
// 26 FP64 instructions and one 16-byte LDS read, where the device library's tanh takes about 100
// instruction slots: the feature kernels are bound by instruction issue.
#pragma once

#include "common.h"

namespace elmfb {

constexpr int kTanhN = 611;            // i = 0 .. 610: up to 19.0625
constexpr double kTanhMax = 19.0625;

// tanh(i/32) as hi + lo, computed at compile time in double-double arithmetic (Dekker 1971):
// E = exp(1/16)^i, tanh = (E - 1) / (E + 1).
struct DD { double h, l; };
constexpr DD dd_fast(double a, double b) {
  const double s = a + b;
  return DD{s, b - (s - a)};
}
constexpr DD dd_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return DD{s, (a - (s - t)) + (b - t)};
}
constexpr DD dd_prod(double a, double b) {
  const double ca = 134217729.0 * a, cb = 134217729.0 * b;
  const double ah = ca - (ca - a), al = a - ah, bh = cb - (cb - b), bl = b - bh;
  const double p = a * b;
  return DD{p, ((ah * bh - p) + ah * bl + al * bh) + al * bl};
}
constexpr DD dd_add(DD a, DD b) {
  const DD s = dd_sum(a.h, b.h);
  return dd_fast(s.h, s.l + (a.l + b.l));
}
constexpr DD dd_mul(DD a, DD b) {
  const DD p = dd_prod(a.h, b.h);
  return dd_fast(p.h, p.l + (a.h * b.l + a.l * b.h));
}
constexpr DD dd_div(DD a, DD b) {
  const double q = a.h / b.h;
  const DD r = dd_add(a, dd_mul(DD{-q, 0.0}, b));
  return dd_add(DD{q, 0.0}, DD{(r.h + r.l) / b.h, 0.0});
}

struct alignas(16) TanhTable {
  double v[kTanhN][2];
  constexpr TanhTable() : v() {
    DD e1{1.0, 0.0}, term{1.0, 0.0};
    for (int n = 1; n < 22; ++n) {     // exp(1/16)
      term = dd_div(dd_mul(term, DD{0.0625, 0.0}), DD{(double)n, 0.0});
      e1 = dd_add(e1, term);
    }
    DD e{1.0, 0.0};
    for (int i = 0; i < kTanhN; ++i) {
      const DD t = dd_div(dd_add(e, DD{-1.0, 0.0}), dd_add(e, DD{1.0, 0.0}));
      v[i][0] = t.h;
      v[i][1] = t.l;
      e = dd_mul(e, e1);
    }
  }
};

// tab: the table (LDS on the device), kTanhN pairs.
__host__ __device__ __forceinline__ double table_tanh(double x, const double2* tab) {
  constexpr double kMagic = 6755399441055744.0;   // 1.5 2^52: the sum's low word is the integer
  double a = __builtin_fabs(x);
  a = a > kTanhMax ? kTanhMax : a;                // NaN stays
  const double s = __builtin_fma(a, 32.0, kMagic);
  uint64_t bits;
  __builtin_memcpy(&bits, &s, 8);
  uint32_t i = (uint32_t)bits;
  i = i < (uint32_t)(kTanhN - 1) ? i : (uint32_t)(kTanhN - 1);
  const double2 T = tab[i];
  const double b = __builtin_fma(s - kMagic, -0.03125, a);
  const double b2 = b * b;
  double p = __builtin_fma(b2, -0.05396372, 2.0 / 15.0);   // -17/315 + (62/2835) 0.85 / 64^2
  p = __builtin_fma(b2, p, -1.0 / 3.0);
  const double b3 = b * b2 * p;                   // t - b
  const double t = b + b3;
  const double q = T.x * t, q2 = q * q;
  const double q3 = q * q2;
  double r = (1.0 - q) + q2;
  r = __builtin_fma(r, __builtin_fma(q3, q3, -q3), r);
  // tanh(a) = T + b + e, the sum T + b kept exactly as hi + lo (|b| <= T or T = 0)
  const double e = __builtin_fma(-(q * (T.x + t)), r, b3) + T.y;
  const double hi = T.x + b;
  const double lo = (T.x - hi) + b;
  return __builtin_copysign(hi + (lo + e), x);
}

#ifdef __HIPCC__
// The table in device memory and its copy into a workgroup's LDS (kTanhN double2; the caller
// synchronises before the first use).
static __device__ const TanhTable kTanhTable{};

__device__ __forceinline__ void stage_tanh(double2* lds) {
  for (int i = threadIdx.x; i < kTanhN; i += blockDim.x)
    lds[i] = double2{kTanhTable.v[i][0], kTanhTable.v[i][1]};
}
#endif

}  // namespace elmfb
