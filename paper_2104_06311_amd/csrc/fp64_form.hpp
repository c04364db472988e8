// FP64 exponentials and logarithms for symbols whose sums FP32 does not hold.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace md {
namespace fp64 {

constexpr double kLn2 = 0.69314718055994530942;
// 2^f for |f| <= 1/2: twelve terms of the exponential series (the next is 6e-15).
__device__ __forceinline__ double exp2_fraction(double f) {
  // ln(2)^n / n!
  double p = 4.4455382718708101e-10;
  p = fma(p, f, 7.0549116208011209e-09);
  p = fma(p, f, 1.0178086009239696e-07);
  p = fma(p, f, 1.3215486790144305e-06);
  p = fma(p, f, 1.5252733804059838e-05);
  p = fma(p, f, 1.5403530393381606e-04);
  p = fma(p, f, 1.3333558146428441e-03);
  p = fma(p, f, 9.6181291076284769e-03);
  p = fma(p, f, 5.5504108664821576e-02);
  p = fma(p, f, 2.4022650695910069e-01);
  p = fma(p, f, kLn2);
  return fma(p, f, 1.0);
}

// 2^-r, r >= 0, as 2^k e with an integer k and e in [2^-1/2, 2^1/2], so that sums can be taken relative to
// any of their terms; k saturates at -2^30.  e is NaN for NaN.
constexpr double kFar = 1073741824.0;
__device__ __forceinline__ bool saturated(int k) { return k < -1073741820; }
__device__ __forceinline__ void exp2_neg(double r, int* k, double* e) {
  constexpr double kMagic = 6755399441055744.0;           // 1.5 * 2^52: an integer in the low word
  const double t = r > kFar ? -kFar : -r;
  const double s = t + kMagic;
  *k = static_cast<int>(static_cast<uint32_t>(__builtin_bit_cast(uint64_t, s)));
  *e = exp2_fraction(t - (s - kMagic));
}
// 2^-r itself (0 beyond the FP64 range).
__device__ __forceinline__ double exp2_neg(double r) {
  int k;
  double e;
  exp2_neg(r, &k, &e);
  return ldexp(e, k);
}

// ln (a / b) of two positive FP64 numbers by `TERMS` terms of 2 artanh(z), z = (a - b) / (a + b), with
// the ratio brought into (1/2, 2) by a power of two, |z| < 1/3: nine terms leave 1e-10, fifteen 1e-16.
// one_octave: both are in [1, 2].
template <int TERMS, bool one_octave>
__device__ __forceinline__ double log_ratio(double a, double b) {
  int k = 0;
  if constexpr (!one_octave) {
    k = __builtin_amdgcn_frexp_exp(a) - __builtin_amdgcn_frexp_exp(b);
    a = __builtin_amdgcn_frexp_mant(a);
    b = __builtin_amdgcn_frexp_mant(b);
  }
  const double q = a + b;
  double r = __builtin_amdgcn_rcp(q);
  r = fma(r, fma(-q, r, 1.0), r);
  if constexpr (TERMS > 9) r = fma(r, fma(-q, r, 1.0), r);
  const double z = (a - b) * r, w = z * z;
  double p = 2.0 / (2 * TERMS - 1);
#pragma unroll
  for (int n = 2 * TERMS - 3; n >= 1; n -= 2) p = fma(p, w, 2.0 / n);
  return one_octave ? z * p : fma(z, p, k * kLn2);
}

}  // namespace fp64
}  // namespace md
