// mg_arith.h -- FP64 quotients of the cell updates: the bits of a division in about
// half its dependent operations.  A division's scaling for exponents near the
// ends of the range is left out, which the updates' numbers never reach.  Also
// compiled for the host, where they are checked against it.
#pragma once
#include <cmath>
#ifdef __HIP__
#define MGG_HD __host__ __device__ __forceinline__
#else
#define MGG_HD inline
#endif

namespace mgg {

// x / 6: the product with the rounded 1/6 is within an ulp of it, its remainder is
// exact in one fused multiply-add, and the correction's rounding is the
// quotient's (Markstein's theorem).
MGG_HD double sixth(double x) {
  const double q = x * (1.0 / 6.0);
  return std::fma(std::fma(-6.0, q, x), 1.0 / 6.0, q);
}
MGG_HD float sixth(float x) { return x / 6.0f; }

// a / b from rcp(b) = (1 + d)/b, the hardware's reciprocal, |d| < 2^-22: one
// Newton step leaves d^2 < 2^-44, and the exact remainder of the product
// corrects it to far less than a rounding, as above.
template <typename Rcp>
MGG_HD double quotient(double a, double b, Rcp rcp) {
  const double r0 = rcp(b);
  const double r = std::fma(std::fma(-b, r0, 1.0), r0, r0);
  const double q = a * r;
  return std::fma(std::fma(-b, q, a), r, q);
}

}  // namespace mgg
