// FP64 powers of two for device code.
#pragma once

#include "fgl_internal.h"

namespace fgl {

// FP64 powers of the plain-FP64, thin, gradient and chain kernels: 2^(y/64)
// for |y| < 2^31 as 2^floor(j/64) (ldexp) times 2^((j mod 64)/64) from the
// 64-entry LDS table t64 times 2^(r/64), j = round(y), |r| <= 1/2, by its
// Taylor series to fifth order (truncation below 4e-17 relative).
__device__ inline void init_t64(double* t64) {
  if (threadIdx.x < 64) t64[threadIdx.x] = exp2((double)threadIdx.x * (1.0 / 64.0));
}
__device__ inline double pow2_64(double y, const double* t64, const DevModel& m) {
  const double MAGIC = 0x1.8p52;                  // rint via the low word
  const double t = y + MAGIC;
  const int j = (int)(uint32_t)__double_as_longlong(t);
  const double r = y - (t - MAGIC);               // |r| <= 1/2
  double p = fma(r, m.c5, m.c4);
  p = fma(r, p, m.c3);
  p = fma(r, p, m.c2);
  p = fma(r, p, m.c1);
  p = fma(r, p, 1.0);
  return ldexp(t64[j & 63] * p, j >> 6);
}

}  // namespace fgl
