// relaxation.h -- the NS relaxation of one node, shared by the 2-D and 3-D
// steps.
#pragma once

#include <hip/hip_runtime.h>

namespace nplbm {

// tau_g = 1/2 + mu / (rho c_s^2)  (eq:N21_1 with nu = mu / rho): 1 / tau_g, 1 -
// 1 / (2 tau_g) and the reciprocal of tau_g - 1/2.  irho = 1 / rho: 3 mu / rho is
// its product corrected by the remainder, as exact as a division; the two
// reciprocals take a division each.  Without the correction, and with one
// reciprocal for both, the worst errors over mu / rho = 1e-4 .. 10 are 4.4 and
// 4.3 units of 2^-53 instead of 2.9 and 2.5, for times that differ by less than
// 1% (777 x 513 N = 4 FP64 58.84 against 58.89 us a step, 1504 x 1400 N = 5 FP32
// 187.9 / 188.2, N = 8 FP64 mixed 748.6 / 748.2, 192^3 N = 3 FP32 702 / 704).  A
// division in place of the correction costs N = 8 FP64 mixed, at the end of
// its registers, a tenth (822).
__host__ __device__ __forceinline__ void ns_relaxation(double mu, double rho, double irho,
                                                       double &itau, double &srcg,
                                                       double &theta) {
  const double m3 = 3.0 * mu, t0 = m3 * irho;
  const double tm = __builtin_fma(__builtin_fma(-rho, t0, m3), irho, t0);
  itau = 1.0 / (0.5 + tm);
  srcg = 1.0 - 0.5 * itau;
  theta = 1.0 / tm;
}

}  // namespace nplbm
