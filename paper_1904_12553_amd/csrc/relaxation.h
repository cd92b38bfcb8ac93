// relaxation.h -- the NS relaxation of one node, shared by the 2-D and 3-D
// steps.
#pragma once

#include <hip/hip_runtime.h>

namespace nplbm {

// tau_g = 1/2 + mu / (rho c_s^2)  (eq:N21_1 with nu = mu / rho): 1 / tau_g, 1 -
// 1 / (2 tau_g) and the reciprocal of tau_g - 1/2.  A division each: with one
// reciprocal for both, and a product with 1 / rho in place of the first
// division, the worst errors over mu / rho = 1e-4 .. 10 are 4.4 and 4.3 units
// of 2^-53 instead of 2.9 and 2.5, for times that differ by less than 0.5%
// (777 x 513 N = 4 FP64 58.84 against 58.92 us a step, 192^3 N = 3 FP32 702 against
// 704, 100 x 84 x 60 N = 4 FP64 168.5 against 168.1).
__host__ __device__ __forceinline__ void ns_relaxation(double mu, double rho, double &itau,
                                                       double &srcg, double &theta) {
  const double tm = 3.0 * mu / rho;
  itau = 1.0 / (0.5 + tm);
  srcg = 1.0 - 0.5 * itau;
  theta = 1.0 / tm;
}

}  // namespace nplbm
