// reduce.h -- what the FP64 reductions of 2-D and 3-D domains share.
#pragma once

#include "nplbm_internal.h"

namespace nplbm {

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Threads of a reduction workgroup.
constexpr int kReduceThreads = 256;

// Combine a block's per-thread accumulators into its partial record:
// entry qmax is a maximum, the others are sums.
template <int Q>
__device__ __forceinline__ void block_record(const double (&acc)[Q], int qmax, double *rec) {
  __shared__ double red[kReduceThreads / 64][Q];
  const int wv = threadIdx.x / 64, ln = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const double r = (q == qmax) ? wave_max(acc[q]) : wave_sum(acc[q]);
    if (ln == 0) red[wv][q] = r;
  }
  __syncthreads();
  const int q = threadIdx.x;
  if (q < Q) {
    double r = red[0][q];
    for (int w = 1; w < kReduceThreads / 64; ++w) r = (q == qmax) ? fmax(r, red[w][q]) : r + red[w][q];
    rec[q] = r;
  }
}

// c_k of a node (eq:N18)
template <int M>
__device__ __forceinline__ double c_of(const Consts<double> &K, int k, const double (&ph)[M]) {
  double ck = K.ca[k];
#pragma unroll
  for (int i = 0; i < M; ++i) ck += K.cA[k][i] * ph[i];
  return ck;
}

// Add one node to the conservation accumulators: the c_k, max |sum c_k - 1|,
// nodes with a non-finite c_k.
template <int M>
__device__ __forceinline__ void diag_add(const Consts<double> &K, const double (&ph)[M],
                                         double (&acc)[M + 3]) {
  double s = 0.0;
  bool bad = false;
#pragma unroll
  for (int k = 0; k <= M; ++k) {
    const double v = c_of<M>(K, k, ph);
    bad |= !isfinite(v);
    acc[k] += v;
    s += v;
  }
  acc[M + 1] = fmax(acc[M + 1], fabs(s - 1.0));
  acc[M + 2] += bad ? 1.0 : 0.0;
}

}  // namespace nplbm
