// Helpers of the adjoint kernels: derivatives of the shifted softplus.
#pragma once
#include "mfma_gemm.h"
#include "pn_internal.h"

namespace pn {

// first three derivatives of ssp: s, s (1 - s), s (1 - s) (1 - 2 s), s = sigmoid(u)
template <typename TN>
__device__ __forceinline__ TN sig(TN u) {
  return sigmoid_d(u);
}
template <typename TN>
__device__ __forceinline__ TN ssp2(TN u) {
  const TN s = sigmoid_d(u);
  return s * (TN(1) - s);
}
template <typename TN>
__device__ __forceinline__ TN ssp3(TN u) {
  const TN s = sigmoid_d(u);
  return s * (TN(1) - s) * (TN(1) - TN(2) * s);
}

}  // namespace pn
