// Chebyshev nodes of the tile expansions and the matrices that turn values at
// the nodes into coefficients.
#pragma once
#include <hip/hip_runtime.h>

#include "far_nodes.h"

namespace xs {

template <int P>
struct FarNodes;
template <>
struct FarNodes<6> {
  static constexpr double x[6] = XS_FAR_X6;
};
template <>
struct FarNodes<12> {
  static constexpr double x[12] = XS_FAR_X12;
};
template <>
struct FarNodes<20> {
  static constexpr double x[20] = XS_FAR_X20;
};
static __device__ const double kFarD6[6 * 6] = XS_FAR_D6;
static __device__ const double kFarD12[12 * 12] = XS_FAR_D12;
static __device__ const double kFarD20[20 * 20] = XS_FAR_D20;
template <int P>
__device__ __forceinline__ const double* far_dct() {
  if constexpr (P == 6) return kFarD6;
  else if constexpr (P == 12) return kFarD12;
  else return kFarD20;
}

// the nodes in memory, for loops over them
static __device__ const float kFarX6f[6] = XS_FAR_X6;
static __device__ const float kFarX12f[12] = XS_FAR_X12;
static __device__ const double kFarX12d[12] = XS_FAR_X12;
static __device__ const double kFarX20d[20] = XS_FAR_X20;
template <typename R, int P>
__device__ __forceinline__ const R* far_x() {
  if constexpr (sizeof(R) == 4) return P == 6 ? kFarX6f : kFarX12f;
  else return P == 12 ? kFarX12d : kFarX20d;
}

}  // namespace xs
