// Launch arguments of the smooth (soft-min) sweeps (wf_soft.hip), shared with the host entry
// points (wf_api.hip).  Nothing here is part of the public ABI (include/wf.h).
#pragma once

#include "wf_internal.h"

namespace wf {

// Arguments of the smooth (soft-min) adjoint: it reads C and the forward's D (Din) and
// writes gC.  (The forward takes the min-plus forward's FwdArgs.)  kx = log2(e) / gamma (the
// weights as base-2 exponentials).
struct SoftArgs {
  const void* C;
  const void* Din;
  const void* gD;       // may be null (zero)
  const void* gscore;   // may be null (zero)
  void* gC;
  int64_t ldc, ldd, ldgd, ldgc;
  int64_t m, n;
  int32_t nb;           // 64-row bands
  int32_t pad;
  double kx;
  Control* ctl;
  uint64_t* bnd;        // adjoint: (nb-1) * n * W words, the last row of each band
};
hipError_t launch_soft_backward(int dtype, const SoftArgs& a, int grid, hipStream_t s);
// The soft-min forward runs in the min-plus forward's band pipeline (wf_fwd.hip) with the
// soft-min cell: a.kx, a.gl set, no checkpoint grid.
hipError_t launch_forward_soft(int dtype, const FwdArgs& a, int grid, hipStream_t s);

// Base-2 exponential and fused multiply-add of the adjoint's weights, in the element type.
// float: the hardware function (v_exp_f32, about one ulp); an exponential that would be
// subnormal (a weight below 2^-126) reads as 0, which changes no sum it enters.
template <typename T>
struct SoftMath;
template <>
struct SoftMath<float> {
  __device__ static __forceinline__ float exp2_(float x) { return __builtin_amdgcn_exp2f(x); }
  __device__ static __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
};
template <>
struct SoftMath<double> {
  __device__ static __forceinline__ double exp2_(double x) { return exp2(x); }
  __device__ static __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
};

}  // namespace wf
