// Activations and their derivatives, as the kernels' epilogues apply them.
#pragma once
#include <hip/hip_runtime.h>

#define DP_ACT_NONE_ 0
#define DP_ACT_RELU_ 1
#define DP_ACT_TANH_ 2

// tanh and the logistic function from one hardware exp2 and one hardware reciprocal
// (v_exp_f32, v_rcp_f32: about 1 ulp each).  Absolute error is at the 1e-7 level, the same
// size as fp32 rounding of the result, far inside the 1e-4 bar on the aggregated gradient;
// the library versions cost several times the MFMA time of a small tile's epilogue.
__device__ __forceinline__ float fast_tanh(float x) {
  const float t = __builtin_amdgcn_exp2f(-2.885390081777927f * fabsf(x)); // exp(-2|x|)
  const float r = (1.f - t) * __builtin_amdgcn_rcpf(1.f + t);
  return copysignf(r, x);
}
__device__ __forceinline__ float fast_sigmoid(float x) {
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}

__device__ __forceinline__ float act_apply(int act, float z) {
  if (act == DP_ACT_RELU_) return z > 0.f ? z : 0.f;
  if (act == DP_ACT_TANH_) return fast_tanh(z);
  return z;
}
// derivative expressed through the activation's output a = act(z)
__device__ __forceinline__ float act_deriv_from_out(int act, float a) {
  if (act == DP_ACT_RELU_) return a > 0.f ? 1.f : 0.f;
  if (act == DP_ACT_TANH_) return 1.f - a * a;
  return 1.f;
}
// lanes swap within pairs: the other column of a 2x2 pool's window
__device__ __forceinline__ float swap1(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
}
