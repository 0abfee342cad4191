// Weight gradients of 3x3 / stride-1 / pad-1 convolutions, per example (norms, optionally the gradients themselves) or
// summed over examples with their clip factors, on the bf16 matrix units (split_bf16.h).  Kernels in split_wgrad.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

struct SplitWgArgs {
  const float *x, *dy;  // [B][C][H][W], [B][D][H][W]
  int B, C, D, H, W;
  // norm: squared norms, slots[(slot0 + (channel block) * z + (block of output channels)) * slot_stride + b], and the
  // gradients (gstore, null: not wanted) as rows [D][9][C], then the bias gradient
  float *slots; long slot_stride; int slot0;
  float *gstore; long gstride;
  // sum: scale[b] times each example; one partial row per run of ex_per_block examples, in the parameter layout
  const float *scale; float *part; long part_stride;
  int ex_per_block;
};

static inline bool split_wgrad_fits(int H, int W) {
  return (W == 4 && H == 4) || (W == 8 && H == 8) || (W == 16 && H % 4 == 0) || (W == 32 && H % 2 == 0);
}
static inline int split_wgrad_slots(int C, int D) { return ((C + 31) / 32) * ((D + 31) / 32); }
// returns the slots per example that it fills
int split_wgrad_norm(hipStream_t st, const SplitWgArgs &a);
// max_split: partial rows there is room for; returns the number it writes
int split_wgrad_sum(hipStream_t st, SplitWgArgs a, int max_split);
