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
  // sum: scale[b] times each example; one partial row per run of bands of rows (4-wide planes: of examples), in the parameter layout
  const float *scale; float *part; long part_stride;
  int bands_per_block; // (set by the launcher)
};

static inline bool split_wgrad_fits(int H, int W) {
  return (W == 4 && H == 4) || (W == 8 && H == 8) || (W == 16 && H % 4 == 0) || (W == 32 && H % 2 == 0);
}
// Per-example gradients, planes wider than 4: two blocks of output channels per workgroup share its input rows, where that
// wastes none and leaves the chip two workgroups per CU.
static inline bool split_wgrad_pairs(int B, int C, int D) {
  const int cb = (C + 31) / 32, db = (D + 31) / 32;
  return db % 2 == 0 && (long)B * cb * (db / 2) >= 512;
}
// Norms on 8x8 planes: whether this kernel is ahead of the one that forms Gram matrices (conv_gram.h), whose workgroup of
// one example takes a time that is flat up to a round of 256 and linear in 9 C + D, while this one's is linear in the blocks.
// Fitted to us, Gram and this (C -> D channels: at 64, 96, 128, 160, 256 examples):
//    64 -> 128   19 13   20 17   20 17   20 22   21 28
//    96 ->  96   23 17   23 20   24 24   24 28   25 40
//   128 -> 128   29 17   29 23   29 28   30 33   31 45
//    96 -> 192   26 22   26 27   26 31   26 36   27 50
//   192 -> 192   40 31   40 40   41 50   40 62   41 91
//   256 -> 256   52 46   52 63   52 81   52 100  53 153   (80 examples: 52 and 55)
static inline bool split_wgrad_beats_gram(int B, int C, int D) {
  if (B > 256) return false; // (not measured)
  const float blocks = (float)((long)B * ((C + 31) / 32) * ((D + 31) / 32));
  const float mine = !split_wgrad_pairs(B, C, D) ? 8.f + 0.0137f * blocks : blocks <= 1024.f ? 17.f : 10.5f + 0.0087f * blocks;
  return mine < 7.f + 0.0176f * (9.f * C + D);
}
// returns the slots per example that it fills
int split_wgrad_norm(hipStream_t st, const SplitWgArgs &a);
// max_split: partial rows there is room for; returns the number it writes
int split_wgrad_sum(hipStream_t st, SplitWgArgs a, int max_split);
