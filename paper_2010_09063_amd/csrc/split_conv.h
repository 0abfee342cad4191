// Forward and backward-data of 3x3 / stride-1 / pad-1 convolutions in direct form on the bf16 matrix units
// (split_bf16.h).  Kernels in split_conv.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

struct SplitConvArgs {
  const float *x;      // [B][Cin][H][W]
  const void *frag;    // split weights (conv_fragments)
  const float *bias;   // [M]: forward; null: backward-data
  const float *a_prev; // backward-data through an activation: its output, [B][M][H][W]
  float *out;          // [B][M][H][W]; not written with a fused max-pool
  float *pool_out; uint8_t *pool_arg; // 2x2 / stride-2 pool after a forward pass: [B][M][H/2][W/2], the maximum's place
  int B, Cin, M, H, W, act;
  int pool;            // 0: none, 1: max, 2: mean
  const float *w;      // two fp16 pieces only: the layer's weights as they are, [M][Cin][9] (backward-data: [Cin][M][9])
};

#define SPLIT_CONV_MAX 32
struct SplitConvWeights {
  struct { long w_off; void *frag; int D, C, flip, f16; } l[SPLIT_CONV_MAX]; // flip: backward-data (rows = C, k = D); f16: for conv_f16.hip
  int n;
};

// planes the kernel is built for: 4, 8, 16 or 32 wide; the 64 pixels of a wave are whole pairs of rows of one image, or
// whole images of at least four rows
static inline bool split_conv_fits(int H, int W) {
  if (W != 4 && W != 8 && W != 16 && W != 32) return false;
  const int rows = 64 / W;
  return H >= 4 && (H & 1) == 0 && (H % rows == 0 || rows % H == 0);
}
static inline size_t split_conv_frag_bytes(int M, int Cin) { return (size_t)((Cin + 15) / 16) * 9 * ((M + 31) / 32) * 3 * 1024; }

void split_conv_launch(hipStream_t st, const SplitConvArgs &a);
