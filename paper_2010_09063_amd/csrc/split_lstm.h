// Weight gradient of the LSTM layer (Section 1, item 2a): [x_t | h_{t-1} | 1]^T dgates_t over the time steps, a
// (Din + H + 1) x 4H matrix in the layer's parameter layout (W_ih, W_hh, b), per example with its squared norm (item 2b) or
// summed over examples with their clip factors (item 3), on the bf16 matrix units (split_bf16.h).  Kernels in split_lstm.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

struct SplitLstmArgs {
  const float *x;      // [B][T][Din]
  const float *hs;     // [B][T][H]   h_t; step t uses h_{t-1} (zero for t = 0)
  const float *dg;     // [B][T][4H]  gate gradients
  // per example: squared norms, one partial per wave, slots[(slot0 + half * 8 + wave) * slot_stride + b], and the gradient (gstore, null: not wanted)
  float *slots; long slot_stride; int slot0;
  float *gstore; long gstride;
  // sum: scale[b] times each example, one partial row per run of 16-step units
  const float *scale; float *part; long part_stride;
  int B, T, Din, H;
  int units_per_wg;    // (set by the launcher)
};

#define SPLIT_LSTM_SLOTS 16 // per example: 2 halves of the columns x 8 waves
#define SPLIT_LSTM_MB 9     // blocks of 32 rows at most
static inline bool split_lstm_fits(int Din, int H) { return Din >= 1 && H >= 1 && Din + H + 1 <= 32 * SPLIT_LSTM_MB && H <= 128; }
// once per device before the first launch (two buffers of up to 17 blocks exceed the default 64 KB of LDS)
bool split_lstm_enable();
int split_lstm_norm(hipStream_t st, const SplitLstmArgs &a); // returns the slots per example that it fills
int split_lstm_sum(hipStream_t st, SplitLstmArgs a, int max_split); // returns the partial rows that it writes
