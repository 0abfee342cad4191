// C[M x N] = A[M x K] W (+ bias): one row per (example, step), a weight matrix that every row shares -- the LSTM's input
// projection and the gradient of its input -- on the bf16 matrix units (split_bf16.h).  Kernels in split_rows.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

struct SplitRowsArgs {
  const float *A; long lda;  // rows of A; reads run up to SPLIT_ROWS_SLACK floats past the end of the last row
  const void *frag;          // the split weights (split_rows_prepare)
  const float *bias;         // [N] or null
  float *C; long ldc;
  long M;
  int K, N;
};
struct SplitWeights { // element (k, n) = W[k * sk + n * sn]
  const float *W; long sk, sn;
  int K, N;
  void *frag;
};

#define SPLIT_ROWS_SLACK 16
#define SPLIT_ROWS_THREADS 512
#define SPLIT_ROWS_K1 112 // up to here a wave holds all of K for two blocks of columns
static inline size_t split_rows_frag_bytes(int K, int N) { return (size_t)((K + 15) / 16) * ((N + 31) / 32) * 3 * 1024; }
// K to 112 with N to 512 (two blocks of 32 columns per wave), or K to 416 with N to 128 (half of K per wave)
static inline bool split_rows_fits(int K, int N) { return (K <= SPLIT_ROWS_K1 && N <= 512) || (K <= 416 && N <= 128); }

// once per device before the first launch with K > SPLIT_ROWS_K1 (two tiles of up to 26 k steps exceed the default 64 KB of LDS)
bool split_rows_enable();
// splits up to two weight matrices in one launch
void split_rows_prepare(hipStream_t st, const SplitWeights *w, int n);
void split_rows_launch(hipStream_t st, const SplitRowsArgs &a);
