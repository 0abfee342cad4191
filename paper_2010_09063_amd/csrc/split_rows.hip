#include "split_rows.h"

#include <algorithm>
#include <type_traits>

#include "split_bf16.h"

// Weight fragments in the order in which a wave reads them: [k step of 16][block of 32 columns][piece][lane][8], lane
// (column = lane % 32, k half = lane / 32); zero beyond K and N.
__global__ __launch_bounds__(64) void split_weights_kernel(const SplitWeights w0, const SplitWeights w1, int n0) {
  const bool second = (int)blockIdx.x >= n0;
  const SplitWeights &w = second ? w1 : w0;
  const int blk = (int)blockIdx.x - (second ? n0 : 0), nb_tot = (w.N + 31) / 32;
  const int ks = blk / nb_tot, nb = blk - ks * nb_tot, lane = threadIdx.x;
  const int n = nb * 32 + (lane & 31), k0 = ks * 16 + 8 * (lane >> 5);
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const bool ok = n < w.N && k0 + j < w.K;
    v[j] = w.W[ok ? (k0 + j) * w.sk + n * w.sn : 0];
    v[j] = ok ? v[j] : 0.f;
  }
  SbFrag f;
  sb_split8(v, f);
  sb_u32x4 *dst = (sb_u32x4 *)w.frag + (long)blk * 192 + lane;
#pragma unroll
  for (int p = 0; p < 3; ++p) dst[64 * p] = f.p[p];
}

// No LDS: a wave owns 32 MB rows and up to four blocks of 32 columns; it reads its rows straight from memory (a lane's
// eight consecutive k are two 16-byte loads), splits them in registers and takes the weight fragments from the L2,
// where its workgroup's four waves read the same ones.  Rows are requested two k steps ahead, fragments one.
// MB = 2 halves the fragment traffic per multiply; MB = 1 and fewer columns per wave where the rows would not fill
// the chip.  The LSTM's input gradient, 131,072 x 100 x 400: 133 us on the fp32 instruction, 112 here; 32,768 rows: 43
// and 33.  (Its input projection, x 400 x 100, is not: four groups of columns each split the rows again and the 7 k
// steps do not cover a wave's prologue and its stores: 195 us against 120 for the kernel that keeps the weights.)
template <int MB, int NB>
__device__ __forceinline__ void split_rows_body(const SplitRowsArgs &a, long row0, int nb0, int nb_tot) {
  const int lane = threadIdx.x & 63, li = lane & 31, lk = lane >> 5;
  const int K = a.K, KS = (K + 15) / 16;
  const float *rows[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) rows[i] = a.A + std::min<long>(row0 + 32 * i + li, a.M - 1) * a.lda + 8 * lk;
  const sb_u32x4 *fr = (const sb_u32x4 *)a.frag + (long)nb0 * 192 + lane;
  const long fstep = (long)nb_tot * 192;
  sb_f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  sb_f32x4u r0[MB][2], r1[MB][2];
  auto fetch = [&](int ks, sb_f32x4u (&r)[MB][2]) {
    const int kc = min(ks, KS - 1) * 16;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      r[i][0] = *reinterpret_cast<const sb_f32x4u *>(rows[i] + kc);
      r[i][1] = *reinterpret_cast<const sb_f32x4u *>(rows[i] + kc + 4);
    }
  };
  auto weights = [&](int ks, SbFrag (&w)[NB]) {
    const sb_u32x4 *f = fr + min(ks, KS - 1) * fstep;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int p = 0; p < 3; ++p) w[j].p[p] = f[j * 192 + p * 64];
  };
  SbFrag w0[NB], w1[NB];
  // one k step: the rows two steps ahead and the next fragments are requested before its multiplies (the scheduling
  // barriers keep them there: left alone the compiler sinks each load to its use, one trip to the L2 per step)
  auto step = [&](auto last, int ks, sb_f32x4u (&r)[MB][2], SbFrag (&w)[NB], SbFrag (&w_next)[NB]) {
    SbFrag x[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = r[i][j >> 2][j & 3];
      if (decltype(last)::value) { // (what lies past K is somebody else's)
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = ks * 16 + 8 * lk + j < K ? v[j] : 0.f;
      }
      sb_split8(v, x[i]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!decltype(last)::value) {
      weights(ks + 1, w_next);
      fetch(ks + 2, r);
    }
    __builtin_amdgcn_sched_barrier(0);
    sb_mfma(x, w, acc);
  };
  fetch(0, r0);
  weights(0, w0);
  fetch(1, r1);
  // (the last step apart: a branch in the loop would wait for everything in flight where its paths join)
  int ks = 0;
  for (; ks + 2 < KS; ks += 2) {
    step(std::false_type{}, ks, r0, w0, w1);
    step(std::false_type{}, ks + 1, r1, w1, w0);
  }
  if (ks + 2 == KS) {
    step(std::false_type{}, ks, r0, w0, w1);
    step(std::true_type{}, ks + 1, r1, w1, w0);
  } else {
    step(std::true_type{}, ks, r0, w0, w1);
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int n = (nb0 + j) * 32 + li;
    const float bv = a.bias != nullptr && n < a.N ? a.bias[n] : 0.f;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) { // accumulator register r of a lane: row 8 (r / 4) + 4 lk + r % 4, column li
        const long row = row0 + 32 * i + 8 * (r >> 2) + 4 * lk + (r & 3);
        if (row < a.M && n < a.N) a.C[row * a.ldc + n] = acc[i][j][r] + bv;
      }
  }
}

template <int MB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void split_rows_kernel(const SplitRowsArgs a, int nb_tot) {
  const long row0 = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * (32 * MB);
  if (row0 >= a.M) return;
  // the column blocks dealt evenly to the groups: 13 over 4 are 4, 3, 3, 3
  const int g = blockIdx.y, n_g = gridDim.y, base = nb_tot / n_g, rem = nb_tot - base * n_g;
  const int nb = base + (g < rem ? 1 : 0), nb0 = g * base + min(g, rem);
  if (nb == 4) split_rows_body<MB, 4>(a, row0, nb0, nb_tot);
  else if (nb == 3) split_rows_body<MB, 3>(a, row0, nb0, nb_tot);
  else if (nb == 2) split_rows_body<MB, 2>(a, row0, nb0, nb_tot);
  else if (nb == 1) split_rows_body<MB, 1>(a, row0, nb0, nb_tot);
}

void split_rows_prepare(hipStream_t st, const SplitWeights *w, int n) {
  auto blocks = [](const SplitWeights &s) { return ((s.K + 15) / 16) * ((s.N + 31) / 32); };
  const int n0 = blocks(w[0]), n1 = n > 1 ? blocks(w[1]) : 0;
  hipLaunchKernelGGL(split_weights_kernel, dim3(n0 + n1), dim3(64), 0, st, w[0], n > 1 ? w[1] : w[0], n0);
}

void split_rows_launch(hipStream_t st, const SplitRowsArgs &a) {
  const int nb_tot = (a.N + 31) / 32;
  int groups = (nb_tot + 3) / 4;
  // 64 rows per wave once that gives every SIMD (1024) a wave; otherwise 32, and fewer columns per wave until it does
  const long w64 = (a.M + 63) / 64, w32 = (a.M + 31) / 32;
  if (w64 * groups >= 2048) {
    dim3 grid((unsigned)((w64 + 3) / 4), groups);
    hipLaunchKernelGGL(split_rows_kernel<2>, grid, dim3(256), 0, st, a, nb_tot);
    return;
  }
  while (groups < nb_tot && w32 * groups < 1024) groups = std::min(nb_tot, groups * 2);
  dim3 grid((unsigned)((w32 + 3) / 4), groups);
  hipLaunchKernelGGL(split_rows_kernel<1>, grid, dim3(256), 0, st, a, nb_tot);
}
