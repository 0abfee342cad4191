#include "split_rows.h"

#include <algorithm>
#include <type_traits>

#include "split_bf16.h"

// Weight fragments in the order in which a wave reads them: [k step of 16][block of 32 columns][piece][lane][8], lane
// (column = lane % 32, k half = lane / 32); zero beyond K and N.
__global__ __launch_bounds__(64) void split_weights_kernel(const SplitWeights w0, const SplitWeights w1, int n0) {
  const bool second = (int)blockIdx.x >= n0;
  const float *W = second ? w1.W : w0.W;
  const long sk = second ? w1.sk : w0.sk, sn = second ? w1.sn : w0.sn;
  const int K = second ? w1.K : w0.K, N = second ? w1.N : w0.N;
  const int blk = (int)blockIdx.x - (second ? n0 : 0), nb_tot = (N + 31) / 32;
  const int ks = blk / nb_tot, nb = blk - ks * nb_tot, lane = threadIdx.x;
  const int n = nb * 32 + (lane & 31), k0 = ks * 16 + 8 * (lane >> 5);
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const bool ok = n < N && k0 + j < K;
    v[j] = W[ok ? (k0 + j) * sk + n * sn : 0];
    v[j] = ok ? v[j] : 0.f;
  }
  SbFrag f;
  sb_split8(v, f);
  sb_u32x4 *dst = (sb_u32x4 *)(second ? w1.frag : w0.frag) + (long)blk * 192 + lane;
#pragma unroll
  for (int p = 0; p < 3; ++p) dst[64 * p] = f.p[p];
}

// Persistent workgroups of eight waves, one per CU, walk over tiles of 32 rows; every wave keeps its share of the weights
// in registers, all three pieces, for the whole run.  A tile is split once, on its way into LDS (two buffers,
// [k step][piece][lane][8]: the order in which the matrix instruction takes it), the next tile's rows travel in
// registers meanwhile.  KH = 1: a wave owns columns, blocks w and 15 - w of up to sixteen; KH = 2: four blocks of columns,
// waves w and w + 4 taking a half of the k steps each and adding up through LDS.  (Weights streamed from the L2 instead
// cost a trip per k step or, requested ahead, more registers than two waves per SIMD have: 195 us for the projection, 111
// for the input gradient.)
#define SR_THREADS SPLIT_ROWS_THREADS
template <int KH, int KSW> // k steps per wave at most
__global__ __launch_bounds__(SR_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void split_rows_kernel(const SplitRowsArgs a) {
  constexpr int KST = KH * KSW, ITEMS = (KST * 64 + SR_THREADS - 1) / SR_THREADS, TILE = KST * 3072;
  extern __shared__ __attribute__((aligned(16))) char lds[]; // 2 x TILE
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K, KS = (K + 15) >> 4, nb_tot = (a.N + 31) >> 5;
  const int kh = KH == 1 ? 0 : wave >> 2;
  const long tiles = (a.M + 31) >> 5;

  // staging items: (k half step, row of the tile), rows along the lanes; odd rows with the opposite sign, as far as the
  // accumulators: a token's gradient adds up thousands of them (split_bf16.h)
  const float sign = lane & 1 ? -1.f : 1.f;
  sb_f32x4u raw[ITEMS][2];
  auto fetch = [&](long tile) {
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      const int it = tid + SR_THREADS * q, kk = it >> 5;
      const long row = std::min<long>(tile * 32 + (it & 31), a.M - 1);
      const float *p = a.A + row * a.lda + (8 * kk < K ? 8 * kk : 0);
      raw[q][0] = *reinterpret_cast<const sb_f32x4u *>(p);
      raw[q][1] = *reinterpret_cast<const sb_f32x4u *>(p + 4);
    }
  };
  auto stash = [&](char *buf) {
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      const int it = tid + SR_THREADS * q, kk = it >> 5;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = 8 * kk + j < K ? sign * raw[q][j >> 2][j & 3] : 0.f; // (what lies past K is somebody else's)
      SbFrag f;
      sb_split8(v, f);
      if (kk < 2 * KST) {
        char *dst = buf + (kk >> 1) * 3072 + ((kk & 1) * 32 + (it & 31)) * 16;
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<sb_u32x4 *>(dst + p * 1024) = f.p[p];
      }
    }
  };
  auto run = [&](auto nb_c) { // column blocks of this wave
    constexpr int NB = decltype(nb_c)::value;
    int blk[NB > 0 ? NB : 1];
    blk[0] = KH == 1 ? wave : wave & 3;
    if constexpr (NB > 1) blk[1] = 15 - wave;
    SbFrag w[KSW][NB > 0 ? NB : 1];
    float bv[NB > 0 ? NB : 1];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
#pragma unroll
      for (int s = 0; s < KSW; ++s) {
        const int ks = min(kh * KSW + s, KS - 1); // (past the last one: multiplied by zeros)
        const sb_u32x4 *f = (const sb_u32x4 *)a.frag + ((long)ks * nb_tot + blk[j]) * 192 + lane;
#pragma unroll
        for (int p = 0; p < 3; ++p) w[s][j].p[p] = f[64 * p];
      }
      const int n = blk[j] * 32 + li;
      bv[j] = a.bias != nullptr && n < a.N ? a.bias[n] : 0.f;
    }
    int b = 0;
    if (blockIdx.x < tiles) fetch(blockIdx.x);
    for (long tile = blockIdx.x; tile < tiles; tile += gridDim.x, b ^= 1) {
      char *buf = lds + b * TILE;
      stash(buf);
      __syncthreads(); // this tile is staged; the buffer before is free once its readers have come here
      fetch(std::min(tile + gridDim.x, tiles - 1)); // (past the last one: read again, unused)
      __builtin_amdgcn_sched_barrier(0);
      sb_f32x16 acc[1][NB > 0 ? NB : 1];
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][j][r] = 0.f;
      if constexpr (NB > 0) {
        SbFrag x[2][1]; // one k step ahead (further ahead there are no registers left)
        auto operand = [&](int s, int pieces) {
#pragma unroll
          for (int p = 0; p < pieces; ++p)
            x[s & 1][0].p[p] = *reinterpret_cast<const sb_u32x4 *>(buf + (kh * KSW + s) * 3072 + p * 1024 + lane * 16);
        };
        operand(0, 3);
#pragma unroll
        for (int s = 0; s < KSW; ++s) {
          if (s + 1 < KSW) operand(s + 1, 3);
          __builtin_amdgcn_sched_barrier(0);
          sb_products<0, 5>(x[s & 1], w[s], acc);
        }
        operand(0, 1); // the leading pieces again, for the large products
#pragma unroll
        for (int s = 0; s < KSW; ++s) {
          if (s + 1 < KSW) operand(s + 1, 1);
          __builtin_amdgcn_sched_barrier(0);
          sb_products<5, 6>(x[s & 1], w[s], acc);
        }
      }
      if constexpr (KH == 2) { // the second half's sums meet the first's in the buffer that was just read
        __syncthreads();
        if (NB > 0 && kh == 1) {
#pragma unroll
          for (int r = 0; r < 16; ++r) *reinterpret_cast<float *>(buf + (((wave & 3) * 16 + r) * 64 + lane) * 4) = acc[0][0][r];
        }
        __syncthreads();
        if (NB > 0 && kh == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[0][0][r] += *reinterpret_cast<const float *>(buf + (((wave & 3) * 16 + r) * 64 + lane) * 4);
        }
      }
      if (kh == 0) {
        const unsigned lane_off = 4u * (4u * lk * (unsigned)a.ldc + li);
        const int rows_left = (int)std::min<long>(32, a.M - tile * 32) - 4 * lk;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          float *cj = a.C + tile * 32 * a.ldc + blk[j] * 32; // (uniform)
          const bool in = blk[j] * 32 + li < a.N;
#pragma unroll
          for (int r = 0; r < 16; ++r) { // accumulator register r of a lane: row 8 (r / 4) + 4 lk + r % 4, column li
            const int ru = 8 * (r >> 2) + (r & 3);
            if (in && ru < rows_left)
              *reinterpret_cast<float *>(reinterpret_cast<char *>(cj + ru * a.ldc) + lane_off) = r & 1 ? bv[j] - acc[0][j][r] : bv[j] + acc[0][j][r];
          }
        }
      }
    }
  };
  if constexpr (KH == 1) {
    if (15 - wave < nb_tot) run(std::integral_constant<int, 2>{});
    else if (wave < nb_tot) run(std::integral_constant<int, 1>{});
    else run(std::integral_constant<int, 0>{});
  } else {
    if ((wave & 3) < nb_tot) run(std::integral_constant<int, 1>{});
    else run(std::integral_constant<int, 0>{});
  }
}

void split_rows_prepare(hipStream_t st, const SplitWeights *w, int n) {
  auto blocks = [](const SplitWeights &s) { return ((s.K + 15) / 16) * ((s.N + 31) / 32); };
  const int n0 = blocks(w[0]), n1 = n > 1 ? blocks(w[1]) : 0;
  hipLaunchKernelGGL(split_weights_kernel, dim3(n0 + n1), dim3(64), 0, st, w[0], n > 1 ? w[1] : w[0], n0);
}

template <int KH, int KSW>
static void launch_one(hipStream_t st, const SplitRowsArgs &a) {
  const size_t lds = 2 * (size_t)KH * KSW * 3072;
  const long tiles = (a.M + 31) / 32;
  hipLaunchKernelGGL((split_rows_kernel<KH, KSW>), dim3((unsigned)std::min<long>(tiles, 256)), dim3(SR_THREADS), lds, st, a);
}

bool split_rows_enable() {
  const hipFuncAttribute at = hipFuncAttributeMaxDynamicSharedMemorySize;
  return hipFuncSetAttribute((const void *)split_rows_kernel<2, 7>, at, 2 * 14 * 3072) == hipSuccess &&
         hipFuncSetAttribute((const void *)split_rows_kernel<2, 10>, at, 2 * 20 * 3072) == hipSuccess &&
         hipFuncSetAttribute((const void *)split_rows_kernel<2, 13>, at, 2 * 26 * 3072) == hipSuccess;
}

void split_rows_launch(hipStream_t st, const SplitRowsArgs &a) {
  const int ks = (a.K + 15) / 16;
  if (a.K <= SPLIT_ROWS_K1) {
    if (ks <= 4) launch_one<1, 4>(st, a);
    else if (ks <= 6) launch_one<1, 6>(st, a);
    else launch_one<1, 7>(st, a);
  } else {
    if (ks <= 14) launch_one<2, 7>(st, a);
    else if (ks <= 20) launch_one<2, 10>(st, a);
    else launch_one<2, 13>(st, a);
  }
}
