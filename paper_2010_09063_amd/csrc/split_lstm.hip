#include "split_lstm.h"

#include <algorithm>
#include <type_traits>

#include "split_bf16.h"

// Two workgroups of eight waves own an example, each a half of the columns and all rows: up to 9 x 8 blocks of 32 x 32,
// waves in two groups of rows and four of columns with up to 5 x 2 blocks in registers (201 x 400: 4 or 3 x 2 or 1).  K is the
// time, sixteen steps at a time: both operands are staged in LDS as the matrix instruction takes them ([block][piece][lane][8],
// lane = column, eight consecutive steps), split once; two buffers, one barrier per unit, the next unit's values in
// registers meanwhile.  A wave stages whole blocks, lanes along the columns.  The workgroups are persistent and the
// pipeline runs on across examples: an example's gradient leaves for memory during the next one's first unit.
// Per unit and SIMD 14 blocks x 6 instructions of 32 cycles against about 2,000 cycles of staging, which the barrier keeps from
// overlapping fully.  Benchmark network, 512 examples x 256 steps, 201 x 400: 238 us on the fp32 instruction, 195 here; 128
// examples 68 and 57; the sum over 50 examples of 201 steps 45 (tiled contraction) and 35.  Any widths: the fp32 kernel took
// multiples of four only, and odd ones went through the tiled contraction.
#define SL_THREADS 512
// A lambda that the compiler leaves as a call keeps what it captures in scratch memory: so it did with three staged blocks per
// wave, and the sum over 64 examples of 256 steps with 128 inputs and 128 units took 153 us instead of 46.
#define SL_INLINE __attribute__((always_inline))

template <int ITEMS, bool NORM>
__global__ __launch_bounds__(SL_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void split_lstm_kernel(const SplitLstmArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Din = a.Din, H = a.H, T = a.T, Gc = 4 * H, M = Din + H + 1;
  const int mb_tot = (M + 31) >> 5, nb_all = (Gc + 31) >> 5, half = blockIdx.y;
  const int nb0 = half ? (nb_all + 1) >> 1 : 0, nb_tot = half ? nb_all >> 1 : (nb_all + 1) >> 1;
  const int n_blk = mb_tot + nb_tot, buf_bytes = n_blk * 3072;
  // this wave's tile; waves w and w + 4 share a SIMD and take the column groups in rotated order
  const int wm = wave >> 2, wn = (wave + 2 * wm) & 3;
  const int mc = wm == 0 ? (mb_tot + 1) >> 1 : mb_tot >> 1, m0 = wm == 0 ? 0 : (mb_tot + 1) >> 1;
  const int nbase = nb_tot >> 2, nrem = nb_tot & 3, nc = nbase + (wn < nrem ? 1 : 0), n0 = wn * nbase + min(wn, nrem);

  // staging: item q is block wave + 8 q, lane (column li, steps 8 lk .. 8 lk + 7 of the unit)
  int kind[ITEMS], col[ITEMS], stride[ITEMS]; // kind 0: nothing, 1: x, 2: h of the step before, 3: the constant 1, 4: gate gradients
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    const int blk = wave + 8 * q;
    if (blk < mb_tot) {
      const int c = blk * 32 + li;
      kind[q] = c < Din ? 1 : (c < Din + H ? 2 : (c == Din + H ? 3 : 0));
      col[q] = c < Din ? c : (c < Din + H ? c - Din : 0);
      stride[q] = kind[q] == 1 ? Din : (kind[q] == 2 ? H : 0);
    } else {
      const int c = (nb0 + blk - mb_tot) * 32 + li;
      const bool ok = blk < n_blk && c < Gc;
      kind[q] = ok ? 4 : 0;
      col[q] = ok ? c : 0;
      stride[q] = ok ? Gc : 0;
    }
  }
  float raw[ITEMS][8];
  auto fetch = [&](int e, int t0) SL_INLINE { // every load unconditional and from a valid address; what it is worth is decided in stash
    const float *xe = a.x + (long)e * T * Din, *he = a.hs + (long)e * T * H, *ge = a.dg + (long)e * T * Gc;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      const float *p = (kind[q] == 2 ? he : (kind[q] == 4 ? ge : xe)) + col[q];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int t = min(t0 + 8 * lk + j, T - 1), s = kind[q] == 2 ? max(t - 1, 0) : t;
        raw[q][j] = p[s * stride[q]];
      }
    }
  };
  // the gate gradients change sign with the example, in sums with the partial row, and so does what is added up here (split_bf16.h)
  auto sign = [&](int e) SL_INLINE { return (NORM ? e : (int)blockIdx.x) & 1 ? -1.f : 1.f; };
  auto stash = [&](char *buf, int e, int t0) SL_INLINE {
    const float f = NORM ? sign(e) : sign(e) * a.scale[e];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      const int blk = wave + 8 * q;
      if (blk >= n_blk) continue; // (uniform)
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int t = t0 + 8 * lk + j;
        const bool ok = t < T && kind[q] != 0;
        float w = kind[q] == 3 ? 1.f : raw[q][j];
        if (kind[q] == 2 && t == 0) w = 0.f;
        if (blk >= mb_tot) w *= f;
        v[j] = ok ? w : 0.f;
      }
      SbFrag fr;
      sb_split8(v, fr);
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<sb_u32x4 *>(buf + blk * 3072 + p * 1024 + lane * 16) = fr.p[p];
    }
  };

  const int units = (T + 15) >> 4; // per example
  // norm: examples blockIdx.x, + gridDim.x, ...; sum: a run of units, whatever their examples
  const long u_first = NORM ? 0 : (long)blockIdx.x * a.units_per_wg;
  const long n_units = NORM ? (long)((a.B - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x) * units
                            : min((long)a.units_per_wg, (long)a.B * units - u_first);
  auto run = [&](auto mc_, auto nc_) SL_INLINE {
    constexpr int MC = decltype(mc_)::value, NC = decltype(nc_)::value;
    constexpr int MA = MC > 0 && NC > 0 ? MC : 1, NA = MC > 0 && NC > 0 ? NC : 1;
    sb_f32x16 acc[MA][NA];
    auto clear = [&]() SL_INLINE {
#pragma unroll
      for (int i = 0; i < MA; ++i)
#pragma unroll
        for (int j = 0; j < NA; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };
    // accumulator register r of a lane: row 8 (r / 4) + 4 lk + r % 4, column li of its block
    auto store = [&](float *g, float sg) SL_INLINE { // g: the matrix in the parameter layout, sg its sign here; returns the sum of the squares
      float q2 = 0.f;
      // (the rows' offsets and lane masks are made here: hoisted out of the loop over units they are 1,600 spilled scalar registers)
      const int gc = __builtin_amdgcn_readfirstlane(Gc);
      if constexpr (MC > 0 && NC > 0) {
#pragma unroll
        for (int i = 0; i < MC; ++i)
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            const int n = (nb0 + n0 + j) * 32 + li;
            float *gi = g + (long)(m0 + i) * 32 * gc; // (uniform)
            const unsigned off = 4u * (unsigned)(4 * lk * Gc + n);
            int left = n < Gc ? M - (m0 + i) * 32 - 4 * lk : 0;
            asm volatile("" : "+v"(left));
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int ru = 8 * (r >> 2) + (r & 3);
              const float v = sg * acc[i][j][r];
              q2 = fmaf(v, v, q2); // (zero beyond the matrix: nothing else was staged)
              if (g != nullptr && ru < left) *reinterpret_cast<float *>(reinterpret_cast<char *>(gi + (long)ru * gc) + off) = v;
            }
          }
      }
      return q2;
    };
    auto finish = [&](int e) SL_INLINE {
      float q2 = store(a.gstore != nullptr ? a.gstore + (long)e * a.gstride : nullptr, sign(e));
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) q2 += __shfl_xor(q2, o, 64);
      if (lane == 0) a.slots[(long)(a.slot0 + half * 8 + wave) * a.slot_stride + e] = q2;
    };
    clear();
    int e = NORM ? (int)blockIdx.x : (int)(u_first / units), u = NORM ? 0 : (int)(u_first - (long)e * units), done = -1;
    fetch(e, 16 * u);
    for (long g = 0; g < n_units; ++g) {
      char *buf = lds + (g & 1) * buf_bytes;
      stash(buf, e, 16 * u);
      __syncthreads(); // unit g is staged; every wave is done with unit g - 1 (it staged g after its multiplies)
      int en = e, un = u + 1;
      if (un == units) { un = 0; en += NORM ? (int)gridDim.x : 1; }
      fetch(min(en, a.B - 1), 16 * un); // (past the last unit: not used)
      __builtin_amdgcn_sched_barrier(0);
      if (NORM && done >= 0) { finish(done); clear(); done = -1; }
      if constexpr (MC > 0 && NC > 0) {
        SbFrag y[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j)
#pragma unroll
          for (int p = 0; p < 3; ++p) y[j].p[p] = *reinterpret_cast<const sb_u32x4 *>(buf + (mb_tot + n0 + j) * 3072 + p * 1024 + lane * 16);
#pragma unroll
        for (int i = 0; i < MC; ++i) {
          SbFrag x[1];
#pragma unroll
          for (int p = 0; p < 3; ++p) x[0].p[p] = *reinterpret_cast<const sb_u32x4 *>(buf + (m0 + i) * 3072 + p * 1024 + lane * 16);
          sb_mfma(x, y, *reinterpret_cast<sb_f32x16 (*)[1][NC]>(&acc[i]));
        }
      }
      if (NORM && u == units - 1) done = e;
      e = en; u = un;
    }
    if (NORM) {
      if (done >= 0) finish(done);
    } else {
      (void)store(a.part + (long)blockIdx.x * a.part_stride, sign(0));
    }
  };
#define SL_NC(mc_) \
  if (nc == 2) run(std::integral_constant<int, mc_>{}, std::integral_constant<int, 2>{}); \
  else if (nc == 1) run(std::integral_constant<int, mc_>{}, std::integral_constant<int, 1>{}); \
  else run(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
  if (mc == 5) { SL_NC(5) } else if (mc == 4) { SL_NC(4) } else if (mc == 3) { SL_NC(3) } else if (mc == 2) { SL_NC(2) }
  else if (mc == 1) { SL_NC(1) } else run(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
#undef SL_NC
}

bool split_lstm_enable() {
  const hipFuncAttribute at = hipFuncAttributeMaxDynamicSharedMemorySize;
  const int bytes = 2 * (SPLIT_LSTM_MB + 8) * 3072;
  return hipFuncSetAttribute((const void *)split_lstm_kernel<2, true>, at, bytes) == hipSuccess &&
         hipFuncSetAttribute((const void *)split_lstm_kernel<2, false>, at, bytes) == hipSuccess &&
         hipFuncSetAttribute((const void *)split_lstm_kernel<3, true>, at, bytes) == hipSuccess &&
         hipFuncSetAttribute((const void *)split_lstm_kernel<3, false>, at, bytes) == hipSuccess;
}

template <bool NORM>
static void launch_one(hipStream_t st, const SplitLstmArgs &a, int groups) {
  const int mb = (a.Din + a.H + 1 + 31) / 32, nb = (4 * a.H + 31) / 32, blk = mb + (nb + 1) / 2;
  dim3 grid(groups, nb > 1 ? 2 : 1);
  const size_t lds = 2 * (size_t)blk * 3072;
  if (blk <= 16) hipLaunchKernelGGL((split_lstm_kernel<2, NORM>), grid, dim3(SL_THREADS), lds, st, a);
  else hipLaunchKernelGGL((split_lstm_kernel<3, NORM>), grid, dim3(SL_THREADS), lds, st, a);
}

int split_lstm_norm(hipStream_t st, const SplitLstmArgs &a) {
  const int halves = 4 * a.H > 32 ? 2 : 1;
  launch_one<true>(st, a, std::min(a.B, 256 / halves)); // one persistent workgroup per CU
  return halves * 8;
}

int split_lstm_sum(hipStream_t st, SplitLstmArgs a, int max_split) {
  const int halves = 4 * a.H > 32 ? 2 : 1;
  const long units = (long)a.B * ((a.T + 15) / 16);
  // one round of workgroups, but runs of at least eight units: a partial row costs its write and a read by the final write
  const int want = (int)std::max<long>(1, std::min<long>(std::min(max_split, 256 / halves), units / 8));
  a.units_per_wg = (int)((units + want - 1) / want);
  const int groups = (int)((units + a.units_per_wg - 1) / a.units_per_wg);
  launch_one<false>(st, a, groups);
  return groups;
}
