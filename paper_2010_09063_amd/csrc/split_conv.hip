#include "split_conv.h"

#include <algorithm>
#include <type_traits>

#include "activations.h"
#include "split_bf16.h"

// A wave works alone: 64 output pixels (two blocks of 32: the even and the odd rows, so that a 2x2 pool window is two
// lanes of both blocks) x 32 output channels, KS waves sharing the input channels of a tile.  Per 16 input channels
// it fetches the haloed pixels with the channel as the register index, splits them once and leaves them in an LDS area
// of its own, channels innermost ([piece][channel half][pixel][8]), so that the operand of every tap is one 16-byte
// read per piece at a constant offset; the weight fragments come from the L2.  No barrier until the KS partial sums
// meet.  The next chunk travels in registers meanwhile.  108 matrix instructions of 32 cycles per chunk against about 300
// others and 54 LDS reads.  What bounds it is not the matrix units, which are busy for 10 to 34 % of the time (25 % for
// 48 -> 48 channels on 32x32 planes at 61 examples, 30 % for 128 -> 128 on 8x8 at 256), but fetching and splitting, the
// operands' reads (1.2 to 1.6 conflict cycles per active LDS cycle on planes up to 16 wide, none on 32) and one or two
// waves per SIMD to cover for each other.
template <int LW>
struct SplitConvGeom {
  static constexpr int W = 1 << LW, ROWS = 64 / W, LD = W + 2;
  static constexpr int PIX = LW == 5 ? 136 : (LW == 4 ? 120 : (LW == 3 ? 120 : 144)); // staged pixels, halo included, at most
  static constexpr int ITEMS = (2 * PIX + 63) / 64, PLANE = 2 * PIX * 16;              // per lane; bytes of one piece
};

template <int LW, int KS, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void split_conv_kernel(const SplitConvArgs a) {
  typedef SplitConvGeom<LW> G;
  constexpr int W = G::W, LD = G::LD, MB = 1; // (blocks of 32 output channels)
  __shared__ __attribute__((aligned(16))) char lds[4][3 * G::PLANE];
  const int lane = threadIdx.x & 63, li = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = wave % KS, H = a.H, HW = H * W, Cin = a.Cin;
  const int seg_rows = min(G::ROWS, H), segs = G::ROWS / seg_rows; // images per tile and their rows
  const int pix = segs * (seg_rows + 2) * LD;
  const int R0 = ((int)blockIdx.x * (4 / KS) + wave / KS) * G::ROWS; // first row of the tile, all images' rows in a line
  const int img0 = R0 / H, y0 = R0 - img0 * H;
  const bool live = img0 < a.B;
  const int mb_tot = (a.M + 31) >> 5, mb0 = blockIdx.y * MB;
  char *my = lds[wave];

  // staging items: (channel half, haloed pixel), lanes along the pixels
  int off[G::ITEMS]; // floats from the first image's plane of the chunk's first channel; < 0: a zero
#pragma unroll
  for (int q = 0; q < G::ITEMS; ++q) {
    const int it = lane + 64 * q, half = it >= pix ? 1 : 0, p = it - half * pix;
    const int seg = p / ((seg_rows + 2) * LD), pr = p - seg * ((seg_rows + 2) * LD), yy = pr / LD;
    const int y = y0 + yy - 1, x = pr - yy * LD - 1;
    const bool ok = it < 2 * pix && x >= 0 && x < W && y >= 0 && y < H && img0 + seg < a.B;
    off[q] = ok ? (seg * Cin + 8 * half) * HW + y * W + x : -1;
  }
  const float *base = a.x + (long)(live ? img0 : 0) * Cin * HW;
  const int chunks = (Cin + 15) >> 4;
  float raw[G::ITEMS][8];
  auto fetch = [&](int ck) {
    const float *b = base + (long)ck * 16 * HW;
#pragma unroll
    for (int q = 0; q < G::ITEMS; ++q) {
      const int o = max(off[q], 0);
      const int lim = RAGGED ? Cin - ck * 16 - (lane + 64 * q >= pix ? 8 : 0) : 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const unsigned at = (unsigned)(!RAGGED || j < lim ? o + j * HW : 0) * 4u; // (always a valid address)
        raw[q][j] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(b) + at);
      }
    }
  };
  auto stash = [&](int ck) {
#pragma unroll
    for (int q = 0; q < G::ITEMS; ++q) {
      const int it = lane + 64 * q;
      const int lim = RAGGED ? Cin - ck * 16 - (it >= pix ? 8 : 0) : 8;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = off[q] >= 0 && (!RAGGED || j < lim) ? raw[q][j] : 0.f;
      SbFrag f;
      sb_split8(v, f);
      if (it < 2 * pix) {
        // (the second half starts at a fixed place whatever the number of pixels)
        char *dst = my + (it >= pix ? G::PIX + it - pix : it) * 16;
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<sb_u32x4 *>(dst + p * G::PLANE) = f.p[p];
      }
    }
  };
  // the lane's pixel of block i: column li % W, row 2 (li / W) + i of the tile
  const int px = li & (W - 1), pr2 = 2 * (li >> LW), pseg = pr2 / seg_rows, py = pr2 - pseg * seg_rows;
  const char *rd = my + (lk * G::PIX + (pseg * (seg_rows + 2) + py) * LD + px) * 16;

  sb_f32x16 acc[MB][2], low[MB][2];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][i][r] = low[m][i][r] = 0.f;
  const sb_u32x4 *fr = (const sb_u32x4 *)a.frag + (long)mb0 * 192 + lane;
  const long fstep = (long)mb_tot * 192;
  if (part < chunks) fetch(part);
  for (int ck = part; ck < chunks; ck += KS) {
    __builtin_amdgcn_wave_barrier();
    stash(ck);
    __builtin_amdgcn_wave_barrier(); // (read by other lanes of this wave: its LDS operations complete in order)
    __builtin_amdgcn_sched_barrier(0);
    fetch(min(ck + KS, chunks - 1)); // (past the last one: read again, unused)
    const sb_u32x4 *f = fr + (long)ck * 9 * fstep;
    SbFrag w[2][MB]; // one tap ahead
    auto weights = [&](int tap, SbFrag (&d)[MB]) {
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int p = 0; p < 3; ++p) d[m].p[p] = f[tap * fstep + m * 192 + p * 64];
    };
    weights(0, w[0]);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      if (tap < 8) weights(tap + 1, w[(tap + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0); // (left alone the compiler sinks each load to its use)
      SbFrag x[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          x[i].p[p] = *reinterpret_cast<const sb_u32x4 *>(rd + p * G::PLANE + ((tap / 3 + i) * LD + tap % 3) * 16);
      sb_mfma2(w[tap & 1], x, acc, low);
    }
  }
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][i][r] += low[m][i][r];

  // the partial sums of the KS waves: each leaves its own in its LDS area and finishes 16 / KS of the sixteen registers
  float sum[2][MB][16 / KS];
  if constexpr (KS > 1) {
    static_assert(MB == 1 && 2 * 16 * 64 * 4 <= 3 * G::PLANE, "partial sums fit the staging area");
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) *reinterpret_cast<float *>(my + ((i * 16 + r) * 64 + lane) * 4) = acc[0][i][r];
    __syncthreads();
    const int w0 = wave - part;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16 / KS; ++r) {
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < KS; ++q)
          v += *reinterpret_cast<const float *>(lds[w0 + q] + ((i * 16 + part * (16 / KS) + r) * 64 + lane) * 4);
        sum[i][0][r] = v;
      }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[i][m][r] = acc[m][i][r];
  }

  const int img = img0 + pseg, y = y0 + py;
  if (img >= a.B) return;
  const unsigned o_lane = (unsigned)((pseg * a.M + 4 * lk) * HW + y * W + px);
  const unsigned po_lane = (unsigned)((pseg * a.M + 4 * lk) * (HW >> 2) + (y >> 1) * (W >> 1) + (px >> 1));
  const bool fwd = a.bias != nullptr;
  auto finish = [&](auto act_c, auto mode_c) { // MODE: 0 forward, 1 + max-pool, 2 + mean pool, 3 backward-data through an activation, 4 backward-data
    constexpr int ACT = decltype(act_c)::value, MODE = decltype(mode_c)::value;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int r0 = 0; r0 < 16 / KS; r0 += 4) {
        const int mu = 32 * (mb0 + m) + 2 * (KS == 1 ? r0 : part * (16 / KS) + r0); // accumulator register r: row 8 (r / 4) + 4 lk + r % 4
        if (mu >= a.M) continue;
        const long plane = ((long)img0 * a.M + mu) * HW;
        float s[2][4], bv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool ok = mu + 4 * lk + r < a.M;
          if (MODE <= 2) bv[r] = a.bias[ok ? mu + 4 * lk + r : 0];
          if (MODE == 3) {
#pragma unroll
            for (int i = 0; i < 2; ++i) s[i][r] = a.a_prev[plane + (ok ? o_lane + (unsigned)(r * HW + i * W) : 0u)];
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (mu + 4 * lk + r >= a.M) continue;
          float v0 = sum[0][m][r0 + r], v1 = sum[1][m][r0 + r];
          if (MODE <= 2) { v0 = act_apply(ACT, v0 + bv[r]); v1 = act_apply(ACT, v1 + bv[r]); }
          if (MODE == 3) { v0 *= act_deriv_from_out(ACT, s[0][r]); v1 *= act_deriv_from_out(ACT, s[1][r]); }
          if (MODE == 1 || MODE == 2) {
            const float u0 = swap1(v0), u1 = swap1(v1); // the window's other column
            if ((px & 1) == 0) {
              const long po = ((long)img0 * a.M + mu) * (HW >> 2) + po_lane + (unsigned)(r * (HW >> 2));
              if (MODE == 1) { // first maximum in row-major order
                float best = v0; int bi = 0;
                if (u0 > best) { best = u0; bi = 1; }
                if (v1 > best) { best = v1; bi = 2; }
                if (u1 > best) { best = u1; bi = 3; }
                a.pool_out[po] = best;
                a.pool_arg[po] = (uint8_t)bi;
              } else {
                a.pool_out[po] = ((v0 + u0) + (v1 + u1)) * 0.25f;
              }
            }
          }
          if (MODE != 1) { // (the plane before a fused max-pool is never read)
            float *o = a.out + plane + (o_lane + (unsigned)(r * HW));
            o[0] = v0;
            o[W] = v1;
          }
        }
      }
  };
  auto with_mode = [&](auto act_c) {
    if (fwd) {
      if (a.pool == 1) finish(act_c, std::integral_constant<int, 1>{});
      else if (a.pool) finish(act_c, std::integral_constant<int, 2>{});
      else finish(act_c, std::integral_constant<int, 0>{});
    } else if (a.act) {
      finish(act_c, std::integral_constant<int, 3>{});
    } else {
      finish(act_c, std::integral_constant<int, 4>{});
    }
  };
  if (a.act == DP_ACT_TANH_) with_mode(std::integral_constant<int, DP_ACT_TANH_>{});
  else if (a.act == DP_ACT_RELU_) with_mode(std::integral_constant<int, DP_ACT_RELU_>{});
  else with_mode(std::integral_constant<int, DP_ACT_NONE_>{});
}

template <int LW, int KS, bool RAGGED>
static void launch_one(hipStream_t st, const SplitConvArgs &a) {
  const int tiles = (a.B * a.H + SplitConvGeom<LW>::ROWS - 1) / SplitConvGeom<LW>::ROWS;
  dim3 grid((tiles + 4 / KS - 1) / (4 / KS), (a.M + 31) / 32);
  hipLaunchKernelGGL((split_conv_kernel<LW, KS, RAGGED>), grid, dim3(256), 0, st, a);
}

template <int LW>
static void launch_lw(hipStream_t st, const SplitConvArgs &a) {
  const long tiles = ((long)a.B * a.H * a.W + 63) / 64;
  const int mbt = (a.M + 31) / 32, chunks = (a.Cin + 15) / 16;
  // one block of 32 output channels per wave (its two accumulators leave no registers for a second block; two with one
  // accumulator took the same time); where that leaves the SIMDs (1024) clearly fewer than two waves each,
  // the input channels are shared by two or four waves (128 -> 128 on 8x8 planes at 256 examples, 1024 waves: 64 us,
  // 2048: 35; 48 -> 48 on 32x32 at 61, 1952 waves: 30 us, 3904: 37)
  if (a.Cin % 16 == 0) {
    if (tiles * mbt >= 1536 || chunks < 2) { launch_one<LW, 1, false>(st, a); return; }
    if (tiles * mbt >= 640 || chunks < 4) { launch_one<LW, 2, false>(st, a); return; }
    launch_one<LW, 4, false>(st, a);
    return;
  }
  if (tiles * mbt >= 1536 || chunks < 2) { launch_one<LW, 1, true>(st, a); return; }
  if (tiles * mbt >= 640 || chunks < 4) { launch_one<LW, 2, true>(st, a); return; }
  launch_one<LW, 4, true>(st, a);
}

void split_conv_launch(hipStream_t st, const SplitConvArgs &a) {
  if (a.W == 32) launch_lw<5>(st, a);
  else if (a.W == 16) launch_lw<4>(st, a);
  else if (a.W == 8) launch_lw<3>(st, a);
  else launch_lw<2>(st, a);
}
