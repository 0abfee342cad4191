// Sequence kernels: the LSTM recurrence (forward and back-propagation through
// time) and the embedding layer's per-example norm / clipped scatter-add.
//
// The recurrence is a chain of T dependent (examples x H)*(H x 4H) products; per step it is far too small for a
// tiled contraction, and examples are independent.  Each workgroup of LSTM_THREADS threads therefore owns one
// example for the whole sequence and keeps W_hh in registers (forward: a quarter of the rows for the four gate
// columns of one hidden unit per thread, summed over a quad of lanes with DPP moves; backward: a sixteenth of the
// columns for four hidden units per thread, summed over a row of lanes), so a step costs no weight traffic at all: only the hidden state goes through LDS
// (broadcast reads).  A step is a chain of dependent phases, so what bounds it is latency: eight waves per
// example (two per SIMD) overlap each other's LDS reads, and every global load is issued a whole step before its
// value is used.  The input projection x_t W_ih + b and the input / weight gradients are hoisted out of the loop
// into the tiled MFMA contraction.  The [B, T, 4H] buffer is reused in place: input projection -> activated
// gates (forward) -> gate gradients (backward).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels_misc.h"
#include "split_f16.h"

#define LSTM_THREADS 512

// x_{b,t} = E[tok[b,t]]: the embedding lookup, written once per step so that the three
// contractions that read it (input projection, per-example and clipped weight gradient)
// address it directly instead of chasing the token id first.
__global__ void emb_gather_kernel(const int *__restrict__ tok, const float *__restrict__ table,
                                  float *__restrict__ xseq, long rows, int D) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * D) return;
  long r = i / D;
  int e = (int)(i - r * D);
  xseq[i] = table[(long)tok[r] * D + e];
}

// The same lookup for rows that are whole 16-byte groups (D a multiple of 4, both pointers 16-byte aligned): a thread
// copies four coordinates, a row's groups lie in consecutive threads.
__global__ void emb_gather4_kernel(const int *__restrict__ tok, const float4 *__restrict__ table,
                                   float4 *__restrict__ xseq, long rows, int D4) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * D4) return;
  const long r = i / D4;
  const int e = (int)(i - r * D4);
  xseq[i] = table[(long)tok[r] * D4 + e];
}

__device__ __forceinline__ float sigmoidf_(float v) { return fast_sigmoid(v); }

// Mean over the T step vectors of a sequence (embedding network, Appendix B): out[b, e] = (1/T) sum_t in[b, t, e].
// One workgroup per example: thread (tl, e) sums the steps tl, tl + ntl, ... of coordinate e (consecutive threads
// read consecutive coordinates of one step), the ntl partial sums of a coordinate are added in a fixed order.
__global__ __launch_bounds__(256) void seq_mean_fwd_kernel(const float *__restrict__ in, float *__restrict__ out,
                                                            int T, int D) {
  __shared__ float part[256];
  const int b = blockIdx.x, tid = threadIdx.x;
  const int dp = D < 256 ? D : 256, ntl = 256 / dp;
  const int e_l = tid % dp, tl = tid / dp;
  const float *p = in + (long)b * T * D;
  for (int e0 = 0; e0 < D; e0 += dp) {
    const int e = e0 + e_l;
    float s = 0.f;
    if (tl < ntl && e < D)
      for (int t = tl; t < T; t += ntl) s += p[(long)t * D + e];
    part[tid] = s;
    __syncthreads();
    if (tl == 0 && e < D) {
      float tot = 0.f;
      for (int q = 0; q < ntl; ++q) tot += part[q * dp + e_l];
      out[(long)b * D + e] = tot / (float)T;
    }
    __syncthreads();
  }
}

// The classifier of a sequence network (a dense layer of at most 16 classes on a vector per example): logits, loss
// gradient (rows of 16, zero beyond the classes), the layer's squared norm (slot, null: not wanted) and the gradient of
// its input, one wave per example.  Lane (class n = lane / 4, quarter of the input) for the logits.  Split-K
// contraction, loss kernel and backward contraction were three launches of 11 + 5 + 6 us at 128 examples.
__global__ __launch_bounds__(256) void class_head_kernel(const float *__restrict__ in, const float *__restrict__ W,
                                                         const float *__restrict__ bias, const int *__restrict__ y,
                                                         float *__restrict__ delta, float *__restrict__ gin,
                                                         float *__restrict__ slot, int B, int D, int N) {
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (b >= B) return;
  const float *a = in + (long)b * D;
  const int n = lane >> 2, q = lane & 3, nc = min(n, N - 1);
  float z = 0.f, sa = 0.f;
  for (int e0 = 0; e0 < D; e0 += 16) { // (four input values per lane in flight)
    float v[4], w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = e0 + 4 * j + q, ec = min(e, D - 1);
      v[j] = a[ec];
      w[j] = W[(long)ec * N + nc];
      if (e >= D) v[j] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) { z = fmaf(v[j], w[j], z); sa = fmaf(v[j], v[j], sa); }
  }
  z += __shfl_xor(z, 1, 64); z += __shfl_xor(z, 2, 64);
  sa += __shfl_xor(sa, 1, 64); sa += __shfl_xor(sa, 2, 64);
  z = n < N ? z + bias[nc] : -INFINITY;
  float mx = z;
#pragma unroll
  for (int o = 4; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  const float ex = n < N ? expf(z - mx) : 0.f;
  float se = ex;
#pragma unroll
  for (int o = 4; o < 64; o <<= 1) se += __shfl_xor(se, o, 64);
  const float d = n < N ? ex * (1.f / se) - (n == y[b] ? 1.f : 0.f) : 0.f;
  float sd = d * d;
#pragma unroll
  for (int o = 4; o < 64; o <<= 1) sd += __shfl_xor(sd, o, 64);
  if (q == 0) delta[(long)b * 16 + n] = d;
  if (slot != nullptr && lane == 0) slot[b] = (sa + 1.f) * sd;
  for (int e0 = 0; e0 < D; e0 += 64) {
    const int e = e0 + lane;
    float g = 0.f;
    for (int m = 0; m < N; ++m) g = fmaf(W[(long)min(e, D - 1) * N + m], __shfl(d, 4 * m, 64), g);
    if (e < D) gin[(long)b * D + e] = g;
  }
}

// ... and its gradient: every step receives g[b, e] / T.  One thread per (b, t, e).
__global__ void seq_mean_bwd_kernel(const float *__restrict__ g, float *__restrict__ gin, long n, int T, int D) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const long bt = i / D;
  const int e = (int)(i - bt * D);
  const long b = bt / T;
  gin[i] = g[b * D + e] / (float)T;
}

// Lane-relative access on a uniform base pointer with an unsigned byte offset: one address register per access
// (a signed or pre-scaled index would be widened to 64 bits per lane).
__device__ __forceinline__ float &lane_at(float *base, unsigned byte_off) {
  return *reinterpret_cast<float *>(reinterpret_cast<char *>(base) + byte_off);
}
__device__ __forceinline__ float lane_ld(const float *base, unsigned byte_off) {
  return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + byte_off);
}

// Quad-lane helpers: the four lanes 4u .. 4u+3 exchange values with DPP moves (no LDS, no barrier).
__device__ __forceinline__ float quad_xor1(float v) { // lanes swap within pairs: quad_perm [1,0,3,2]
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ float quad_xor2(float v) { // pairs swap: quad_perm [2,3,0,1]
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));
}
template <int Q>
__device__ __forceinline__ float quad_bcast(float v) { // every lane of the quad gets lane Q's value
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), Q * 0x55, 0xF, 0xF, true));
}

__device__ __forceinline__ float row_swap8(float v) { // the halves of a row of sixteen lanes change places
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, true));
}
__device__ __forceinline__ float quad_mirror(float v) { // each quad in reverse order: quad_perm [3,2,1,0]
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x1B, 0xF, 0xF, true));
}
__device__ __forceinline__ float half_mirror(float v) { // each eight lanes in reverse order
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true));
}

// Forward.  gates: in  x_t W_ih + b for every (b, t); out activated i, f, g, o.
// hs, cs: [B, T, H] hidden and cell states; hlast [B, H] = h_T, or the mean of every h_t (mean != 0: the sequence mean
// that follows the layer in the Appendix B network costs one addition a step here and was a launch of 33 us at 128
// examples).  H <= 128, HP >= H.
// Thread (u = tid / 4, q = tid % 4) belongs to hidden unit u and holds, for all four gates
// of that unit, the quarter q of the rows of W_hh (k in [q*QL, q*QL + QL)).  A step is then: quarter product (QL
// broadcast words of h from LDS instead of all H), sum over the quad with two DPP exchanges per gate, lane q
// activates and stores gate q, the quad shares the four activated gates, every lane updates the unit's cell
// state, lane 0 publishes h.  h is double-buffered in LDS, so ONE barrier per step suffices: a step reads one
// buffer and writes the other, and every wave has finished reading a buffer before the barrier after which it is
// written again.
template <int HP>
__global__ __launch_bounds__(LSTM_THREADS) void lstm_fwd_kernel(float *__restrict__ gates, const float *__restrict__ Whh,
                                                                      float *__restrict__ hs, float *__restrict__ cs,
                                                                      float *__restrict__ hlast, int mean, int B, int T, int H) {
  constexpr int QL = (HP + 3) / 4;        // rows of W_hh per quarter
  constexpr int QLP = (QL + 3) & ~3;      // the quarter's stride in LDS (16-byte aligned)
  __shared__ __attribute__((aligned(16))) float h_s[2][4 * QLP];
  const int tid = threadIdx.x;
  const int b = blockIdx.x; // the grid is exactly B workgroups
  const int G = 4 * H;
  const int u = tid >> 2, q = tid & 3;
  const bool unit_ok = u < H;
  const int ul = unit_ok ? u : 0;
  float w[4][QL];
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int i = 0; i < QL; ++i) {
      const int k = q * QL + i;
      w[g][i] = (unit_ok && k < H) ? Whh[(long)k * G + g * H + ul] : 0.f;
    }
  for (int i = tid; i < 2 * 4 * QLP; i += LSTM_THREADS) (&h_s[0][0])[i] = 0.f;
  float c_reg = 0.f, h_sum = 0.f;
  const unsigned colb = 4u * (q * H + ul), ub = 4u * ul;
  const int hpos = (ul / QL) * QLP + ul % QL; // where unit u's h sits in a buffer
  float *const grow0 = gates + (long)b * T * G;
  float *const hrow0 = hs + (long)b * T * H, *const crow0 = cs + (long)b * T * H;
  __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0): the weight loads end here, not at their first use inside the loop
  __syncthreads();
  auto step = [&](const int t, const float xcur, float &xnext, const float *hin, float *hout) {
    unsigned colx = colb, ux = ub; // (re-materialised inside the loop: hoisted, they would be widened to 64 bits)
    asm volatile("" : "+v"(colx), "+v"(ux));
    xnext = lane_ld(grow0 + (long)min(t + 1, T - 1) * G, colx);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const float *hq = hin + q * QLP;
#pragma unroll
    for (int i = 0; i + 4 <= QL; i += 4) {
      const float4 h4 = *reinterpret_cast<const float4 *>(hq + i);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        acc[g] = fmaf(h4.x, w[g][i], acc[g]); acc[g] = fmaf(h4.y, w[g][i + 1], acc[g]);
        acc[g] = fmaf(h4.z, w[g][i + 2], acc[g]); acc[g] = fmaf(h4.w, w[g][i + 3], acc[g]);
      }
    }
#pragma unroll
    for (int i = QL & ~3; i < QL; ++i) {
      const float hv = hq[i];
#pragma unroll
      for (int g = 0; g < 4; ++g) acc[g] = fmaf(hv, w[g][i], acc[g]);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      acc[g] += quad_xor1(acc[g]);
      acc[g] += quad_xor2(acc[g]);
    }
    // lane q activates gate q (order i, f, g, o: gate 2 is the tanh one)
    const float mine = q == 0 ? acc[0] : (q == 1 ? acc[1] : (q == 2 ? acc[2] : acc[3]));
    const float pre = mine + xcur;
    const float v = q == 2 ? fast_tanh(pre) : sigmoidf_(pre);
    if (unit_ok) lane_at(grow0 + (long)t * G, colx) = v;
    const float gi = quad_bcast<0>(v), gf = quad_bcast<1>(v), gg = quad_bcast<2>(v), go = quad_bcast<3>(v);
    c_reg = gf * c_reg + gi * gg;
    const float h = go * fast_tanh(c_reg);
    if (unit_ok && q == 0) {
      hout[hpos] = h;
      lane_at(hrow0 + (long)t * H, ux) = h;
      lane_at(crow0 + (long)t * H, ux) = c_reg;
      h_sum += h;
      if (t == T - 1) lane_at(hlast + (long)b * H, ux) = mean ? h_sum / (float)T : h;
    }
    __syncthreads();
  };
  float xa = lane_ld(grow0, colb), xb;
  int t = 0;
  for (; t + 1 < T; t += 2) {
    step(t, xa, xb, h_s[0], h_s[1]);
    step(t + 1, xb, xa, h_s[1], h_s[0]);
  }
  if (t < T) step(t, xa, xb, h_s[0], h_s[1]);
}

typedef float lstm_f32x4 __attribute__((ext_vector_type(4)));

// The same for two examples per workgroup, which is ahead where every compute unit has two (above 256 examples).
//
// A step's product W_hh^T h is on the matrix units, operands as two fp16 pieces of a scaled value (split_f16.h): weights by
// the largest of their column, h, which lies between -1 and 1, by 2^14.  v_mfma_f32_4x4x4_16b_f16 is sixteen products of
// 4 x 4: a block is one hidden unit, its rows the four gates, so that a lane's accumulators are the four gates of its
// unit, and its columns are (example, piece).  The two pieces of the weights have accumulators of their own.  A wave owns
// sixteen units; its weights (8 KS registers) stay for all T steps, h goes through LDS, [column][k], double-buffered,
// with one barrier a step.  Lanes p = 0 of a unit and example activate gates i and g, p = 1 f and o.
// 256 steps, H = 100, 512 examples: 282 -> 224 us; the vector kernel issues 100 multiply-adds and 50 others per wave and step
// and is bound by that.  Here 104 matrix instructions of 4.7 ns per SIMD and step are 0.49 us of 0.87, the chain of
// activations, exchange and reads the rest; with one example (half of the columns) they take as long, and the vector kernel
// is ahead: 168 against 211 us at 128.
// A weight is off by up to 2^-40 of its column's largest, a sum (of 128 at most, |h| <= 1) by 2^-33 of it.  From 2^12 on that could
// show in a gate's argument, where the unit behind the large weight is off: such networks are multiplied in fp32, by
// v_mfma_f32_4x4x1_16b_f32 in the same blocks, columns (example, twice): 354 us instead of 243, the vector kernel 288 (one
// multiply-add at a time took 2,860).
#define LSTM_WILD 4096.f
// fewest units that a kernel of KS is launched with
template <int KS>
constexpr int lstm_units_from() { return KS == 4 ? 1 : 8 * KS - 23; }
// that product of a block: this lane's row of weights with the block's operand in LDS; four sums, each operand read four
// multiplies of four ahead (all at once they would not fit beside the weights)
template <int KS>
__device__ __forceinline__ lstm_f32x4 lstm_fp32_product(const float (&w)[8 * KS], const float *x) {
  lstm_f32x4 s[4] = {}, v[2 * KS];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const lstm_f32x4 *>(x + 4 * i);
#pragma unroll
  for (int i = 0; i < 2 * KS; ++i) {
    if (i + 4 < 2 * KS) v[i + 4] = *reinterpret_cast<const lstm_f32x4 *>(x + 4 * i + 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = __builtin_amdgcn_mfma_f32_4x4x1f32(w[4 * i + j], v[i][j], s[j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  return (s[0] + s[1]) + (s[2] + s[3]);
}
template <int KS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_fwd2_kernel(float *__restrict__ gates, const float *__restrict__ Whh,
                                                                       float *__restrict__ hs, float *__restrict__ cs,
                                                                       float *__restrict__ hlast, int mean, int B, int T, int H) {
  typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
  typedef lstm_f32x4 f32x4;
  constexpr int KP = 8 * KS + 8; // halves of a column in LDS (columns on different banks)
  __shared__ __attribute__((aligned(16))) _Float16 h_s[2][4 * KP];
  const int tid = threadIdx.x, q = tid & 3, u = tid >> 2; // quad: a unit; lane of the quad: a column
  const int e = q >> 1, p = q & 1, b0 = 2 * (int)blockIdx.x;
  const int b = min(b0 + e, B - 1); // (an example past the last one: the last one again, not stored)
  const int G = 4 * H;
  const bool unit_ok = u < H, store = unit_ok && b0 + e < B;
  const int ul = unit_ok ? u : 0;
  // the weights of gate q of the unit, and what takes the four gates' scales out
  float wv[8 * KS], top = 0.f;
#pragma unroll
  for (int k = 0; k < 8 * KS; ++k) {
    wv[k] = Whh[(long)min(k, H - 1) * G + q * H + ul];
    if (k >= lstm_units_from<KS>()) wv[k] = k < H ? wv[k] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < 8 * KS; k += 2) top = sf_max3(wv[k], wv[k + 1], top);
  for (int i = tid; i < 2 * 4 * KP; i += blockDim.x) (&h_s[0][0])[i] = (_Float16)0.f;
  float c_reg = 0.f, h_sum = 0.f;
  const unsigned colb = 4u * (p * H + ul), ub = 4u * ul, eb = (unsigned)(b - b0) * (unsigned)T * 4u; // (gates p and p + 2)
  float *const grow0 = gates + (long)b0 * T * G;
  float *const hrow0 = hs + (long)b0 * T * H, *const crow0 = cs + (long)b0 * T * H;
  const bool wild = __syncthreads_or(top >= LSTM_WILD); // (the weight loads end here, not at their first use inside the loop)
  // activations, state and what is written, from this lane's two gates' arguments; returns h
  auto cell = [&](const int t, const float pre0, const float pre1, const unsigned colx, const unsigned ux) {
    // (order i, f, g, o: gate 2 is the tanh one)
    const float v0 = sigmoidf_(pre0), v1 = p ? sigmoidf_(pre1) : fast_tanh(pre1);
    if (store) {
      lane_at(grow0 + (long)t * G, colx) = v0;
      lane_at(grow0 + (long)t * G, colx + 8u * H) = v1;
    }
    const float o0 = quad_xor1(v0), o1 = quad_xor1(v1);
    c_reg = (p ? v0 : o0) * c_reg + (p ? o0 : v0) * (p ? o1 : v1);
    return (p ? v1 : o1) * fast_tanh(c_reg);
  };
  auto write = [&](const int t, const float h, const unsigned ux) {
    if (store) lane_at((p ? crow0 : hrow0) + (long)t * H, ux) = p ? c_reg : h;
    h_sum += h;
    if (t == T - 1 && store && p == 0) hlast[(long)b * H + ul] = mean ? h_sum / (float)T : h;
  };
  const unsigned col0 = colb + eb * (unsigned)G, u0 = ub + eb * (unsigned)H;
  if (wild) {
    float *const hf = reinterpret_cast<float *>(&h_s[0][0]) + e * KP; // [step parity][example][unit]
    static_assert(sizeof(h_s) == 4 * KP * sizeof(float), "h in fp32");
    for (int t = 0; t < T; ++t) {
      const float *gr = grow0 + (long)t * G, *hp = hf + (t & 1) * 2 * KP;
      const float x0 = lane_ld(gr, col0), x1 = lane_ld(gr, col0 + 8u * H);
      const f32x4 s = lstm_fp32_product<KS>(wv, hp);
      const float h = cell(t, (p ? s[1] : s[0]) + x0, (p ? s[3] : s[2]) + x1, col0, u0);
      if (unit_ok && p == 0) hf[((t + 1) & 1) * 2 * KP + u] = h;
      write(t, h, u0);
      __syncthreads();
    }
    return;
  }
  f16x4 w[2][2 * KS];
  float un[4];
  {
    const uint32_t ex = sf_exponent(__float_as_uint(top));
    const float sc = sf_scale(ex), back = sf_unscale(ex) * 6.103515625e-5f; // (h's 2^14 as well)
    un[0] = quad_bcast<0>(back); un[1] = quad_bcast<1>(back); un[2] = quad_bcast<2>(back); un[3] = quad_bcast<3>(back);
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = wv[4 * i + j] * sc;
        const _Float16 hi = (_Float16)v;
        w[0][i][j] = hi;
        w[1][i][j] = (_Float16)(v - (float)hi);
      }
    }
  }
  auto step = [&](const int t, const float x0, const float x1, float &n0, float &n1, const _Float16 *hin, _Float16 *hout) {
    unsigned colx = colb, ux = ub, ex = eb; // (re-materialised inside the loop: hoisted, they would be widened to 64 bits)
    asm volatile("" : "+v"(colx), "+v"(ux), "+v"(ex));
    colx += ex * (unsigned)G; ux += ex * (unsigned)H;
    {
      const float *nx = grow0 + (long)min(t + 1, T - 1) * G;
      n0 = lane_ld(nx, colx); n1 = lane_ld(nx, colx + 8u * H);
    }
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const _Float16 *hq = hin + q * KP;
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const uint4 t4 = *reinterpret_cast<const uint4 *>(hq + 8 * i);
      const f16x4 h0 = __builtin_bit_cast(f16x4, make_uint2(t4.x, t4.y)), h1 = __builtin_bit_cast(f16x4, make_uint2(t4.z, t4.w));
      acc[0] = __builtin_amdgcn_mfma_f32_4x4x4f16(w[0][2 * i], h0, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_4x4x4f16(w[1][2 * i], h0, acc[1], 0, 0, 0);
      acc[0] = __builtin_amdgcn_mfma_f32_4x4x4f16(w[0][2 * i + 1], h1, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_4x4x4f16(w[1][2 * i + 1], h1, acc[1], 0, 0, 0);
    }
    float s[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float v = acc[0][g] + acc[1][g]; // this lane's piece of h; the other one is next door
      s[g] = (v + quad_xor1(v)) * un[g];
    }
    const float h = cell(t, (p ? s[1] : s[0]) + x0, (p ? s[3] : s[2]) + x1, colx, ux);
    if (unit_ok) { // the piece of h for the lane's column
      const float hsc = h * 16384.f;
      const _Float16 hi = (_Float16)hsc, lo = (_Float16)(hsc - (float)hi);
      hout[q * KP + u] = p ? lo : hi;
    }
    write(t, h, ux);
    __syncthreads();
  };
  float xa0 = lane_ld(grow0, col0), xa1 = lane_ld(grow0, col0 + 8u * H), xb0, xb1;
  int t = 0;
  for (; t + 1 < T; t += 2) {
    step(t, xa0, xa1, xb0, xb1, h_s[0], h_s[1]);
    step(t + 1, xb0, xb1, xa0, xa1, h_s[1], h_s[0]);
  }
  if (t < T) step(t, xa0, xa1, xb0, xb1, h_s[0], h_s[1]);
}

// Back-propagation through time.  gates: in activated gates, out d(loss)/d(gate pre-activations).
// One workgroup per example.  Its product dL/dh_{t-1} = W_hh dgates_t is dealt out as (four hidden units kk = tid / 16, a
// sixteenth s = tid % 16 of the 4H columns).  The sixteen partial sums of the four units are added so that the unit
// 4 kk + s / 4 ends up in the quad of lanes s / 4, where lane s % 4 makes that gate's gradient of it: a step is product,
// sum, gate gradient, LDS write and one barrier, and everything else that the step needs is there before its product.
// (With a gate's part of one unit per thread the sums went through LDS to the two waves that updated the cells, two
// barriers a step.)  256 steps, H = 100: 222 -> 173 us at 128 examples, 306 -> 294 us at 512, two examples per compute unit.
// Bound by the issue of vector instructions, 100 multiply-adds and about 60 others per wave and step: 1,280 of the 1,600
// cycles of a step for two waves per SIMD, all of them for four.  (128 registers, so that two workgroups share a
// compute unit, are two short: they spill.)
// dh_out is [B, H].  SEQ = false: the gradient of h_T, which is all that the loss sees.  SEQ = true: the gradient of the
// mean over every h_t: each step adds its share dh_out / T to what the later steps send back.
template <int HP, bool SEQ>
__global__ __launch_bounds__(LSTM_THREADS, (HP <= 100 ? 4 : 2)) void lstm_bwd_kernel(float *__restrict__ gates, const float *__restrict__ cs,
                                                                 const float *__restrict__ Whh,
                                                                 const float *__restrict__ dh_out, int B, int T, int H) {
  constexpr int QC = HP / 4;                // columns per thread: the flat index g * HP + j cut into sixteen
  constexpr int QCP = ((QC + 3) / 4 | 1) * 4; // a sixteenth's stride in LDS: 16-byte reads, an odd number of them apart (no bank twice)
  __shared__ __attribute__((aligned(16))) float dg_s[2][16 * QCP];
  const int tid = threadIdx.x;
  const int b = blockIdx.x; // the grid is exactly B workgroups
  const int G = 4 * H;
  const int kk = tid >> 4, s16 = tid & 15, q = tid & 3;
  const int u = 4 * kk + (s16 >> 2);
  const bool unit_ok = u < H;
  const int ul = unit_ok ? u : 0;
  float w[4][QC];
#pragma unroll
  for (int i = 0; i < QC; ++i) {
    const int f = s16 * QC + i, g = f / HP, j = f - g * HP;
#pragma unroll
    for (int m = 0; m < 4; ++m) w[m][i] = (4 * kk + m < H && j < H) ? Whh[(long)(4 * kk + m) * G + g * H + j] : 0.f;
  }
  for (int i = tid; i < 2 * 16 * QCP; i += LSTM_THREADS) (&dg_s[0][0])[i] = 0.f;
  // the thread's gate column, its unit and the place of its gradient in LDS, in one register: the weights leave few
  const unsigned where = (q * H + ul) | ul << 10 | ((4 * q + ul / QC) * QCP + ul % QC) << 18;
  float *const grow0 = gates + (long)b * T * G;
  const float *const crow0 = cs + (long)b * T * H;
  float dh_own = dh_out[(long)b * H + ul];
  if (SEQ) dh_own /= (float)T;
  float dc = 0.f;
  __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0): the weight loads end here, not at their first use inside the loop
  __syncthreads();
  // Step t with its activated gate, c_t and c_{t-1}; requests the gate of step t - 1 and c_{t-2} (rows clamped at 0).
  // din is what step t + 1 wrote (zeros at the last step).
  auto step = [&](const int t, const float v, const float ct, const float cp, float &vnext, float &cnext, const float *din,
                  float *dout) {
    unsigned at = where; // (taken apart inside the loop: hoisted, the offsets would be widened to 64 bits)
    asm volatile("" : "+v"(at));
    vnext = lane_ld(grow0 + (long)max(t - 1, 0) * G, 4 * (at & 1023));
    cnext = lane_ld(crow0 + (long)max(t - 2, 0) * H, 4 * (at >> 10 & 255));
    // beside dL/dh: a gate's gradient is dL/dc_t (output gate: dL/dh_t) times `k`, dL/dc_t = dc + dL/dh_t * a
    const float gi = quad_bcast<0>(v), gf = quad_bcast<1>(v), gg = quad_bcast<2>(v), go = quad_bcast<3>(v);
    const float tc = fast_tanh(ct);
    const float a = go * (1.f - tc * tc);
    const float cprev = t > 0 ? cp : 0.f;
    float k = fmaf(-v, v, q == 2 ? 1.f : v); // the activation's derivative: 1 - v^2 of a tanh, v - v^2 of a sigmoid
    const float k0 = q == 0 ? gg : gi, k1 = q == 1 ? cprev : tc;
    k *= (q & 1) ? k1 : k0;
    __builtin_amdgcn_sched_barrier(0);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const float *dq = din + s16 * QCP;
#pragma unroll
    for (int i = 0; i + 4 <= QC; i += 4) {
      const float4 d4 = *reinterpret_cast<const float4 *>(dq + i);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        acc[m] = fmaf(d4.x, w[m][i], acc[m]); acc[m] = fmaf(d4.y, w[m][i + 1], acc[m]);
        acc[m] = fmaf(d4.z, w[m][i + 2], acc[m]); acc[m] = fmaf(d4.w, w[m][i + 3], acc[m]);
      }
      if (i % 8 == 4) __builtin_amdgcn_sched_barrier(0); // (all reads at once would take registers that the weights need)
    }
#pragma unroll
    for (int i = QC & ~3; i < QC; ++i) {
      const float dv = dq[i];
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[m] = fmaf(dv, w[m][i], acc[m]);
    }
    // sums: the halves of a row exchange two units each, then its quads one, then the quad adds up
    const bool hi = s16 >= 8, odd = (s16 & 4) != 0;
    const float r0 = (hi ? acc[2] : acc[0]) + row_swap8(hi ? acc[0] : acc[2]);
    const float r1 = (hi ? acc[3] : acc[1]) + row_swap8(hi ? acc[1] : acc[3]);
    float dh = (odd ? r1 : r0) + half_mirror(odd ? r0 : r1);
    dh += quad_xor1(dh);
    dh += quad_xor2(dh);
    if (SEQ || t == T - 1) dh += dh_own;
    const float dct = dc + dh * a;
    const float d = (q == 3 ? dh : dct) * k;
    dc = dct * gf;
    if (unit_ok) {
      asm volatile("" : "+v"(at));
      dout[at >> 18] = d;
      lane_at(grow0 + (long)t * G, 4 * (at & 1023)) = d;
    }
    __syncthreads();
  };
  float va = lane_ld(grow0 + (long)(T - 1) * G, 4 * (q * H + ul)), vb;
  float c0 = lane_ld(crow0 + (long)(T - 1) * H, 4 * ul), c1 = lane_ld(crow0 + (long)max(T - 2, 0) * H, 4 * ul), c2;
  int t = T - 1;
  for (; t > 0; t -= 2) {
    step(t, va, c0, c1, vb, c2, dg_s[0], dg_s[1]);
    step(t - 1, vb, c1, c2, va, c1, dg_s[1], dg_s[0]);
    c0 = c2;
  }
  if (t == 0) step(0, va, c0, c1, vb, c2, dg_s[0], dg_s[1]);
}

// The same for two examples per workgroup on the matrix units, as lstm_fwd2_kernel: a wave owns sixteen units, in blocks of
// (four units) x (gate): a block of v_mfma_f32_4x4x4_16b_f16 multiplies four units' rows of one gate's H columns by that
// gate's gradients, columns (example, piece); the four gates' sums meet within a row of sixteen lanes, each unit's in the
// quad of lanes that owns it, where lanes p = 0 make the gradients of gates i and g, p = 1 f and o.
// Gate gradients have no bound: they are scaled to 2^11 of the largest of the step after (going back in time), and where a
// step's own largest lies more than 2^3 from that, all write theirs once more with its own scale before anyone reads.
// The second pieces, of weights and gradients, are 2^11 times what the first ones leave, which their own accumulators and
// columns take out again: a gradient is off by up to 2^-44 of the example's largest, a weight by 2^-51 of its row's.  What lies
// 2^20 below the largest gradient keeps its bits so; further below, it would show in a unit none of whose weights lead to the
// large ones: networks with weights that are zero or below 2^-26 of their row's largest are multiplied in fp32, as those with
// large weights (one in 700 random ones): 256 steps at 512 examples 450 us instead of 284, the vector kernel 334.
// 100 steps, H = 100, 512 examples: 170 -> 123 us.
template <int KS, bool SEQ>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_bwd2_kernel(float *__restrict__ gates, const float *__restrict__ cs,
                                                                       const float *__restrict__ Whh, const float *__restrict__ dh_out,
                                                                       int B, int T, int H) {
  typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
  typedef lstm_f32x4 f32x4;
  constexpr int KP = KS < 16 ? 120 : 136; // halves of a (gate, column) in LDS: 16-byte reads of sixteen of them on different banks
  __shared__ __attribute__((aligned(16))) _Float16 d_s[2][16 * KP];
  __shared__ uint32_t top[3][2]; // [step][example]: a step's largest gradient
  int tid = threadIdx.x;
  const int G = 4 * H, b0 = 2 * (int)blockIdx.x;
  float wv[8 * KS], most = 0.f, least = INFINITY;
  {
    const int row = (tid >> 6) * 16 + 4 * ((tid >> 4) & 3) + (tid & 3); // the block's units, this lane's of them
    const float *wr = Whh + (long)min(row, H - 1) * G + ((tid >> 2) & 3) * H;
#pragma unroll
    for (int j = 0; j < 8 * KS; ++j) {
      wv[j] = wr[min(j, H - 1)];
      least = fminf(least, fabsf(wv[j])); // (past the last column: the last one again)
      if (j >= lstm_units_from<KS>()) wv[j] = j < H ? wv[j] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < 8 * KS; j += 2) most = sf_max3(wv[j], wv[j + 1], most);
  }
  for (int i = tid; i < 2 * 16 * KP; i += blockDim.x) (&d_s[0][0])[i] = (_Float16)0.f;
  if (tid < 6) top[tid >> 1][tid & 1] = 0;
  float widest = fmaxf(most, quad_mirror(half_mirror(most))); // of the row's four gates
  widest = fmaxf(widest, row_swap8(widest));
  const bool wild = __syncthreads_or(widest >= LSTM_WILD || least < widest * 0x1p-26f); // (large ones as in lstm_fwd2_kernel: where such a weight's gate is saturated)
  asm volatile("" : "+v"(tid)); // (what follows is not worked out, and kept, before the weights are loaded)
  const int lane = tid & 63, q = tid & 3, u = tid >> 2, e = q >> 1, p = q & 1;
  const int b = min(b0 + e, B - 1); // (an example past the last one: the last one again, not stored)
  const bool unit_ok = u < H, store = unit_ok && b0 + e < B;
  const int ul = unit_ok ? u : 0;
  const int bg = (lane >> 2) & 3; // the block's gate
  const unsigned colb = 4u * (p * H + ul), ub = 4u * ul, eb = (unsigned)(b - b0) * (unsigned)T * 4u; // (gates p and p + 2)
  float *const grow0 = gates + (long)b0 * T * G;
  const float *const crow0 = cs + (long)b0 * T * H;
  float dh_own = dh_out[(long)b * H + ul];
  if (SEQ) dh_own /= (float)T;
  float dc = 0.f;
  uint32_t used[2] = {27u, 27u};  // exponents that the two examples' gradients in LDS are scaled by
  uint32_t guess[2] = {27u, 27u}; // the last step's largest, which the next one's are scaled by
  // beside dL/dc_t (output gate: dL/dh_t): this lane's two gates' factors, what dL/dh_t adds to dL/dc_t and what goes on to
  // dL/dc_{t-1}; va, vb: the activated gates, ct, cp: c_t and c_{t-1}
  struct Factors { float ka, kb, a, gf; };
  auto factors = [&](const int t, const float va, const float vb, const float ct, const float cp) {
    const float oa = quad_xor1(va), ob = quad_xor1(vb);
    const float gi = p ? oa : va, gf = p ? va : oa, gg = p ? ob : vb, go = p ? vb : ob;
    const float tc = fast_tanh(ct), cprev = t > 0 ? cp : 0.f;
    return Factors{fmaf(-va, va, va) * (p ? cprev : gg), fmaf(-vb, vb, p ? vb : 1.f) * (p ? tc : gi), go * (1.f - tc * tc), gf};
  };
  auto cell = [&](const int t, const float dh, const Factors &f, const unsigned colx, float &da, float &db) {
    const float dct = dc + dh * f.a;
    da = dct * f.ka; db = (p ? dh : dct) * f.kb;
    dc = dct * f.gf;
    if (store) {
      lane_at(grow0 + (long)t * G, colx) = da;
      lane_at(grow0 + (long)t * G, colx + 8u * H) = db;
    }
  };
  const unsigned col0 = colb + eb * (unsigned)G, u0 = ub + eb * (unsigned)H;
  // the four gates' sums of the block's units: the halves of a row of sixteen lanes exchange two units each, then its quads
  // one; this lane's unit
  auto gates_sum = [&](const f32x4 s) {
    const bool hi = lane & 8, odd = lane & 4;
    const float r0 = (hi ? s[2] : s[0]) + row_swap8(hi ? s[0] : s[2]);
    const float r1 = (hi ? s[3] : s[1]) + row_swap8(hi ? s[1] : s[3]);
    return (odd ? r1 : r0) + quad_mirror(half_mirror(odd ? r0 : r1));
  };
  if (wild) {
    float *const df = reinterpret_cast<float *>(&d_s[0][0]) + e * 4 * KP; // [step parity][example][gate][unit]
    static_assert(sizeof(d_s) == 16 * KP * sizeof(float), "gate gradients in fp32");
    for (int t = T - 1, n = 0; t >= 0; --t, ++n) {
      const float *gr = grow0 + (long)t * G, *dp = df + (n & 1) * 8 * KP + bg * KP;
      const Factors f = factors(t, lane_ld(gr, col0), lane_ld(gr, col0 + 8u * H), lane_ld(crow0 + (long)t * H, u0), lane_ld(crow0 + (long)max(t - 1, 0) * H, u0));
      float dh = gates_sum(lstm_fp32_product<KS>(wv, dp)), da, db;
      if (SEQ || t == T - 1) dh += dh_own;
      cell(t, dh, f, col0, da, db);
      if (unit_ok) {
        float *o = df + ((n + 1) & 1) * 8 * KP + p * KP + u;
        o[0] = da; o[2 * KP] = db;
      }
      __syncthreads();
    }
    return;
  }
  f16x4 w[2][2 * KS];
  f32x4 un;
  {
    const uint32_t ex = sf_exponent(__float_as_uint(most));
    const float sc = sf_scale(ex), back = sf_unscale(ex), piece = p ? 1.f / 2048.f : 1.f;
    un[0] = quad_bcast<0>(back) * piece; un[1] = quad_bcast<1>(back) * piece; un[2] = quad_bcast<2>(back) * piece; un[3] = quad_bcast<3>(back) * piece;
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = wv[4 * i + j] * sc;
        const _Float16 hi = (_Float16)v;
        w[0][i][j] = hi;
        w[1][i][j] = (_Float16)((v - (float)hi) * 2048.f);
      }
    }
  }
  auto exponent = [](uint32_t bits) { return max(bits >> 23, 27u); };
  // n counts the steps; din: what step t + 1 wrote
  auto step = [&](const int t, const int n, const float va, const float vb, const float ct, const float cp, float &na, float &nb, float &cnext,
                  const _Float16 *din, _Float16 *dout) {
    unsigned colx = colb, ux = ub, ex = eb; // (re-materialised inside the loop: hoisted, they would be widened to 64 bits)
    asm volatile("" : "+v"(colx), "+v"(ux), "+v"(ex));
    colx += ex * (unsigned)G; ux += ex * (unsigned)H;
    {
      const float *ng = grow0 + (long)max(t - 1, 0) * G;
      na = lane_ld(ng, colx); nb = lane_ld(ng, colx + 8u * H);
      cnext = lane_ld(crow0 + (long)max(t - 2, 0) * H, ux);
    }
    const Factors f = factors(t, va, vb, ct, cp);
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const _Float16 *dq = din + (bg * 4 + q) * KP;
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const uint4 t4 = *reinterpret_cast<const uint4 *>(dq + 8 * i);
      const f16x4 d0 = __builtin_bit_cast(f16x4, make_uint2(t4.x, t4.y)), d1 = __builtin_bit_cast(f16x4, make_uint2(t4.z, t4.w));
      acc[0] = __builtin_amdgcn_mfma_f32_4x4x4f16(w[0][2 * i], d0, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_4x4x4f16(w[1][2 * i], d0, acc[1], 0, 0, 0);
      acc[0] = __builtin_amdgcn_mfma_f32_4x4x4f16(w[0][2 * i + 1], d1, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_4x4x4f16(w[1][2 * i + 1], d1, acc[1], 0, 0, 0);
    }
    f32x4 s;
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] = fmaf(acc[1][r], 1.f / 2048.f, acc[0][r]) * un[r];
    float dh = gates_sum(s);
    dh += quad_xor1(dh); // the other piece
    dh *= __uint_as_float(((e ? used[1] : used[0]) - 11u) << 23);
    if (SEQ || t == T - 1) dh += dh_own;
    float da, db;
    cell(t, dh, f, colx, da, db);
    // this step's largest, for the next one's scale
    uint32_t *const mine = top[n % 3];
    float m = unit_ok ? fmaxf(fabsf(da), fabsf(db)) : 0.f;
    m = fmaxf(m, quad_xor1(m));
    m = fmaxf(m, quad_mirror(half_mirror(m)));
    m = fmaxf(m, row_swap8(m));
    if ((lane & 13) == 0) atomicMax(&mine[e], __float_as_uint(m)); // (lanes 0 and 2 of a row: the examples)
    if (tid < 2) top[(n + 1) % 3][tid] = 0;
    auto put = [&](uint32_t ee) {
      const float sc = __uint_as_float((265u - ee) << 23); // 2^11 over the power of two
      _Float16 *o = dout + (p * 4 + 2 * e) * KP + u;       // [gate][example, piece][unit]
      const float ya = da * sc, yb = db * sc;
      const _Float16 ha = (_Float16)ya, hb = (_Float16)yb;
      o[0] = ha; o[KP] = (_Float16)((ya - (float)ha) * 2048.f);
      o[8 * KP] = hb; o[9 * KP] = (_Float16)((yb - (float)hb) * 2048.f);
    };
    if (unit_ok) put(e ? guess[1] : guess[0]);
    __syncthreads();
    const uint32_t x0 = exponent(mine[0]), x1 = exponent(mine[1]);
    const int off0 = (int)x0 - (int)guess[0], off1 = (int)x1 - (int)guess[1];
    const bool again0 = off0 > 3 || off0 < -3, again1 = off1 > 3 || off1 < -3; // too large, or small enough to lose bits
    if (again0 || again1) { // (an example's scales never depend on the other one)
      if (unit_ok && (e ? again1 : again0)) put(e ? x1 : x0);
      if (again0) guess[0] = x0;
      if (again1) guess[1] = x1;
      __syncthreads();
    }
    used[0] = guess[0]; used[1] = guess[1];
    guess[0] = x0; guess[1] = x1;
  };
  float va = lane_ld(grow0 + (long)(T - 1) * G, col0), vb = lane_ld(grow0 + (long)(T - 1) * G, col0 + 8u * H), wa, wb;
  float c0 = lane_ld(crow0 + (long)(T - 1) * H, u0), c1 = lane_ld(crow0 + (long)max(T - 2, 0) * H, u0), c2;
  int t = T - 1, n = 0;
  for (; t > 0; t -= 2, n += 2) {
    step(t, n, va, vb, c0, c1, wa, wb, c2, d_s[0], d_s[1]);
    step(t - 1, n + 1, wa, wb, c1, c2, va, vb, c1, d_s[1], d_s[0]);
    c0 = c2;
  }
  if (t == 0) step(0, n, va, vb, c0, c1, wa, wb, c2, d_s[0], d_s[1]);
}

// Embedding layer, per-example squared norm: row v of g_i is the sum of dx_{i,t}
// over the steps t whose token is v, so repeated tokens are added before squaring.
// One workgroup per example: bitonic sort of (token, t) keys in LDS, then a chunked
// segmented sum over the sorted steps.
#define EMB_TMAX 1024
#define EMB_NC 16 // chunks of the sorted steps
// Bitonic sort of KPT*256 keys, element m*256 + tid in kr[m]: exchanges at distance >= 256 stay inside the thread,
// distances 64 and 128 go through LDS (3 such passes for 256 keys), the shorter ones are wave shuffles.
template <int KPT>
__device__ __forceinline__ void emb_sort_keys(uint32_t (&kr)[KPT], uint32_t *key, const int tid) {
  constexpr int N = KPT * 256;
#pragma unroll
  for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j >= 256) {
#pragma unroll
        for (int m = 0; m < KPT; ++m) {
          const int pm = m ^ (j >> 8);
          if (pm > m) {
            const bool up = (((m << 8) + tid) & k) == 0;
            const uint32_t a = kr[m], c = kr[pm];
            if ((a > c) == up) { kr[m] = c; kr[pm] = a; }
          }
        }
      } else {
        if (j >= 64) {
#pragma unroll
          for (int m = 0; m < KPT; ++m) key[(m << 8) + tid] = kr[m];
          __syncthreads();
        }
#pragma unroll
        for (int m = 0; m < KPT; ++m) {
          const int i = (m << 8) + tid;
          const uint32_t other = j >= 64 ? key[i ^ j] : (uint32_t)__shfl_xor((int)kr[m], j, 64);
          const bool keep_min = ((i & j) == 0) == ((i & k) == 0);
          kr[m] = keep_min ? min(kr[m], other) : max(kr[m], other);
        }
        if (j >= 64) __syncthreads();
      }
    }
  }
}

template <int KPT>
__global__ __launch_bounds__(256) void emb_norm_kernel(const int *__restrict__ tok, const float *__restrict__ dx,
                                                        float *__restrict__ slot, int T, int D) {
  __shared__ uint32_t key[EMB_TMAX];
  __shared__ float red[4];
  const int b = blockIdx.x, tid = threadIdx.x;
  uint32_t kr[KPT];
#pragma unroll
  for (int m = 0; m < KPT; ++m) {
    const int i = (m << 8) + tid;
    kr[m] = i < T ? (((uint32_t)tok[(long)b * T + i] << 10) | (uint32_t)i) : 0xFFFFFFFFu;
  }
  emb_sort_keys<KPT>(kr, key, tid);
#pragma unroll
  for (int m = 0; m < KPT; ++m) key[(m << 8) + tid] = kr[m];
  __syncthreads();
  // Segmented sum over the sorted steps, in a fixed order.  The T steps are cut into EMB_NC chunks; a work item
  // (coordinate e, chunk c) walks its chunk: runs of one token that lie inside the chunk are squared at once, the
  // part before the chunk's first run start (lead) and after its last one (tail) are left for the pass below,
  // where one thread per coordinate stitches the chunks together.  (A single walk over all T steps per
  // coordinate leaves all but D threads idle behind T dependent loads.)
  constexpr int ET = 128;                 // coordinates per tile
  __shared__ float lead[EMB_NC][ET], tail[EMB_NC][ET];
  __shared__ int has_head[EMB_NC];
  const int L = (T + EMB_NC - 1) / EMB_NC;
  float tot = 0.f;
  for (int e0 = 0; e0 < D; e0 += ET) {
    const int de = min(ET, D - e0);
    for (int it = tid; it < de * EMB_NC; it += 256) {
      const int c = it / de, e = e0 + (it - c * de);
      const int p0 = c * L, p1 = min(T, p0 + L);
      float acc = 0.f, ld = 0.f;
      bool seen = false;
      uint32_t prev = p0 > 0 && p0 < p1 ? key[p0 - 1] >> 10 : 0xFFFFFFFFu; // (no token has this value: step 0 is a head)
      for (int pb = p0; pb < p1; pb += 8) { // eight loads in flight, then their sums in order
        float v[8];
        uint32_t kk[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          kk[j] = key[min(pb + j, p1 - 1)];
          v[j] = dx[((long)b * T + (kk[j] & 1023u)) * D + e];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (pb + j < p1) {
            const uint32_t tk = kk[j] >> 10;
            if (tk != prev) {
              if (seen) tot += acc * acc; else ld = acc;
              acc = 0.f; seen = true; prev = tk;
            }
            acc += v[j];
          }
      }
      lead[c][e - e0] = seen ? ld : acc;
      tail[c][e - e0] = seen ? acc : 0.f;
      if (e == e0) has_head[c] = seen;
    }
    __syncthreads();
    if (tid < de) {
      float carry = 0.f;
      for (int c = 0; c < EMB_NC; ++c) {
        carry += lead[c][tid];
        if (has_head[c]) { tot += carry * carry; carry = tail[c][tid]; }
      }
      tot += carry * carry;
    }
    __syncthreads();
  }
  for (int o = 32; o > 0; o >>= 1) tot += __shfl_xor(tot, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = tot;
  __syncthreads();
  if (tid == 0) slot[b] = red[0] + red[1] + red[2] + red[3];
}

// Clipped sum of the embedding gradient, G_E[v, :] = sum over steps (b, t) with
// tok[b, t] = v of s_b * dx[b, t, :], as a segmented reduction instead of one float
// atomic per element: the steps are bucketed by token with a counting sort (integer
// atomics only), every bucket is cut into chunks of EMB_CH steps, and one workgroup
// sums one chunk.  A token that fits in one chunk is written with plain stores; only
// the few hot tokens that span several chunks combine with fp32 atomics.
#define EMB_CH 64

#define EMB_LDS_V 12288 // vocabularies up to this size get a per-workgroup LDS histogram

// count[v] += occurrences of v.  A Zipf-distributed batch sends a large share of its
// steps to a handful of tokens, and same-address global atomics serialise, so each
// workgroup of 1024 steps first counts in LDS and issues one global atomic per
// distinct token it saw (the thread that hit the LDS bin first owns the flush).
__global__ __launch_bounds__(1024) void emb_count_kernel(const int *__restrict__ tok, int *__restrict__ count, long n,
                                                          int V) {
  extern __shared__ int bins[];
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (V > EMB_LDS_V) { if (i < n) atomicAdd(&count[tok[i]], 1); return; }
  for (int v = threadIdx.x; v < V; v += 1024) bins[v] = 0;
  __syncthreads();
  int t = -1, old = -1;
  if (i < n) { t = tok[i]; old = atomicAdd(&bins[t], 1); }
  __syncthreads();
  if (old == 0) atomicAdd(&count[t], bins[t]);
}

// one workgroup of 1024: exclusive scans of count[v] (-> start[v]) and of the chunk
// counts ceil(count[v]/EMB_CH) (-> chunk0[v]); start[V], chunk0[V] hold the totals;
// cursor[v] is reset to 0 for the fill pass.
__global__ __launch_bounds__(1024) void emb_scan_kernel(const int *__restrict__ count, int *__restrict__ start,
                                                         int *__restrict__ chunk0, int *__restrict__ cursor, int V) {
  __shared__ int wa[16], wb[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (V + 1023) / 1024;
  const int lo = min(V, tid * per), hi = min(V, lo + per);
  int a = 0, b = 0;
  for (int v = lo; v < hi; ++v) { a += count[v]; b += (count[v] + EMB_CH - 1) / EMB_CH; }
  // inclusive scan of the 1024 range totals: shuffles inside a wave, then the 16 wave totals
  int ia = a, ib = b;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int xa = __shfl_up(ia, o, 64), xb = __shfl_up(ib, o, 64);
    if (lane >= o) { ia += xa; ib += xb; }
  }
  if (lane == 63) { wa[wave] = ia; wb[wave] = ib; }
  __syncthreads();
  if (wave == 0) {
    int ta = lane < 16 ? wa[lane] : 0, tb = lane < 16 ? wb[lane] : 0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int xa = __shfl_up(ta, o, 64), xb = __shfl_up(tb, o, 64);
      if (lane >= o) { ta += xa; tb += xb; }
    }
    if (lane < 16) { wa[lane] = ta; wb[lane] = tb; }
  }
  __syncthreads();
  const int offa = wave > 0 ? wa[wave - 1] : 0, offb = wave > 0 ? wb[wave - 1] : 0;
  int ra = offa + ia - a, rb = offb + ib - b; // exclusive prefix of this thread's range
  for (int v = lo; v < hi; ++v) {
    start[v] = ra; chunk0[v] = rb; cursor[v] = 0;
    ra += count[v]; rb += (count[v] + EMB_CH - 1) / EMB_CH;
  }
  if (tid == 1023) { start[V] = wa[15]; chunk0[V] = wb[15]; }
}

// list[start[v] + rank] = step index, rank unique within the bucket: the workgroup reserves a
// range of its bucket with one global atomic per distinct token, steps take their rank in LDS.
__global__ __launch_bounds__(1024) void emb_fill_kernel(const int *__restrict__ tok, const int *__restrict__ start,
                                                         int *__restrict__ cursor, int *__restrict__ list, long n,
                                                         int V) {
  extern __shared__ int bins[];
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (V > EMB_LDS_V) {
    if (i < n) { const int v = tok[i]; list[start[v] + atomicAdd(&cursor[v], 1)] = (int)i; }
    return;
  }
  for (int v = threadIdx.x; v < V; v += 1024) bins[v] = 0;
  __syncthreads();
  int t = -1, old = -1;
  if (i < n) { t = tok[i]; old = atomicAdd(&bins[t], 1); }
  __syncthreads();
  if (old == 0) bins[t] = atomicAdd(&cursor[t], bins[t]); // the bin now holds this workgroup's base rank
  __syncthreads();
  if (i < n) list[start[t] + bins[t] + old] = (int)i;
}

// The three kernels above in one launch, for small batches (up to 2^15 steps, vocabularies that fit the LDS
// histogram): count in LDS, scan, then hand out the positions of every bucket from LDS cursors.  One workgroup walks
// through all the steps twice, so its time grows with the batch -- measured 98 us at 131,072 Zipf-distributed steps
// (the hot tokens serialise the LDS atomics) against 57 us for the three launches -- while three launches cost
// 15-20 us each however small the batch; hence the limit.  The order of the steps inside a bucket depends on the
// order in which the LDS atomics retire, as it does with the three-kernel route.
#define EMB_ONE_MAX_ROWS (1 << 15)
__global__ __launch_bounds__(1024) void emb_bucket_one_kernel(const int *__restrict__ tok, int *__restrict__ start,
                                                               int *__restrict__ chunk0, int *__restrict__ list, int n,
                                                               int V) {
  extern __shared__ int bins[]; // [V]
  __shared__ int wa[16], wb[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int v = tid; v < V; v += 1024) bins[v] = 0;
  __syncthreads();
  for (int i = tid; i < n; i += 1024) atomicAdd(&bins[tok[i]], 1);
  __syncthreads();
  // exclusive scans of the counts and of the chunk counts; every thread owns a run of consecutive tokens
  const int per = (V + 1023) / 1024;
  const int lo = min(V, tid * per), hi = min(V, lo + per);
  int a = 0, b = 0;
  for (int v = lo; v < hi; ++v) { const int c = bins[v]; a += c; b += (c + EMB_CH - 1) / EMB_CH; }
  int ia = a, ib = b;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int xa = __shfl_up(ia, o, 64), xb = __shfl_up(ib, o, 64);
    if (lane >= o) { ia += xa; ib += xb; }
  }
  if (lane == 63) { wa[wave] = ia; wb[wave] = ib; }
  __syncthreads();
  if (wave == 0) {
    int ta = lane < 16 ? wa[lane] : 0, tb = lane < 16 ? wb[lane] : 0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int xa = __shfl_up(ta, o, 64), xb = __shfl_up(tb, o, 64);
      if (lane >= o) { ta += xa; tb += xb; }
    }
    if (lane < 16) { wa[lane] = ta; wb[lane] = tb; }
  }
  __syncthreads();
  int ra = (wave > 0 ? wa[wave - 1] : 0) + ia - a, rb = (wave > 0 ? wb[wave - 1] : 0) + ib - b;
  for (int v = lo; v < hi; ++v) {
    const int c = bins[v];
    start[v] = ra; chunk0[v] = rb;
    bins[v] = ra; // the bucket's cursor for the fill pass
    ra += c; rb += (c + EMB_CH - 1) / EMB_CH;
  }
  if (tid == 1023) { start[V] = wa[15]; chunk0[V] = wb[15]; }
  __syncthreads();
  for (int i = tid; i < n; i += 1024) list[atomicAdd(&bins[tok[i]], 1)] = i;
}

// one workgroup per chunk; workgroups past the last chunk exit.  acc must be zero
// on entry (rows of tokens that do not occur stay zero).
__global__ __launch_bounds__(256) void emb_reduce_kernel(const int *__restrict__ start, const int *__restrict__ chunk0,
                                                          const int *__restrict__ list, const float *__restrict__ dx,
                                                          const float *__restrict__ scale, float *__restrict__ acc,
                                                          int V, int T, int D) {
  __shared__ int ent[EMB_CH];
  __shared__ float sc[EMB_CH];
  __shared__ float part[256];
  const int chunk = blockIdx.x;
  if (chunk >= chunk0[V]) return;
  // token whose chunk range contains `chunk`: last v with chunk0[v] <= chunk
  int lo = 0, hi = V;
  while (hi - lo > 1) { int mid = (lo + hi) >> 1; if (chunk0[mid] <= chunk) lo = mid; else hi = mid; }
  const int v = lo, ci = chunk - chunk0[v];
  const int cnt = start[v + 1] - start[v];
  const int e0 = ci * EMB_CH, n = min(EMB_CH, cnt - e0);
  const int tid = threadIdx.x;
  if (tid < n) {
    const int en = list[start[v] + e0 + tid];
    ent[tid] = en;
    sc[tid] = scale ? scale[en / T] : 1.f;
  }
  __syncthreads();
  // two groups of 128 threads each take every other step; thread e < D of a group owns coordinate e
  const int grp = tid >> 7, e = tid & 127;
  for (int ebase = 0; ebase < D; ebase += 128) {
    float a = 0.f;
    if (ebase + e < D)
      for (int i = grp; i < n; i += 2) a += sc[i] * dx[(long)ent[i] * D + ebase + e];
    part[tid] = a;
    __syncthreads();
    if (grp == 0 && ebase + e < D) {
      const float tot = part[e] + part[128 + e];
      float *dst = acc + (long)v * D + ebase + e;
      if (cnt <= EMB_CH) *dst = tot; else unsafeAtomicAdd(dst, tot);
    }
    __syncthreads();
  }
}
