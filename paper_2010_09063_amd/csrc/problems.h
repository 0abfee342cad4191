// The contractions of the private step: operand pairs of gemm_tile_kernel with their epilogues, and the list of
// instantiations, which is cut into groups so that the groups compile in parallel (gemm_group.hip, once per group).
#pragma once
#include "activations.h"
#include "operands.h"

template <class A_, class B_>
struct ProbBase {
  typedef A_ A;
  typedef B_ B;
  int M, N, K, k_chunk, tiles_n, tiles, splits, groups;
  A a;
  B b;
};

// out[m*ld + n] = act(acc + bias[n])                                  (dense forward, LSTM input projection)
template <class A_, class B_>
struct ProbBiasAct : ProbBase<A_, B_> {
  static constexpr bool kReduce = false;
  float *out; const float *bias; int ld, act;
  DEVI void store(int, int, int m, int n, float v) const { out[(long)m * ld + n] = act_apply(act, v + bias[n]); }
};

// out[z*zstride + m*ld + n] = acc                                     (batched plain product)
template <class A_, class B_>
struct ProbBatchOut : ProbBase<A_, B_> {
  static constexpr bool kReduce = false;
  float *out; long zstride; int ld;
  DEVI void store(int z, int, int m, int n, float v) const { out[z * zstride + (long)m * ld + n] = v; }
};

// out[m*ld + n] = acc * act'(a_prev[m*ld + n])                        (dense backward-data)
template <class A_, class B_>
struct ProbBwdAct : ProbBase<A_, B_> {
  static constexpr bool kReduce = false;
  float *out; const float *a_prev; int ld, act;
  DEVI void store(int, int, int m, int n, float v) const {
    long o = (long)m * ld + n;
    out[o] = act ? v * act_deriv_from_out(act, a_prev[o]) : v;
  }
};

// conv forward: m = output channel, n = pixel (b, p): out[b, m, p] = act(acc + bias[m])
template <class A_, class B_>
struct ProbConvFwd : ProbBase<A_, B_> {
  static constexpr bool kReduce = false;
  float *out; const float *bias; int D, P, act; FastDiv dP;
  DEVI void store(int, int, int m, int n, float v) const {
    int b = (int)dP.div(n), p = n - b * P;
    out[((long)b * D + m) * P + p] = act_apply(act, v + bias[m]);
  }
};

// conv backward-data: m = input channel, n = input pixel (b, ih*W+iw): out[b, m, hw] = acc * act'(a_prev)
template <class A_, class B_>
struct ProbConvBwd : ProbBase<A_, B_> {
  static constexpr bool kReduce = false;
  float *out; const float *a_prev; int C, HW, act; FastDiv dHW;
  DEVI void store(int, int, int m, int n, float v) const {
    int b = (int)dHW.div(n), r = n - b * HW;
    long o = ((long)b * C + m) * HW + r;
    out[o] = act ? v * act_deriv_from_out(act, a_prev[o]) : v;
  }
};

// split-K partial of a clipped sum: part[split*stride + m*ldm + n]; if bias_col >= 0 the column
// n == bias_col goes to bias_off + m instead (conv: bias gradient is the ones-tap column).
template <class A_, class B_>
struct ProbPartial : ProbBase<A_, B_> {
  static constexpr bool kReduce = false;
  float *part; long stride; int ldm, bias_col; long bias_off;
  DEVI void store(int, int split, int m, int n, float v) const {
    long o = (n == bias_col) ? bias_off + m : (long)m * ldm + n;
    part[split * stride + o] = v;
  }
};

// per-example weight-gradient tile, squared and summed: slot[(slot0 + tile)*slot_stride + z]
template <class A_, class B_>
struct ProbSqNorm : ProbBase<A_, B_> {
  static constexpr bool kReduce = true;
  float *slots; long slot_stride; int slot0;
  float *gstore; long gstride; // optional: example z's gradient is also written to gstore[z*gstride + m*N + n]
  DEVI float contrib(int z, int m, int n, float v) const {
    if (gstore) gstore[z * gstride + (long)m * this->N + n] = v;
    return v * v;
  }
  DEVI void store_tile(int z, int tile, float s) const { slots[(long)(slot0 + tile) * slot_stride + z] = s; }
};

// ---------------------------------------------------------------- instantiations

#define DP_GEMM_INST1(EXT_, BM_, BN_, WM_, WN_, ...)                                                          \
  EXT_ template __global__ void gemm_tile_kernel<TileCfg<BM_, BN_, WM_, WN_>, __VA_ARGS__, true>(const __VA_ARGS__);  \
  EXT_ template __global__ void gemm_tile_kernel<TileCfg<BM_, BN_, WM_, WN_>, __VA_ARGS__, false>(const __VA_ARGS__);
#define DP_GEMM_INST(EXT_, ...)                                                                               \
  DP_GEMM_INST1(EXT_, 128, 128, 2, 2, __VA_ARGS__) DP_GEMM_INST1(EXT_, 64, 64, 2, 2, __VA_ARGS__)             \
  DP_GEMM_INST1(EXT_, 32, 32, 1, 1, __VA_ARGS__) DP_GEMM_INST1(EXT_, 32, 128, 1, 4, __VA_ARGS__)              \
  DP_GEMM_INST1(EXT_, 128, 32, 4, 1, __VA_ARGS__) DP_GEMM_INST1(EXT_, 64, 128, 2, 2, __VA_ARGS__)             \
  DP_GEMM_INST1(EXT_, 128, 64, 2, 2, __VA_ARGS__)
#define DP_GEMM_GROUP_0(EXT_) \
  DP_GEMM_INST(EXT_, ProbPartial<OpRowMajor<true>, OpKMajor<true, false>>) \
  DP_GEMM_INST(EXT_, ProbPartial<OpRowMajor<false>, OpKMajor<false, false>>)
#define DP_GEMM_GROUP_1(EXT_) \
  DP_GEMM_INST(EXT_, ProbBiasAct<OpRowMajor<true>, OpKMajor<true, false>>) \
  DP_GEMM_INST(EXT_, ProbBiasAct<OpRowMajor<false>, OpKMajor<false, false>>)
#define DP_GEMM_GROUP_2(EXT_) \
  DP_GEMM_INST(EXT_, ProbBwdAct<OpRowMajor<true>, OpRowMajor<true>>) \
  DP_GEMM_INST(EXT_, ProbBwdAct<OpRowMajor<false>, OpRowMajor<false>>)
#define DP_GEMM_GROUP_3(EXT_) \
  DP_GEMM_INST(EXT_, ProbPartial<OpKMajor<true, true>, OpKMajor<true, false>>) \
  DP_GEMM_INST(EXT_, ProbPartial<OpKMajor<false, true>, OpKMajor<false, false>>)
#define DP_GEMM_GROUP_4(EXT_) \
  DP_GEMM_INST(EXT_, ProbConvFwd<OpRowMajor<true>, OpConvPatch<true>>) \
  DP_GEMM_INST(EXT_, ProbConvFwd<OpRowMajor<false>, OpConvPatch<true>>)
#define DP_GEMM_GROUP_5(EXT_) \
  DP_GEMM_INST(EXT_, ProbConvBwd<OpConvWeightT, OpConvDeltaGather>) \
  DP_GEMM_INST(EXT_, ProbBatchOut<OpKMajor<false, false>, OpKMajor<false, false>>)
#define DP_GEMM_GROUP_6(EXT_) \
  DP_GEMM_INST(EXT_, ProbSqNorm<OpRowMajor<true>, OpConvPatch<false>>) \
  DP_GEMM_INST(EXT_, ProbSqNorm<OpRowMajor<false>, OpConvPatch<false>>)
#define DP_GEMM_GROUP_7(EXT_) \
  DP_GEMM_INST(EXT_, ProbPartial<OpChanPix, OpConvPatch<false>>)
#define DP_GEMM_GROUP_8(EXT_) \
  DP_GEMM_INST(EXT_, ProbSqNorm<OpLstmIn<true>, OpKMajor<true, false>>) \
  DP_GEMM_INST(EXT_, ProbSqNorm<OpLstmIn<false>, OpKMajor<false, false>>)
#define DP_GEMM_GROUP_9(EXT_) \
  DP_GEMM_INST(EXT_, ProbPartial<OpLstmIn<true>, OpKMajor<true, false>>) \
  DP_GEMM_INST(EXT_, ProbPartial<OpLstmIn<false>, OpKMajor<false, false>>)
#define DP_GEMM_GROUPS 10

#ifndef DP_GEMM_GROUP
DP_GEMM_GROUP_0(extern)
DP_GEMM_GROUP_1(extern)
DP_GEMM_GROUP_2(extern)
DP_GEMM_GROUP_3(extern)
DP_GEMM_GROUP_4(extern)
DP_GEMM_GROUP_5(extern)
DP_GEMM_GROUP_6(extern)
DP_GEMM_GROUP_7(extern)
DP_GEMM_GROUP_8(extern)
DP_GEMM_GROUP_9(extern)
#endif
