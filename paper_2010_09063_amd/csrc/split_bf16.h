// fp32 products on the bf16 matrix units, without giving up fp32 operands.
//
// An fp32 value is the exact sum of three bf16 values (8 + 8 + 8 significand bits, each the rounded remainder of the one
// before), and a product of two such sums is nine bf16 products, of which the six down to 2^-16 of the largest are
// taken; the three that are dropped are together below 2^-24 of it with random sign, and a 32 x 32 x 16 instruction adds
// sixteen products to the fp32 accumulator at once where v_mfma_f32_32x32x2_f32 rounds after every second one.
// Measured against 64 bits the sums are no further off than the fp32 instruction's.  Six instructions of 32 cycles per 16
// of K against eight of 64.  (An infinite operand gives NaN: its remainder is inf - inf.  So it does in the
// minimal-filtering kernels.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 sb_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 sb_bf16x8 __attribute__((ext_vector_type(8)));
typedef float sb_f32x2 __attribute__((ext_vector_type(2)));
typedef float sb_f32x16 __attribute__((ext_vector_type(16)));
typedef float sb_f32x4u __attribute__((ext_vector_type(4), aligned(4))); // rows need not start on 16 bytes
typedef uint32_t sb_u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t sb_pack(float a, float b) { // v_cvt_pk_bf16_f32
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((sb_f32x2){a, b}, sb_bf16x2));
}
// two values -> their three pieces, packed two by two
__device__ __forceinline__ void sb_split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
  h = sb_pack(a, b);
  a -= __uint_as_float(h << 16); b -= __uint_as_float(h & 0xFFFF0000u);
  m = sb_pack(a, b);
  a -= __uint_as_float(m << 16); b -= __uint_as_float(m & 0xFFFF0000u);
  l = sb_pack(a, b);
}
struct SbFrag { sb_u32x4 p[3]; }; // eight consecutive k of one row, as the matrix instruction takes them
__device__ __forceinline__ void sb_split8(const float (&v)[8], SbFrag &f) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t h, m, l;
    sb_split2(v[2 * j], v[2 * j + 1], h, m, l);
    f.p[0][j] = h; f.p[1][j] = m; f.p[2][j] = l;
  }
}
// The instruction cuts off what lies below the accumulator's last bit, downwards: a long sum of all six products in one
// accumulator comes out low by 5e-8 of its size (K = 1024, signed operands, root mean square error 4.8e-7; the fp32
// instruction: 3e-9 and 5.8e-7), and a sum over many such values, a bias gradient behind several layers, shows it.  So where
// results feed further sums the five small products have an accumulator of their own, added at the end: 2e-9 and 1.7e-7.
template <int NI, int NJ>
__device__ __forceinline__ void sb_mfma2(const SbFrag (&a)[NI], const SbFrag (&b)[NJ], sb_f32x16 (&acc)[NI][NJ], sb_f32x16 (&low)[NI][NJ]) {
  constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int q = 0; q < 6; ++q)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        sb_f32x16 &d = q < 5 ? low[i][j] : acc[i][j];
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sb_bf16x8, a[i].p[pa[q]]),
                                                    __builtin_bit_cast(sb_bf16x8, b[j].p[pb[q]]), d, 0, 0, 0);
      }
}
// acc[i][j] += A[i] B[j] for NI x NJ blocks of 32 x 32 x 16, smallest terms first.  The blocks take turns: an instruction
// that adds to the accumulator of the one before waits for it.
template <int NI, int NJ>
__device__ __forceinline__ void sb_mfma(const SbFrag (&a)[NI], const SbFrag (&b)[NJ], sb_f32x16 (&acc)[NI][NJ]) {
  constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int q = 0; q < 6; ++q)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sb_bf16x8, a[i].p[pa[q]]),
                                                            __builtin_bit_cast(sb_bf16x8, b[j].p[pb[q]]), acc[i][j], 0, 0, 0);
}
