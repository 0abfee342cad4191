// fp32 products on the bf16 matrix units, without giving up fp32 operands (Henry, Tang, Heinecke, "Leveraging the bfloat16
// Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019).
//
// An fp32 value is the exact sum of three bf16 values (8 + 8 + 8 significand bits, each the rounded remainder of the one
// before), and a product of two such sums is nine bf16 products, of which the six down to 2^-16 of the largest are
// taken; the three that are dropped are together below 2^-24 of it with random sign, and a 32 x 32 x 16 instruction adds
// sixteen products to the fp32 accumulator at once where v_mfma_f32_32x32x2_f32 rounds after every second one.
// Measured against 64 bits the sums are no further off than the fp32 instruction's.  Six instructions of 32 cycles per 16
// of K against eight of 64.  Every finite operand is split exactly.  An infinite one gives NaN in all that it is multiplied
// with, also where fp32 gives an infinity: its remainder is inf - inf, and infinity times a piece that is zero.  So it does in
// the minimal-filtering kernels.  (The example's norm is NaN on the fp32 kernels too: a saturated unit's zero times infinity.)
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
  const float top = __uint_as_float(0x7F7F0000u); // the largest bf16: what lies above, a mask of the type's lowest value, would round to infinity
  h = sb_pack(__builtin_amdgcn_fmed3f(a, -top, top), __builtin_amdgcn_fmed3f(b, -top, top));
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
// The instruction rounds its sums with a bias downwards: it cuts off what lies below the last bits of the largest term, the
// accumulator among them.  For one product matrix that is nothing (1e-9 to 1e-8 of its size, its random error 3e-8 to
// 2e-7), but what adds up many of them shows it: the sum of 128 products of K = 256 was low by 1.0e-7 to 1.8e-7 of its size,
// with a root mean square error of 2.1e-7 to 3.7e-7 (the fp32 instruction: below 6e-9, and 2.0e-7 to 3.7e-7).  Hence
// - the sign of one operand alternates between products that are added up later (examples, rows, the shares of a contraction
//   among waves), and the result's with it: half of the errors point upwards (below 2e-8, and 2.0e-7 to 3.3e-7).  In
//   split_rows.hip, split_lstm.hip and split_wgrad.hip, where it costs nothing that can be measured;
// - the small products, which have the most bits to lose, do not meet a large sum inside the instruction where that can be had:
//   in an accumulator of their own, added at the end (sb_mfma2: one product matrix of K = 1024 off by 1.7e-7 instead of
//   4.8e-7), or before all of the large ones in the same accumulator (split_rows.hip, which has all of K at hand).

// acc[i][j] += the products FIRST .. LAST - 1 of A[i] B[j], smallest first (five small ones, then the one of the leading
// pieces), for NI x NJ blocks of 32 x 32 x 16.  The blocks take turns: an instruction that adds to the accumulator of the one
// before waits for it.
template <int FIRST, int LAST, int NI, int NJ>
__device__ __forceinline__ void sb_products(const SbFrag (&a)[NI], const SbFrag (&b)[NJ], sb_f32x16 (&acc)[NI][NJ]) {
  constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int q = FIRST; q < LAST; ++q)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sb_bf16x8, a[i].p[pa[q]]),
                                                            __builtin_bit_cast(sb_bf16x8, b[j].p[pb[q]]), acc[i][j], 0, 0, 0);
}
template <int NI, int NJ>
__device__ __forceinline__ void sb_mfma(const SbFrag (&a)[NI], const SbFrag (&b)[NJ], sb_f32x16 (&acc)[NI][NJ]) {
  sb_products<0, 6>(a, b, acc);
}
template <int NI, int NJ>
__device__ __forceinline__ void sb_mfma2(const SbFrag (&a)[NI], const SbFrag (&b)[NJ], sb_f32x16 (&acc)[NI][NJ], sb_f32x16 (&low)[NI][NJ]) {
  sb_products<0, 5>(a, b, low);
  sb_products<5, 6>(a, b, acc);
}
