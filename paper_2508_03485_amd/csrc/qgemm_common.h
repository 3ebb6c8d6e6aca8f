// Pieces of the int8 GEMM's epilogue that qgemm.hip and qgemm_wide.hip share.
#pragma once
#include "lrq_internal.h"

namespace lrq {
namespace {

// two floats -> two bf16 (round-to-nearest-even, v_cvt_pk_bf16_f32), a in the low half
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// fp32(a + zero * colsum).  The sum can exceed 32 bits.  Up to kZpF64K channels it is a whole number below 2^53 (|zero| <= 2^31,
// |colsum| <= 127 K, |a| <= 127^2 K), so fp64 holds it exactly and the conversion rounds it once, as it would a 64-bit integer; that
// takes three instructions where the 64-bit multiply and conversion take about twenty (2333 x 1152 -> 1091: 2 us of a 15 us
// launch).  Longer rows take the integers, in a kernel of their own (ZP64), so that the others do not carry them.
constexpr int kZpF64K = 32768;
__device__ __forceinline__ float zp_sum(int a, double zero, double colsum) { return (float)fma(zero, colsum, (double)a); }
__device__ __forceinline__ float zp_sum64(int a, double zero, double colsum) {
    return (float)((long long)a + (long long)(int)zero * (long long)(int)colsum);
}

}  // namespace
}  // namespace lrq
