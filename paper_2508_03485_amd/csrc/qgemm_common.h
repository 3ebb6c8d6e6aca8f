// Pieces of the int8 GEMM that its kernels share: operand decoding, rescale.
#pragma once
#include "lrq_internal.h"

namespace lrq {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned perm(unsigned hi, unsigned lo, unsigned sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// Raw operand codes of one lane for one K block and one 32-channel tile: its 16-byte slot of the code tiling, i.e. the
// 16 codes (k = 16 (lane / 16) + [0, 16) of the block) of channel lane % 16 of the tile in dwords 0, 1 and those of channel
// 16 + lane % 16 in dwords 2, 3; one nibble each, either bit-width.
template <int BITS>
struct BRaw {
    unsigned d[4];
};

template <int BITS>
__device__ __forceinline__ BRaw<BITS> load_braw(const uint8_t* __restrict__ p) {
    BRaw<BITS> r;
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    r.d[0] = v.x; r.d[1] = v.y; r.d[2] = v.z; r.d[3] = v.w;
    return r;
}

// Decode the 4 codes of operand dword g (0..3) of the slot's channel s (0 | 1).  Raw dword 2s + g/2 holds 8
// codes, byte j = code[j] | code[4+j] << 4.
// 4-bit: the level table has 16 entries (L[0..1] codes 0..7, L[2..3] codes 8..15 = negative twin): two 8-entry byte
// permutes and a third that picks per byte by the code's sign bit.  C = 0x03020100 must live in a VGPR so that the
// pick selector is a single v_and_or_b32.
// 3-bit: 8-entry table, the masked nibbles are the selectors of one byte permute.
template <int BITS>
__device__ __forceinline__ unsigned decode_dword(const BRaw<BITS>& raw, const unsigned L[4], int s, int g, unsigned C) {
    const unsigned w = raw.d[2 * s + g / 2];
    if constexpr (BITS == 4) {
        unsigned idx, pick;
        if (g % 2 == 0) {
            idx = w & 0x07070707u;
            pick = ((w >> 1) & 0x04040404u) | C;
        } else {
            idx = (w >> 4) & 0x07070707u;
            pick = ((w >> 5) & 0x04040404u) | C;
        }
        const unsigned a = perm(L[1], L[0], idx);
        const unsigned b = perm(L[3], L[2], idx);
        return perm(b, a, pick);
    } else {
        const unsigned idx = (g % 2 == 0 ? w : (w >> 4)) & 0x07070707u;
        return perm(L[1], L[0], idx);
    }
}

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
