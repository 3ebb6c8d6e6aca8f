// Pieces of the rotate + quantize kernels that rotate_quant.hip and qlinear_few.hip share: fp64 on the exact values of the bf16 inputs.
#pragma once
#include "lrq_internal.h"

#include <math.h>

namespace lrq {
namespace {

constexpr int kWave = 64;

__device__ __forceinline__ void load8_bf16(const uint16_t* __restrict__ p, double v[8]) {
    const uint4 raw = *reinterpret_cast<const uint4*>(p);
    const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = (double)__uint_as_float(w[i] << 16);
        v[2 * i + 1] = (double)__uint_as_float(w[i] & 0xffff0000u);
    }
}

// v[i] *= ps[i] for 8 consecutive channels: a bf16 value times an fp32 value is exact in fp64.
__device__ __forceinline__ void prescale8(const float* __restrict__ ps, double v[8]) {
    const float4 a = reinterpret_cast<const float4*>(ps)[0], b = reinterpret_cast<const float4*>(ps)[1];
    v[0] *= (double)a.x; v[1] *= (double)a.y; v[2] *= (double)a.z; v[3] *= (double)a.w;
    v[4] *= (double)b.x; v[5] *= (double)b.y; v[6] *= (double)b.z; v[7] *= (double)b.w;
}

// n-point butterfly network on v[0..n), ascending strides first_stride, 2*first_stride, ... for `stages`
// stages, (a, b) -> (a + b, a - b).
template <int N, int FIRST = 1>
__device__ __forceinline__ void butterflies(double* v, int stages) {
#pragma unroll
    for (int s = 0, st = FIRST; st < N; ++s, st <<= 1) {
        if (s < stages) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if ((i & st) == 0) {
                    const double a = v[i], b = v[i + st];
                    v[i] = a + b;
                    v[i + st] = a - b;
                }
            }
        }
    }
}

// ---- per-token quantizer ---------------------------------------------------------------------------------
// Symmetric form: amax = max |u|, inv = qmax / amax, code = rint(u * inv), scale = amax / (qmax sqrt(h)).
// Zero-point form (Eq. 1 as printed): range = max u - min u, L = 2^b - 1, inv = L / range, z = rint(min u * inv),
// x_q = clamp(rint(u * inv) - z, 0, L), s = range / L; stored as q = x_q - 2^(b-1) and zero = z + 2^(b-1), so
// that x_f = scale (q + zero), scale = s / sqrt(h).  A constant token takes x_q = 0 and (s, z) = (|c|, sign c).
struct RowQ {
    double inv;     // multiplier of u
    double zsub;    // zero-point form: what is subtracted from rint(u * inv) before the clamp to [-half, half-1]
    float scale;
    int izero;
};

__device__ __forceinline__ RowQ rowq_sym(double amax, const QuantSpec& qs) {
    RowQ r;
    r.inv = amax > 0.0 ? qs.qmax / amax : 0.0;
    r.zsub = 0.0;
    r.scale = (float)(amax / qs.norm);
    r.izero = 0;
    return r;
}

__device__ __forceinline__ RowQ rowq_asym(double vmax, double vmin, const QuantSpec& qs) {
    RowQ r;
    const double rng = vmax - vmin;
    double sc, z;
    if (rng > 0.0) {
        r.inv = qs.L / rng;
        sc = rng / qs.L;
        z = rint(vmin * r.inv);
        r.zsub = z + qs.half;
    } else {
        r.inv = 0.0;
        sc = vmin != 0.0 ? fabs(vmin) : 1.0;
        z = vmin > 0.0 ? 1.0 : (vmin < 0.0 ? -1.0 : 0.0);
        r.zsub = qs.half;                       // every code is x_q = 0, i.e. q = -2^(b-1)
    }
    r.scale = (float)(sc / qs.sqrt_h);
    r.izero = (int)(z + qs.half);
    return r;
}

constexpr double kMagic = 6755399441055744.0;   // 1.5 * 2^52: adding it rounds to an integer, ties to even

// One code (low byte of the result).  The product, the magic sum and the later steps round separately
// (this file is compiled with floating-point contraction off).
template <bool ASYM>
__device__ __forceinline__ unsigned code1(double u, const RowQ& p, double half) {
    if constexpr (!ASYM) {
        return (unsigned)__double2loint(u * p.inv + kMagic);
    } else {
        const double r = (u * p.inv + kMagic) - kMagic;
        const double t = fmin(fmax(r - p.zsub, -half), half - 1.0);
        return (unsigned)__double2loint(t + kMagic);
    }
}

// four codes -> one dword of int8
template <bool ASYM>
__device__ __forceinline__ unsigned pack4(const double* v, const RowQ& p, double half) {
    unsigned b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = code1<ASYM>(v[i], p, half);
    const unsigned lo = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u);
    return (hi << 16) | lo;
}

// Packed 4-bit codes: eight codes q[0..7] in [-7, 7] make one dword; byte j holds q[j] + 8 in its low nibble and
// q[4 + j] + 8 in its high nibble.  lo4 / hi4: the int8 codes q[0..3] / q[4..7], one per byte.
__device__ __forceinline__ unsigned pack_nibbles8(unsigned lo4, unsigned hi4) {
    return ((lo4 ^ 0x08080808u) & 0x0f0f0f0fu) | (((hi4 ^ 0x08080808u) & 0x0f0f0f0fu) << 4);
}

// Four int8 codes in [-7, 7] (one per byte) -> their FP8 E4M3 bit patterns: two 8-entry byte tables (0 .. 7 and the
// negative values by their low three bits) and a pick by the code's bit 3, which is set exactly for the negative ones.
__device__ __forceinline__ unsigned fp8x4_from_codes(unsigned w) {
    const unsigned idx = w & 0x07070707u;
    const unsigned pick = ((w >> 1) & 0x04040404u) | 0x03020100u;
    const unsigned pos = __builtin_amdgcn_perm(0x4e4c4a48u, 0x44403800u, idx);     // 0, 1, 2, 3 | 4, 5, 6, 7
    const unsigned neg = __builtin_amdgcn_perm(0xb8c0c4c8u, 0xcaccce00u, idx);   // -, -7, -6, -5 | -4, -3, -2, -1
    return __builtin_amdgcn_perm(neg, pos, pick);
}

// zero: NULL (symmetric form) or the zero-point form's output
inline QuantSpec make_spec(int act_bits, int h, int32_t* zero, const float* prescale = nullptr) {
    QuantSpec qs;
    qs.asym = zero != nullptr;
    qs.qmax = (double)((1 << (act_bits - 1)) - 1);
    qs.sqrt_h = sqrt((double)h);
    qs.norm = qs.qmax * qs.sqrt_h;
    qs.L = (double)((1 << act_bits) - 1);
    qs.half = (double)(1 << (act_bits - 1));
    qs.zero = zero;
    qs.prescale = prescale;
    qs.packed = 0;
    qs.fp8 = 0;
    return qs;
}

// order-preserving map of a double onto unsigned 64-bit keys (for LDS atomic max on signed values)
__device__ __forceinline__ unsigned long long okey(double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double okey_inv(unsigned long long k) {
    const unsigned long long b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
    return __longlong_as_double((long long)b);
}

constexpr int E32 = 32;

template <int CTRL>
__device__ __forceinline__ double quad_swap(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

}  // namespace
}  // namespace lrq
