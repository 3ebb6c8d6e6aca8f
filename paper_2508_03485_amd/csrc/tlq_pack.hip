// Twin-Log Quantization of a weight matrix: calibrate (search-based clipping), encode, build the
// per-channel int8 level table and pack (Method, "Twin-Log Quantization for Weights").  Offline step:
// one workgroup per output channel, fp64 throughout.
#include "lrq_internal.h"

namespace lrq {
namespace {

constexpr int NT = 256;
constexpr int kWave = 64;

struct Red4 {
    double pmax, pmin, nmax, nmin;
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}
__device__ __forceinline__ double wave_maxd(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}
__device__ __forceinline__ double wave_mind(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ __forceinline__ double block_sum(double v, double* red) {
    v = wave_sum(v);
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i) r += red[i];
    __syncthreads();
    return r;
}

__device__ __forceinline__ double clampd(double v, double lo, double hi) { return fmin(fmax(v, lo), hi); }

// ---- grid search of the clip factors (Eq. hyperparameters clip), both signs at once ------------------------------------
// A candidate is one value of the clip factor (and, in the extension with a lower clip, one value of gamma):
// s = (c W_max - g W_min) / intervals, z = round(g W_min / s); its objective per sign is sum (W_f - W)^2 over the weights of
// that sign.  The sum has a fixed order: thread j adds the terms of k = j, j + NT, j + 2 NT, ... one after the other, then
// the NT partial sums are added in ascending j - so which of two close candidates is the smaller one does not depend on a
// reduction tree.
// What bounds the search: fp64 vector work, about twenty instructions per weight and candidate.  It is arranged so that little
// else is left:
//   * a weight belongs to one sign, so one pass over the weights serves both searches (no idle lanes in a pass per sign);
//   * a candidate has at most eight levels per sign, so exp2 runs once per level (into an LDS table), not once per weight;
//   * the quotient W' / s is a multiplication by 1 / s: with |W' / s| <= 2^20 the product is within 2^-31 of the quotient,
//     which settles the rounding unless it lies within 1e-7 of a half-integer - only then is the division itself taken;
//   * NC candidates go together: their ordered sums, 256 dependent additions each, run side by side in 2 NC lanes
//     instead of one after the other in every lane;
//   * a thread's weights and their logarithms stay in registers (K <= 6144), longer rows keep the logarithms in LDS.
// Measured at 4608 x 1152 with 21 candidates per sign: 1490 us with a pass per sign, an exp2 and a division per weight and
// candidate and one ordered sum after the other; 177 us in this form with selects by sign, 169 us with masks
// (about 65 us of them the logarithms, the encoding and the packing, 5 us each candidate).
constexpr int PSTRIDE = NT + 1;          // one double of padding: the lanes that sum in parallel read distinct banks
constexpr double kMagic = 6755399441055744.0;   // 1.5 * 2^52: adding it rounds to an integer, ties to even

struct Candidate {
    double s, inv, z;
    int zlow;                            // z + lowest level index of the sign
    int mode;                            // 0: skipped, 1: 1 / s settles the rounding (see above) and levels have finite squares, 2: always divide
};

// NC candidates per pass: 8 (NC * 2 * 257 doubles of partial sums are 33 KB: four workgroups per CU), 4 where a row of
// logarithms leaves no room for more.
template <int NC>
struct __attribute__((aligned(16))) SearchLds {
    double part[NC][2][PSTRIDE];
    double level[NC][2][8];
    Candidate cand[NC][2];
    double err[NC][2];
    double best_err[2], best_s[2], best_z[2];
    float best_c[2], best_g[2];
};

__device__ __forceinline__ double log2_abs(double w) { return w != 0.0 ? log2(fabs(w)) : 0.0; }
__device__ __forceinline__ double level_index(double ell, double s, double z, double qlo, double qhi) {
    return clampd(rint(ell / s) - z, qlo, qhi);
}

// Elements k = base + e NT + t of the row, e < NE: REGS: the row fits NT * NE elements and el / wv hold it all along; otherwise
// they are read from ell (LDS) and w for every pass.
template <int NE, bool REGS, int NC, bool MASKS>
__device__ void search_clip(const float* __restrict__ w, const double* __restrict__ ell, double (&el)[NE], float (&wv)[NE], int K,
                            const bool (&has)[2], const double (&wmax)[2], const double (&wmin)[2],
                            const float* __restrict__ agrid, int na, const float* __restrict__ bgrid, int nb,
                            const float* __restrict__ ggrid, int ngamma, int half, SearchLds<NC>& S) {
    const int t = threadIdx.x;
    const int ng = ngamma > 0 ? ngamma : 1;
    const int total = (na > nb ? na : nb) * ng;
    if (t < 2) {
        S.best_err[t] = INFINITY;
        S.best_s[t] = 1.0;
        S.best_z[t] = has[t] ? rint(wmin[t]) : 0.0;
        S.best_c[t] = 1.0f;
        S.best_g[t] = 1.0f;
    }
    // MASKS: 1.0 where the weight has the sign, 0.0 elsewhere.  A fused multiply-add by it adds the square or + 0.0 exactly as a
    // select and an addition do, in one instruction instead of three (the loop is bound by issue).  It needs finite squares:
    // threads with an infinity or a NaN always take the general form, and so do candidates with huge levels (mode 2).
    // Which grids take them: masks_from.
    static_assert(REGS || !MASKS, "the masks belong to weights in registers");
    double is_pos[MASKS ? NE : 1], is_neg[MASKS ? NE : 1];
    bool not_finite = false;
    if constexpr (MASKS) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            is_pos[e] = wv[e] > 0.0f ? 1.0 : 0.0;
            is_neg[e] = wv[e] < 0.0f ? 1.0 : 0.0;
            not_finite |= !(fabsf(wv[e]) < INFINITY);
            asm volatile("" : "+v"(is_pos[e]), "+v"(is_neg[e]));              // kept, not derived again
        }
    }
    for (int c0 = 0; c0 < total; c0 += NC) {
        const int nc = total - c0 < NC ? total - c0 : NC;
        if (t < NC * 2) {
            const int j = t / 2, side = t % 2, ci = (c0 + j) / ng, gi = (c0 + j) % ng;
            Candidate c = {1.0, 1.0, 0.0, 0, 0};
            if (j < nc && ci < (side ? nb : na) && has[side]) {
                const float c32 = side ? bgrid[ci] : agrid[ci], g32 = ngamma > 0 ? ggrid[gi] : 1.0f;
                const double T = (double)c32 * wmax[side], B = (double)g32 * wmin[side];
                if (T > B) {
                    c.s = (T - B) / (double)(side ? half : half - 1);
                    c.z = rint(B / c.s);
                    c.inv = 1.0 / c.s;
                    c.mode = fmax(fmax(fabs(wmax[side]), fabs(wmin[side])) * c.inv, fabs(c.z)) <= 1048576.0 &&
                                     fmax(fabs(T), fabs(B)) <= 240.0 ? 1 : 2;        // levels below 2^480: finite squares
                    c.zlow = c.mode == 1 ? (int)c.z + side : 0;
                }
            }
            S.cand[j][side] = c;
        }
        __syncthreads();
        if (t < NC * 16) {
            const int j = t / 16, side = (t / 8) % 2, i = t % 8;
            const Candidate c = S.cand[j][side];
            if (i < half) S.level[j][side][i] = c.mode ? exp2(c.s * ((double)(i + side) + c.z)) : 0.0;   // skipped: finite all the same
        }
        __syncthreads();
        for (int base = 0; base < K; base += NT * NE) {
            if constexpr (!REGS) {
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    const int k = base + e * NT + t;
                    wv[e] = k < K ? w[k] : 0.0f;
                    el[e] = k < K ? ell[k] : 0.0;
                }
            }
            for (int j = 0; j < nc; ++j) {
                const Candidate cp = S.cand[j][0], cn = S.cand[j][1];
                double ep = base ? S.part[j][0][t] : 0.0, en = base ? S.part[j][1][t] : 0.0;
                const double ep0 = ep, en0 = en;
                bool unsettled = cp.mode == 2 || cn.mode == 2 || not_finite;
                // what is derived from a weight (sign, double) is derived again for every candidate, not kept in registers
#pragma unroll
                for (int e = 0; e < NE; ++e) asm volatile("" : "+v"(wv[e]));
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    const bool neg = wv[e] < 0.0f;
                    const double y = el[e] * (neg ? cn.inv : cp.inv);
                    const double m = y + kMagic;
                    unsettled |= !(fabs(y - (m - kMagic)) < 0.4999999);
                    const int i = min(max(__double2loint(m) - (neg ? cn.zlow : cp.zlow), 0), half - 1);
                    const double d = S.level[j][neg ? 1 : 0][i] - fabs((double)wv[e]);
                    const double d2 = d * d;
                    if constexpr (MASKS) {                        // d2 or + 0.0, which leaves the other sign's sum as it is
                        ep = fma(d2, is_pos[e], ep);
                        en = fma(d2, is_neg[e], en);
                    } else {
                        ep = ep + (wv[e] > 0.0f ? d2 : 0.0);
                        en = en + (neg ? d2 : 0.0);
                    }
                    if (e % 3 == 2) __builtin_amdgcn_sched_barrier(0);   // three in flight
                }
                if (unsettled) {                                  // rare: this thread's terms again, with the quotient itself
                    ep = ep0;
                    en = en0;
#pragma unroll
                    for (int e = 0; e < NE; ++e) {
                        const double wk = (double)wv[e];
                        const bool neg = wk < 0.0;
                        if (neg || wk > 0.0) {                    // a NaN weight belongs to neither sign
                            const double s = neg ? cn.s : cp.s, z = neg ? cn.z : cp.z, lo = neg ? 1.0 : 0.0;
                            const double d = exp2(s * (level_index(el[e], s, z, lo, lo + (double)(half - 1)) + z)) - fabs(wk);
                            if (neg) en = en + d * d; else ep = ep + d * d;
                        }
                        __builtin_amdgcn_sched_barrier(0);        // one element after the other: few registers
                    }
                }
                S.part[j][0][t] = ep;
                S.part[j][1][t] = en;
            }
        }
        __syncthreads();
        if (t < 2 * nc) {
            const double* p = S.part[t / 2][t % 2];
            // eight values are fetched while the eight before them are added: the chain then waits for its additions only
            double cur[8], nxt[8], r = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) cur[i] = p[i];
#pragma unroll 16
            for (int b = 8; b <= NT; b += 8) {
                const int at = b < NT ? b : 0;
#pragma unroll
                for (int i = 0; i < 8; ++i) nxt[i] = p[at + i];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 8; ++i) r = r + cur[i];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 8; ++i) cur[i] = nxt[i];
            }
            S.err[t / 2][t % 2] = S.cand[t / 2][t % 2].mode ? r : INFINITY;
        }
        __syncthreads();
        if (t < 2) {                                          // first minimum wins, candidates in grid order
            for (int j = 0; j < nc; ++j) {
                const double e = S.err[j][t];
                if (S.cand[j][t].mode && e < S.best_err[t]) {
                    S.best_err[t] = e;
                    S.best_s[t] = S.cand[j][t].s;
                    S.best_z[t] = S.cand[j][t].z;
                    S.best_c[t] = (t ? bgrid : agrid)[(c0 + j) / ng];
                    S.best_g[t] = ngamma > 0 ? ggrid[(c0 + j) % ng] : 1.0f;
                }
            }
        }
        __syncthreads();
    }
}

// Round-to-nearest-even bf16 of a double.  The detour over fp32 could round twice only when the fp32 value lands
// exactly on a bf16 midpoint; the sign of what the first rounding dropped then decides the tie.
__device__ __forceinline__ uint16_t f64_to_bf16_rne(double x) {
    const float f = (float)x;
    unsigned u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);     // inf / nan
    const double d = fabs(x) - fabs((double)f);
    if ((u & 0xffffu) == 0x8000u && d != 0.0) return (uint16_t)((u >> 16) + (d > 0.0 ? 1u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Round-to-nearest-even FP8 E4M3 (1 sign, 4 exponent bits with bias 7, 3 mantissa bits, no infinities, largest value
// 448, subnormals in steps of 2^-9) of a double, saturating.
__device__ __forceinline__ uint8_t f64_to_e4m3_rne(double x) {
    const unsigned sgn = x < 0.0 ? 0x80u : 0u;
    const double a = fmin(fabs(x), 448.0);
    if (!(a > 0.0)) return (uint8_t)sgn;
    int e = ilogb(a);
    e = e < -6 ? -6 : e;                                   // below 2^-6 everything shares the subnormal spacing
    double n = rint(ldexp(a, 3 - e));                      // multiples of 2^(e - 3): 8 .. 16 for a normal, 0 .. 8 below
    if (n >= 16.0) { n = 8.0; ++e; }
    if (e > 8 || (e == 8 && n > 14.0)) return (uint8_t)(sgn | 0x7eu);
    if (n < 8.0) return (uint8_t)(sgn | (unsigned)n);      // subnormal (n = 8 at e = -6 is the smallest normal)
    return (uint8_t)(sgn | ((unsigned)(e + 7) << 3) | ((unsigned)n - 8u));
}

template <int NE, bool REGS, int NC, bool MASKS>
__global__ __launch_bounds__(NT, !REGS || NE > 12 ? 2 : (NE > 6 ? 3 : 4)) void tlq_quantize_pack_kernel(
    const float* __restrict__ W, int N, int K, int bits, int I, const float* __restrict__ agrid, int na,
    const float* __restrict__ bgrid, int nb, uint8_t* __restrict__ codes_out, double* __restrict__ s_pos,
    double* __restrict__ s_neg, int32_t* __restrict__ z_pos, int32_t* __restrict__ z_neg,
    float* __restrict__ alpha, float* __restrict__ beta, int8_t* __restrict__ lut, float* __restrict__ wscale,
    uint8_t* __restrict__ gemm_codes, int32_t* __restrict__ colsum, const float* __restrict__ ggrid, int ngamma,
    float* __restrict__ gamma_pos, float* __restrict__ gamma_neg, uint16_t* __restrict__ levels,
    double* __restrict__ err_pos, double* __restrict__ err_neg, uint8_t* __restrict__ lut_fp8, float* __restrict__ wscale_fp8) {
    // LDS: search state (its partial sums double as reduction scratch outside the search), then the row: its logarithms, each
    // of which later gives its low byte to the code (REGS: codes only)
    extern __shared__ __attribute__((aligned(16))) unsigned char sm[];
    SearchLds<NC>& S = *reinterpret_cast<SearchLds<NC>*>(sm);
    double* red = &S.part[0][0][0];
    double* ell = reinterpret_cast<double*>(sm + sizeof(SearchLds<NC>));
    int8_t* code = reinterpret_cast<int8_t*>(ell);
    constexpr int CS = REGS ? 1 : 8;                    // bytes from one code to the next
    const int n = blockIdx.x, t = threadIdx.x;
    const float* w = W + (size_t)n * K;
    const int half = 1 << (bits - 1), nlev = 1 << bits;

    // W' = log2|W| and the per-sign extrema over the masked positions
    double pmax = -INFINITY, pmin = INFINITY, nmax = -INFINITY, nmin = INFINITY;
    double el[NE];
    float wv[NE];
    auto logarithm = [&](float wk32) {
        const double wk = (double)wk32;
        const double l = log2_abs(wk);
        if (wk > 0.0) { pmax = fmax(pmax, l); pmin = fmin(pmin, l); }
        if (wk < 0.0) { nmax = fmax(nmax, l); nmin = fmin(nmin, l); }
        return l;
    };
    if constexpr (REGS) {
#pragma unroll
        for (int e = 0; e < NE; ++e) wv[e] = e * NT + t < K ? w[e * NT + t] : 0.0f;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            el[e] = logarithm(wv[e]);
            __builtin_amdgcn_sched_barrier(0);           // one element after the other: few registers
        }
    } else {
        for (int k = t; k < K; k += NT) ell[k] = logarithm(w[k]);
    }
    pmax = wave_maxd(pmax); pmin = wave_mind(pmin); nmax = wave_maxd(nmax); nmin = wave_mind(nmin);
    Red4* r4 = reinterpret_cast<Red4*>(red);
    if (t % kWave == 0) r4[t / kWave] = Red4{pmax, pmin, nmax, nmin};
    __syncthreads();
    for (int i = 0; i < NT / kWave; ++i) {
        pmax = fmax(pmax, r4[i].pmax); pmin = fmin(pmin, r4[i].pmin);
        nmax = fmax(nmax, r4[i].nmax); nmin = fmin(nmin, r4[i].nmin);
    }
    __syncthreads();
    const bool has_p = pmax >= pmin, has_n = nmax >= nmin;   // +-inf sentinels survive on an empty side
    if (!has_p) pmax = pmin = 0.0;
    if (!has_n) nmax = nmin = 0.0;

    const bool has[2] = {has_p, has_n};
    const double wmax[2] = {pmax, nmax}, wmin[2] = {pmin, nmin};
    search_clip<NE, REGS, NC, MASKS>(w, ell, el, wv, K, has, wmax, wmin, agrid, na, bgrid, nb, ggrid, ngamma, half, S);
    const double sp = S.best_s[0], zp = S.best_z[0], ep = S.best_err[0], sn = S.best_s[1], zn = S.best_z[1], en = S.best_err[1];
    const float al = S.best_c[0], be = S.best_c[1], gp = S.best_g[0], gn = S.best_g[1];

    if (t == 0) {
        s_pos[n] = sp; s_neg[n] = sn; z_pos[n] = (int32_t)zp; z_neg[n] = (int32_t)zn;
        alpha[n] = al; beta[n] = be;
        if (gamma_pos) gamma_pos[n] = gp;
        if (gamma_neg) gamma_neg[n] = gn;
        if (err_pos) err_pos[n] = ep;
        if (err_neg) err_neg[n] = en;
    }

    // level table: e(c) = s+(c + z+) for c >= 0, s-(-c + z-) for c < 0; exponent split and integerisation
    double v = 0.0;
    if (t < nlev) {
        const int c = t < half ? t : t - nlev;              // signed code whose low bits are t
        const double e = c >= 0 ? sp * ((double)c + zp) : sn * ((double)(-c) + zn);
        double mag;
        if (I < 0) {
            mag = exp2(e);
        } else {
            const double f = floor(e), r = e - f;
            const double mant = rint(exp2(r) * (double)(1 << I));
            mag = ldexp(mant, (int)f - I);
        }
        v = c >= 0 ? mag : -mag;
        red[t] = fabs(v);
    }
    __syncthreads();
    double vmax = 0.0;
    for (int i = 0; i < nlev; ++i) vmax = fmax(vmax, red[i]);
    const float ws = (float)(vmax / 127.0);
    __shared__ int lutv[16];
    if (t < 16) {
        int8_t entry = 0;
        if (t < nlev) entry = (int8_t)(int)clampd(rint(v / (double)ws), -127.0, 127.0);
        lut[(size_t)n * 16 + t] = entry;
        lutv[t] = entry;
        if (levels) levels[(size_t)n * 16 + t] = t < nlev ? f64_to_bf16_rne(v) : (uint16_t)0;
    }
    if (t == 0) wscale[n] = ws;

    // the same levels with I = 3 as FP8 E4M3 operands: divided by the power of two that puts the largest in [128, 256)
    if (lut_fp8 && wscale_fp8) {
        __syncthreads();
        double v3 = 0.0;
        if (t < nlev) {
            const int c = t < half ? t : t - nlev;
            const double e = c >= 0 ? sp * ((double)c + zp) : sn * ((double)(-c) + zn);
            const double f = floor(e), r = e - f;
            const double mag = ldexp(rint(exp2(r) * 8.0), (int)f - 3);
            v3 = c >= 0 ? mag : -mag;
            red[t] = mag;
        }
        __syncthreads();
        double m3 = 0.0;
        for (int i = 0; i < nlev; ++i) m3 = fmax(m3, red[i]);
        const int ex = (m3 > 0.0 ? ilogb(m3) : 0) - 7;
        if (t < 16) lut_fp8[(size_t)n * 16 + t] = t < nlev ? f64_to_e4m3_rne(ldexp(v3, -ex)) : (uint8_t)0;
        if (t == 0) wscale_fp8[n] = ldexpf(1.0f, ex);
        __syncthreads();
    }

    // codes (Eq. log-based quantizer); the negative twin is clamped to [1, 2^(b-1)]
    auto encode = [&](int k, double l, float wk) {
        const bool neg = wk < 0.0f;
        const double lo = neg ? 1.0 : 0.0;
        const int c = (int)level_index(l, neg ? sn : sp, neg ? zn : zp, lo, lo + (double)(half - 1));
        code[k * CS] = (int8_t)(wk == 0.0f ? 0 : (neg ? -c : c));
    };
    if constexpr (REGS) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            if (e * NT + t < K) encode(e * NT + t, el[e], wv[e]);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        for (int k = t; k < K; k += NT) encode(k, ell[k], w[k]);
    }
    __syncthreads();

    const unsigned mask = (unsigned)nlev - 1u;
    {   // sum of the channel's decoded levels (exact in fp64: |sum| <= 127 K)
        double part = 0.0;
        for (int k = t; k < K; k += NT) part += (double)lutv[(unsigned)code[k * CS] & mask];
        const double tot = block_sum(part, red);
        if (t == 0) colsum[n] = (int32_t)tot;
    }
    if (bits == 4) {
        // canonical: byte j = code[2j] | code[2j+1] << 4, written 4 bytes at a time
        uint32_t* dst = reinterpret_cast<uint32_t*>(codes_out + (size_t)n * (K / 2));
        for (int g = t; g < K / 8; g += NT) {
            unsigned canon = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) canon |= ((unsigned)code[(g * 8 + i) * CS] & mask) << (4 * i);
            dst[g] = canon;
        }
    } else {
        // canonical: 8 codes -> 24-bit little-endian group
        uint8_t* dst = codes_out + (size_t)n * (K / 8 * 3);
        for (int g = t; g < K / 8; g += NT) {
            unsigned v24 = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) v24 |= ((unsigned)code[(g * 8 + i) * CS] & mask) << (3 * i);
            dst[g * 3 + 0] = (uint8_t)(v24 & 255u);
            dst[g * 3 + 1] = (uint8_t)((v24 >> 8) & 255u);
            dst[g * 3 + 2] = (uint8_t)(v24 >> 16);
        }
    }
    // GEMM layout, either bit-width: one nibble per code (a 3-bit code leaves its top bit clear, so that a single
    // AND turns a dword into four byte-permute selectors); byte j of a dword = code[k+j] | code[k+4+j] << 4
    for (int g = t; g < K / 8; g += NT) {
        unsigned tiled = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            tiled |= (((unsigned)code[(g * 8 + j) * CS] & mask) | (((unsigned)code[(g * 8 + 4 + j) * CS] & mask) << 4)) << (8 * j);
        // slot (n % 16, 16-k group kq) of the unit; the channel's half of its 32-tile picks the slot's 8-byte half
        const int kb = g / 8, r = g % 8, kq = r / 2, d = r % 2;
        const size_t unit = (size_t)(n / kGemmTileN) * (K / kGemmBlockK) + kb;
        const size_t off = (unit * 64 + (n % 16) + 16 * kq) * 16 + (((n % kGemmTileN) / 16) * 2 + d) * 4;
        *reinterpret_cast<uint32_t*>(gemm_codes + off) = tiled;
    }
}

}  // namespace

// From how many candidates on a search with ne weights a thread adds through masks: they take 4 ne registers, to be set up and, at the
// occupancy that the launch bounds ask for, spilled in part (3, 5, 6, 9, 12 weights: 2, 4, 11, 2, 25 registers), and save
// instructions of every candidate.  us with selects / with masks for 1, 4, 8, 21 candidates: 4608 x 768 50.8 / 51.4, 60.8 / 60.7,
// 74.8 / 73.8, 140.2 / 135.2; 4608 x 1152 57.9 / 59.0, 72.1 / 72.0, 91.9 / 89.7, 176.9 / 169.3; 4096 x 1536 57.8 / 59.8,
// 71.9 / 72.8, 91.8 / 90.0, 175.3 / 168.6; 4000 x 2304 82.4 / 83.2, 104.3 / 102.7, 133.1 / 128.1, 248.5 / 232.8; 9216 x 3072
// 201.9 / 221.9, 265.5 / 282.5, 345.4 / 355.7, 671.9 / 643.6 (16 candidates: 561.1 / 557.5); 1152 x 4608 54.0 / 54.8, 68.7 / 68.0,
// 88.7 / 85.5, 166.6 / 155.0.  24 weights a thread lose at 21 candidates too (1500 x 6144: 245 / 277).
static int masks_from(int ne) { return ne <= 5 ? 4 : (ne <= 6 ? 6 : (ne <= 9 ? 3 : (ne <= 12 ? 16 : 3))); }

hipError_t launch_tlq_quantize_pack(hipStream_t st, const float* W, int N, int K, int bits, int I,
                                    const float* alpha_grid, int n_alpha, const float* beta_grid, int n_beta,
                                    const lrq_tlq_weight& out, const float* gamma_grid, int n_gamma, float* gamma_pos,
                                    float* gamma_neg) {
    // Weights per thread: the smallest count that holds the row (K = 1152 fills 4.5 of 5); above 6144 the row goes through the
    // registers in passes of 16.  There the row's logarithms leave room for few partial sums beside a second workgroup on the CU: a
    // grid of one or two candidates takes two at a time (6528 x 8328, one candidate: 860 us, eight at a time 1076).
    auto go = [&](auto kernel, size_t lds) {
        const hipError_t e = allow_large_lds(reinterpret_cast<const void*>(kernel), 158 * 1024);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(N), dim3(NT), lds, st, W, N, K, bits, I, alpha_grid, n_alpha, beta_grid, n_beta, out.codes,
                           out.s_pos, out.s_neg, out.z_pos, out.z_neg, out.alpha, out.beta, out.lut, out.wscale, out.gemm_codes,
                           out.colsum, gamma_grid, n_gamma, gamma_pos, gamma_neg, out.levels, out.err_pos, out.err_neg,
                           out.lut_fp8, out.wscale_fp8);
        return hipGetLastError();
    };
    const int ne = (K + NT - 1) / NT, candidates = (n_alpha > n_beta ? n_alpha : n_beta) * (n_gamma > 0 ? n_gamma : 1);
    const size_t lds = sizeof(SearchLds<8>) + (size_t)K;
#define LRQ_REGS(NE) \
    if (ne <= NE) return candidates >= masks_from(NE) ? go(tlq_quantize_pack_kernel<NE, true, 8, true>, lds) : go(tlq_quantize_pack_kernel<NE, true, 8, false>, lds);
    LRQ_REGS(3) LRQ_REGS(5) LRQ_REGS(6) LRQ_REGS(9) LRQ_REGS(12) LRQ_REGS(18)
#undef LRQ_REGS
    if (ne <= 24) return go(tlq_quantize_pack_kernel<24, true, 8, false>, lds);
    const size_t row = (size_t)K * sizeof(double);
    if (candidates <= 2) return go(tlq_quantize_pack_kernel<16, false, 2, false>, sizeof(SearchLds<2>) + row);
    if (K <= 12288) return go(tlq_quantize_pack_kernel<16, false, 8, false>, sizeof(SearchLds<8>) + row);
    return go(tlq_quantize_pack_kernel<16, false, 4, false>, sizeof(SearchLds<4>) + row);
}

}  // namespace lrq
