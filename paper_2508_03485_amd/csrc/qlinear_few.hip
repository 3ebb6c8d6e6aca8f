// The linear layer on a few tokens in one launch (gfx950): conditioning linears of a handful of tokens, whose time is
// launches and latency.  As two kernels 2 x 1152 -> 6912 took 2.8 + 3.7 us and the gap between them.  Here every workgroup rotates and
// quantizes all rows itself (M K <= kFewElements: 32 elements a thread, once; the same stages in the same order as the kernels of rotate_quant.hip,
// so the same codes) while its first weight codes are on their way, keeps the codes in LDS and multiplies its 32 channels as
// qgemm_small_kernel does: K split over eight waves, integer partial sums joined in LDS.  Bound by latency: one trip to memory for x and the
// codes, the row maximum's barrier, the join.
#include "qgemm_common.h"
#include "rotate_common.h"

namespace lrq {
namespace {

constexpr int BK = kGemmBlockK;
constexpr int SW = 8;                                // waves of a workgroup
constexpr int kFewElements = 32 * 64 * SW;           // 16384
constexpr int UB = 3;                                // K blocks in flight per wave
constexpr int EX_ROW = 34;                           // doubles of a thread in the exchange of the longer blocks
constexpr int PART_BYTES = SW * 2 * 64 * 16;

// codes (rows of K + 16 bytes), then the exchange of blocks past 128 or the partial sums
inline size_t lds_bytes(int M, int K, int h) {
    const size_t codes = ((size_t)M * (K + 16) + 15) & ~(size_t)15;
    const size_t exch = h > 128 ? (size_t)M * (K / E32) * EX_ROW * sizeof(double) : 0;
    return codes + (exch > PART_BYTES ? exch : PART_BYTES);
}

// LOG2H: 5 stands for blocks of up to 32 (log2h at run time, 0 = no rotation), 6 .. 10 for 64 .. 1024
template <int BITS, int LOG2H, bool ASYM>
__global__ __launch_bounds__(64 * SW) void qlinear_few_kernel(const uint16_t* __restrict__ X, int M, int K, int log2h, QuantSpec qs, int N,
                                                              const uint8_t* __restrict__ gcodes, const int8_t* __restrict__ lut,
                                                              const float* __restrict__ wscale, const float* __restrict__ bias, int out_fp32,
                                                              void* __restrict__ Y, const int32_t* __restrict__ colsum) {
    constexpr int UNIT = 64 * 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];      // codes, then exchange / partial sums
    __shared__ unsigned long long amax_bits[2][16];
    __shared__ float scale[16];
    __shared__ int zero[16];
    const int t = threadIdx.x, lane = t % 64, wv = t / 64, tn = blockIdx.x;
    const int KB = K / BK, crow = K + 16, lpr = K / E32;
    unsigned char* const codes = lds;
    double* const ex = reinterpret_cast<double*>(lds + (size_t)((M * crow + 15) & ~15));

    // weights: level tables of the lane's two channels, codes of the wave's first blocks
    unsigned L[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        int n = tn * 32 + h * 16 + lane % 16;
        if (n >= N) n = N - 1;
        const uint4 lv = *reinterpret_cast<const uint4*>(lut + (size_t)n * 16);
        L[h][0] = lv.x; L[h][1] = lv.y; L[h][2] = lv.z; L[h][3] = lv.w;
    }
    const uint8_t* bptr = gcodes + (size_t)tn * KB * UNIT + (size_t)lane * 16;
    BRaw<BITS> b[UB];
    auto load_b = [&](int kb0) {
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int kb = kb0 + u * SW < KB ? kb0 + u * SW : KB - 1;          // past the end: loaded, not used
            b[u] = load_braw<BITS>(bptr + (size_t)kb * UNIT);
        }
    };
    load_b(wv);

    // ---- rotate and quantize: thread t holds 32 neighbouring elements of row t / lpr
    const int rw = t / lpr, slot = t % lpr;
    const bool live = rw < M;
    double v[E32];
    {
        const uint16_t* src = X + (size_t)(live ? rw : M - 1) * K + (size_t)slot * E32;
#pragma unroll
        for (int c = 0; c < 4; ++c) load8_bf16(src + c * 8, v + c * 8);
        if (qs.prescale) {
#pragma unroll
            for (int c = 0; c < 4; ++c) prescale8(qs.prescale + slot * E32 + c * 8, v + c * 8);
        }
    }
    if (t < 32) amax_bits[t / 16][t % 16] = 0ull;
    butterflies<E32>(v, LOG2H == 5 ? log2h : 5);
    if constexpr (LOG2H == 6 || LOG2H == 7) {
        const double sg = (t & 1) ? -1.0 : 1.0;
#pragma unroll
        for (int i = 0; i < E32; ++i) v[i] = fma(v[i], sg, quad_swap<0xB1>(v[i]));
    }
    if constexpr (LOG2H == 7) {
        const double sg = (t & 2) ? -1.0 : 1.0;
#pragma unroll
        for (int i = 0; i < E32; ++i) v[i] = fma(v[i], sg, quad_swap<0x4E>(v[i]));
    }
    // longer blocks: the G lanes of a block, neighbours in one wave, exchange it transposed; afterwards lane j holds the elements
    // 32 r + e0 + k, r = 0 .. G - 1, k = 0 .. EPL - 1
    constexpr int G = LOG2H >= 8 ? 1 << (LOG2H - 5) : 1, EPL = 32 / G;
    const int j = t % G, e0 = j * EPL;
    if constexpr (LOG2H >= 8) {
        double2* dst = reinterpret_cast<double2*>(ex + (size_t)t * EX_ROW);
        if (live) {
#pragma unroll
            for (int i = 0; i < E32 / 2; ++i) dst[i] = make_double2(v[2 * i], v[2 * i + 1]);
        }
        wave_sync();
        if (live) {
#pragma unroll
            for (int r = 0; r < G; ++r)
#pragma unroll
                for (int k = 0; k < EPL; ++k) v[r * EPL + k] = ex[(size_t)(t - j + r) * EX_ROW + e0 + k];
        }
        butterflies<E32, EPL>(v, LOG2H - 5);
    }
    double m = ASYM ? -INFINITY : 0.0, m2 = -INFINITY;
#pragma unroll
    for (int i = 0; i < E32; ++i) {
        if constexpr (ASYM) { m = fmax(m, v[i]); m2 = fmax(m2, -v[i]); }
        else m = fmax(m, fabs(v[i]));
    }
    m = fmax(m, quad_swap<0xB1>(m));
    m = fmax(m, quad_swap<0x4E>(m));
    if constexpr (ASYM) {
        m2 = fmax(m2, quad_swap<0xB1>(m2));
        m2 = fmax(m2, quad_swap<0x4E>(m2));
    }
    __syncthreads();
    if (live && (t & 3) == 0) {
        if constexpr (ASYM) {
            atomicMax(&amax_bits[0][rw], okey(m));
            atomicMax(&amax_bits[1][rw], okey(m2));
        } else {
            atomicMax(&amax_bits[0][rw], (unsigned long long)__double_as_longlong(m));
        }
    }
    __syncthreads();
    if (live) {
        RowQ p;
        if constexpr (ASYM) p = rowq_asym(okey_inv(amax_bits[0][rw]), -okey_inv(amax_bits[1][rw]), qs);
        else p = rowq_sym(__longlong_as_double((long long)amax_bits[0][rw]), qs);
        if (slot == 0) {
            scale[rw] = p.scale;
            if constexpr (ASYM) zero[rw] = p.izero;
        }
        unsigned char* dst = codes + (size_t)rw * crow;
        if constexpr (LOG2H < 8) {
            unsigned out[8];
#pragma unroll
            for (int g = 0; g < 8; ++g) out[g] = pack4<ASYM>(v + 4 * g, p, qs.half);
            uint4* d4 = reinterpret_cast<uint4*>(dst + slot * E32);
            d4[0] = make_uint4(out[0], out[1], out[2], out[3]);
            d4[1] = make_uint4(out[4], out[5], out[6], out[7]);
        } else {
            dst += (slot - j) * E32 + e0;
#pragma unroll
            for (int r = 0; r < G; ++r)
#pragma unroll
                for (int k = 0; k < EPL; ++k) dst[r * 32 + k] = (unsigned char)code1<ASYM>(v[r * EPL + k], p, qs.half);
        }
    }
    __syncthreads();

    // ---- product: this wave's K blocks
    unsigned C = 0x03020100u;
    asm volatile("" : "+v"(C));
    const unsigned char* aptr = codes + (size_t)(lane % 16 < M ? lane % 16 : M - 1) * crow + (lane / 16) * 16;
    v4i acc[2] = {v4i{0, 0, 0, 0}, v4i{0, 0, 0, 0}};
    for (int kb0 = wv; kb0 < KB; kb0 += SW * UB) {
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int kb = kb0 + u * SW;
            if (kb < KB) {
                const v4i a = *reinterpret_cast<const v4i*>(aptr + (size_t)kb * BK);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v4i bd;
#pragma unroll
                    for (int g = 0; g < 4; ++g) bd[g] = (int)decode_dword<BITS>(b[u], L[h], h, g, C);
                    acc[h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bd, a, acc[h], 0, 0, 0);
                }
            }
        }
        if (kb0 + SW * UB < KB) load_b(kb0 + SW * UB);
    }
    v4i(*part)[2][64] = reinterpret_cast<v4i(*)[2][64]>(ex);                // the exchange is over
    part[wv][0][lane] = acc[0];
    part[wv][1][lane] = acc[1];
    __syncthreads();
    // one thread per (accumulator tile, lane): token lane % 16, four neighbouring channels
    if (t < 128) {
        const int tile = t / 64, row = lane % 16, n = tn * 32 + tile * 16 + 4 * (lane / 16);
        if (row < M && n < N) {
            v4i s = part[0][tile][lane];
#pragma unroll
            for (int w = 1; w < SW; ++w) s += part[w][tile][lane];
            const float sv = scale[row];
            const double zv = ASYM ? (double)zero[row] : 0.0;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                if (n + x < N) {
                    const float tot = ASYM ? zp_sum(s[x], zv, (double)colsum[n + x]) : (float)s[x];
                    const float y = (tot * sv) * wscale[n + x] + (bias ? bias[n + x] : 0.0f);
                    const size_t at = (size_t)row * N + n + x;
                    if (out_fp32) reinterpret_cast<float*>(Y)[at] = y;
                    else reinterpret_cast<uint16_t*>(Y)[at] = (uint16_t)pack_bf16(y, 0.0f);
                }
            }
        }
    }
}

template <int BITS, int LOG2H>
hipError_t launch(hipStream_t st, const uint16_t* X, int M, int K, int log2h, const QuantSpec& qs, const lrq_tlq_weight& w, const float* bias,
                  int fp32, void* Y) {
    const size_t bytes = lds_bytes(M, K, 1 << log2h);
    const dim3 grid((w.N + 31) / 32), block(64 * SW);
    auto go = [&](auto kernel) {
        if (bytes > 60 * 1024) {
            const hipError_t e = allow_large_lds(reinterpret_cast<const void*>(kernel), 158 * 1024);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, grid, block, bytes, st, X, M, K, log2h, qs, w.N, w.gemm_codes, w.lut, w.wscale, bias, fp32, Y, w.colsum);
        return hipGetLastError();
    };
    return qs.asym ? go(qlinear_few_kernel<BITS, LOG2H, true>) : go(qlinear_few_kernel<BITS, LOG2H, false>);
}

template <int BITS>
hipError_t launch_block(hipStream_t st, const uint16_t* X, int M, int K, int h, const QuantSpec& qs, const lrq_tlq_weight& w, const float* bias,
                        int fp32, void* Y) {
    int l = 0;
    while ((1 << l) < h) ++l;
    switch (l) {
        case 6: return launch<BITS, 6>(st, X, M, K, l, qs, w, bias, fp32, Y);
        case 7: return launch<BITS, 7>(st, X, M, K, l, qs, w, bias, fp32, Y);
        case 8: return launch<BITS, 8>(st, X, M, K, l, qs, w, bias, fp32, Y);
        case 9: return launch<BITS, 9>(st, X, M, K, l, qs, w, bias, fp32, Y);
        case 10: return launch<BITS, 10>(st, X, M, K, l, qs, w, bias, fp32, Y);
        default: return launch<BITS, 5>(st, X, M, K, l, qs, w, bias, fp32, Y);
    }
}

}  // namespace

// Every workgroup repeats the rotation, so there must not be more of them than CUs.  us per call, one launch / two: 2 x 1152 -> 6912 5.6 / 8.8,
// 14 x 1152 -> 6912 6.0 / 8.7, 5 x 3072 -> 8192 7.2 / 9.2, 16 x 1024 -> 8192 6.4 / 9.1, 3 x 4608 -> 4608 7.8 / 9.9.  Past 256 workgroups, in device
// time (a graph of calls; called one by one the host's rate hides up to 2 us of it), -> 10240: 2 x 1152 with h = 32, 64, 128 7.3 / 6.2, 6.9 / 6.5,
// 8.4 / 6.6, 4 x 1024 with h = 256, 1024 8.4 / 7.2, 7.5 / 7.5, 8 x 2048 with h = 512 11.9 / 8.6, 5 x 3072 with h = 64, 1024 8.9 / 8.2, 12.6 / 9.3;
// -> 24576 all lose more.  Registers let two workgroups share a CU in 19 of the 24 forms (all but h = 128 and the symmetric h = 256),
// LDS does not for long exchanges; sharing one, two rotations take nearly twice as long.
bool qlinear_few_applies(int M, int N, int K, int had_block) {
    return M <= 16 && K % 128 == 0 && (long)M * K <= kFewElements && had_block <= 1024 && (N + 31) / 32 <= 256;
}

hipError_t launch_qlinear_few(hipStream_t st, const uint16_t* X, int M, int K, int had_block, int act_bits, bool asym, const float* prescale,
                              const lrq_tlq_weight& w, const float* bias, int out_dtype, void* Y) {
    QuantSpec qs = make_spec(act_bits, had_block, nullptr, prescale);
    qs.asym = asym;                                  // zero-points stay in LDS
    const int fp32 = out_dtype == LRQ_OUT_FP32;
    return w.bits == 4 ? launch_block<4>(st, X, M, K, had_block, qs, w, bias, fp32, Y) : launch_block<3>(st, X, M, K, had_block, qs, w, bias, fp32, Y);
}

}  // namespace lrq
