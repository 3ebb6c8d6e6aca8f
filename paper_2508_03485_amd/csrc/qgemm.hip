// Decode + int8 MFMA GEMM + rescale (gfx950):
//   Y[t,n] = scale_t * wscale_n * sum_k q[t,k] * lut_n[code[n,k]]  (+ bias_n)
// Activation codes q (int8, [M,K]) are staged through LDS (three rotating buffers) and shared by the four
// waves of a workgroup; every wave owns its own 64 output channels, streams the packed 3/4-bit TLQ codes of
// those channels straight from global memory into registers and decodes them there with per-lane
// level tables (byte permutes), so decoded weights never touch LDS.  v_mfma_i32_16x16x64_i8 does the
// contraction with int32 accumulation ("SpeedUp and Latency": INT8 x INT8, higher-precision accumulate): one
// instruction per 16 x 16 output tile and K block of 64.  (On pseudo-random operands the chip sustains 3.9 POP/s with
// this instruction and 3.3 POP/s with v_mfma_i32_32x32x32_i8: the matrix pipe is power-limited and this shape draws
// less per operation.)
// The epilogue rescales in fp32 and goes through LDS so that every lane stores 16 contiguous bytes.
#include "qgemm_common.h"

namespace lrq {
namespace {

constexpr int WAVES = 4;
constexpr int BK = kGemmBlockK;     // 64
constexpr int PLANE_PAD = 32;          // padding of a plane (swept 0 / 16 / 32 / 48: 32 leaves the fewest bank conflicts)
constexpr int AF_DIST = 2;             // A fragments are read this many row tiles (one pair) ahead of their use
constexpr int PLANE = 32 * 16 + PLANE_PAD;     // bytes of one (row tile, 16-byte k chunk) plane in LDS, padded
constexpr int EPI_ROW = 64 * 2 + 16;   // bytes of one staged output row of a wave (up to 64 bf16 / 32 fp32) + pad
constexpr int EPI_WAVE = 32 * EPI_ROW; // one 32-row slab per wave

// One K block of the main loop.  The A tiles rotate through three LDS buffers: block kb multiplies from `cur`
// (tile kb), stages tile kb+2 (held in aS, which is then reloaded with tile kb+4) into `st`, and - because tile kb+1
// in `nx` has been complete since the previous barrier - reads the first A fragments of block kb+1 before its own
// closing barrier, so that the next block starts on the matrix cores without waiting for LDS.
// bdCur holds the decoded B operands of block kb (one per 16-column tile); bRaw holds the raw codes of block kb+1, which
// are decoded into bdNxt between the matrix instructions of this block (so that the decode issues in their shadow) and
// then reloaded with block kb+3 (the other raw set, block kb+2, is in flight meanwhile).
// Packed 4-bit activation codes (A4P): a 16-byte chunk holds 32 codes, eight per dword, byte j of a dword = code[j] + 8 in
// the low nibble and code[4 + j] + 8 in the high nibble.  It is widened on its way into LDS to two 16-byte chunks of
// bytes in [1, 15]; the constant offset 8 leaves through the epilogue as a zero-point of -8 (times the channel's level sum).
template <bool A4P>
__device__ __forceinline__ void stage_a(unsigned char* dst, v4i a) {
    if constexpr (!A4P) {
        *reinterpret_cast<v4i*>(dst) = a;
    } else {
        v4i lo, hi;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const unsigned w = (unsigned)a[d];
            const unsigned l = w & 0x0f0f0f0fu, h = (w >> 4) & 0x0f0f0f0fu;
            if (d < 2) { lo[2 * d] = (int)l; lo[2 * d + 1] = (int)h; }
            else { hi[2 * (d - 2)] = (int)l; hi[2 * (d - 2) + 1] = (int)h; }
        }
        *reinterpret_cast<v4i*>(dst) = lo;
        *reinterpret_cast<v4i*>(dst + PLANE) = hi;
    }
}

template <int BITS, int RT, int NTW, int ALOADS, bool A4P>
__device__ __forceinline__ void kblock(unsigned char* smem, int cur, int st, int nx, v4i (&aS)[ALOADS],
                                       BRaw<BITS> (&bRaw)[NTW], int kb, int KB,
                                       const int8_t* const (&aptr)[ALOADS], const int (&aoff)[ALOADS],
                                       const uint8_t* const (&bptr)[NTW], const unsigned (&L)[2 * NTW][4], unsigned C,
                                       const v4i (&bdCur)[2 * NTW], v4i (&bdNxt)[2 * NTW], v4i (&acc)[RT][2 * NTW], int rd_off,
                                       v4i (&afp)[AF_DIST]) {
    constexpr int UNIT = 64 * 16;
    constexpr int CT = 2 * NTW;                     // 16-column tiles of a wave
    constexpr int ABK = A4P ? BK / 2 : BK;          // bytes of a token row per K block
    const unsigned char* Acur = smem + cur;
#pragma unroll
    for (int i = 0; i < ALOADS; ++i) stage_a<A4P>(&smem[st + aoff[i]], aS[i]);
    const int ka = kb + 4 < KB ? kb + 4 : KB - 1;
    const int kbn = kb + 3 < KB ? kb + 3 : KB - 1;
#pragma unroll
    for (int i = 0; i < ALOADS; ++i) aS[i] = *reinterpret_cast<const v4i*>(aptr[i] + (size_t)ka * ABK);
    v4i af[RT];
    constexpr int DPB = (CT * 4 + RT - 1) / RT;     // operand dwords decoded per row tile
    constexpr int DIST = AF_DIST;                   // A fragments are read this many row tiles ahead
#pragma unroll
    for (int p = 0; p < DIST; ++p) af[p] = afp[p];
    // Order of the matrix instructions (operand changes cost power, decode needs issue slots between them).  4-bit codes: two row
    // tiles at a time, one operand changing per instruction; 3-bit codes, whose decode is a third shorter: one row tile at a time,
    // back and forth over the column tiles, except in 64-row tiles.  One order for all costs some of them (us, row by row / pairs:
    // 35100 x 12288 -> 3072 at 4 bits 1235 / 1228, at 3 bits 1035 / 1070; 2502 x 12288 -> 1152, one tile per CU, 64.3 / 61.3 and
    // 50.2 / 56.2; 64-row tiles at 3 bits, 2500 x 12288 -> 896, 48.4 / 46.5).
    constexpr int WALK = BITS == 4 || RT == 4 ? 2 : 1;
    static_assert(AF_DIST == 2 && RT % 2 == 0, "the first pair of the next block is read at row tile RT - 2");
#pragma unroll
    for (int p = 0; p < RT; p += WALK) {
        if (p == RT - 2) {          // next block's first fragments, early enough to land before the closing barrier
#pragma unroll
            for (int pp = 0; pp < DIST; ++pp)
                afp[pp] = *reinterpret_cast<const v4i*>(&smem[nx + (pp / 2) * 4 * PLANE + (pp % 2) * 256 + rd_off]);
        }
#pragma unroll
        for (int pp = p + DIST; pp < p + DIST + WALK; ++pp)
            if (pp < RT) af[pp] = *reinterpret_cast<const v4i*>(&Acur[(pp / 2) * 4 * PLANE + (pp % 2) * 256 + rd_off]);
#pragma unroll
        for (int d = 0; d < WALK * DPB; ++d) {
            const int dd = p * DPB + d, ct = dd / 4;
            if (dd < CT * 4) bdNxt[ct][dd % 4] = (int)decode_dword<BITS>(bRaw[ct / 2], L[ct], ct % 2, dd % 4, C);
        }
#pragma unroll
        for (int c = 0; c < WALK * CT; ++c) {
            const int ct = WALK == 2 ? c / 2 : (p % 2 ? CT - 1 - c : c);
            const int i = WALK == 2 ? p + ((c + 1) / 2) % 2 : p;
            acc[i][ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bdCur[ct], af[i], acc[i][ct], 0, 0, 0);
        }
        if (p + WALK == RT) {
#pragma unroll
            for (int j = 0; j < NTW; ++j) bRaw[j] = load_braw<BITS>(bptr[j] + (size_t)kbn * UNIT);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
}

// BM rows x (4 waves x NTW x 32) columns per workgroup; RT = BM / 16 row tiles and 2 NTW column tiles of 16 per wave.  Shapes in use
// (launch_qgemm picks): 128 x 256 (NTW = 2, 128 accumulator registers per lane, two workgroups per CU), 160 x 128, 128 x 128
// (NTW = 1, 64 accumulator registers, three per CU) and 64 x 128 (256-row shapes - half the decode work per MFMA - measured
// no faster, or slower, on every workload).  ZP: zero-point form (epilogue term).
template <int BITS, int BM, int NTW, bool ZP, bool A4P = false, bool ZP64 = false>
__global__ __launch_bounds__(256, BM * NTW <= 128 ? 3 : (BM * NTW <= 256 ? 2 : 1)) void qgemm_kernel(
    const int8_t* __restrict__ q, const float* __restrict__ scale, int M, int K, int N,
    const uint8_t* __restrict__ gcodes, const int8_t* __restrict__ lut, const float* __restrict__ wscale,
    const float* __restrict__ bias, int out_fp32, void* __restrict__ Y, int tiles_m, int tiles_n,
    const int32_t* __restrict__ zero, const int32_t* __restrict__ colsum, int const_zero) {
    static_assert(!A4P || ZP, "the packed form needs the zero-point term of the epilogue");
    constexpr int RT = BM / 16, CT = 2 * NTW;
    constexpr int WN = 32 * NTW, BN = WAVES * WN;
    constexpr int ABUF = (BM / 32) * 4 * PLANE;
    constexpr int ACHUNKS = A4P ? BM * 2 : BM * 4;                 // 16-byte chunks of the A tile in global memory
    constexpr int ALOADS = (ACHUNKS + 255) / 256;                  // per thread (not a multiple of the threads: some are fetched twice)
    constexpr int ABK = A4P ? BK / 2 : BK;
    constexpr int LDS_BYTES = (3 * ABUF > WAVES * EPI_WAVE) ? 3 * ABUF : WAVES * EPI_WAVE;
    __shared__ __attribute__((aligned(16))) unsigned char smem[LDS_BYTES];
    __shared__ __attribute__((aligned(16))) float sc[BM];
    __shared__ __attribute__((aligned(16))) int zr[ZP ? BM : 4];      // per-token zero-points (zero-point form only)
    __shared__ __attribute__((aligned(16))) float wsc[BN], bs[BN];    // scale and bias of the tile's channels
    __shared__ __attribute__((aligned(16))) int csum[ZP ? BN : 4];    // their level sums (zero-point form only)

    // XCD-aware tile order.  Consecutive workgroup ids go round-robin over the 8 XCDs (each with its own L2), so
    // XCD x is handed a contiguous range of a linear tile order; that order walks 8-row-tile groups n-fastest
    // within 8 consecutive m (grouped ordering), so the ~64 tiles resident on an XCD at any time form an
    // 8 x 8 patch that shares each row panel of q and each channel panel of W eight ways through that L2.
    const int ntiles = tiles_m * tiles_n;
    int tile;
    {
        const int x = blockIdx.x % 8, i = blockIdx.x / 8;
        const int base = ntiles / 8, rem = ntiles % 8;           // XCD x owns base + (x < rem) tiles
        tile = x * base + (x < rem ? x : rem) + i;
    }
    int tm, tn;
    {
        constexpr int GM = 8;
        const int per_group = GM * tiles_n;
        const int group = tile / per_group, first_m = group * GM;
        const int gsize = tiles_m - first_m < GM ? tiles_m - first_m : GM;
        const int r = tile % per_group;
        tm = first_m + r % gsize;
        tn = r / gsize;
    }
    const int m0 = tm * BM, n0 = tn * BN;

    const int t = threadIdx.x, lane = t % 64, wv = t / 64;
    const int KB = K / BK;
    const int ntile32 = (N + 31) / 32;
    constexpr int UNIT = 64 * 16;

    // level tables of the lane's channel (lane % 16) in each of the wave's 16-column tiles, and the lane's slot of every
    // 32-channel tile
    unsigned L[CT][4];
    const uint8_t* bptr[NTW];
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
        int tl = (n0 + wv * WN) / 32 + j;
        if (tl >= ntile32) tl = ntile32 - 1;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int n = tl * 32 + h * 16 + lane % 16;
            if (n >= N) n = N - 1;
            const uint4 lv = *reinterpret_cast<const uint4*>(lut + (size_t)n * 16);
            L[2 * j + h][0] = lv.x; L[2 * j + h][1] = lv.y; L[2 * j + h][2] = lv.z; L[2 * j + h][3] = lv.w;
        }
        bptr[j] = gcodes + (size_t)tl * KB * UNIT + (size_t)lane * (UNIT / 64);
    }

    // A tile loader: BM*4 chunks of 16 bytes; chunk id -> (row, 16-byte column)
    const int8_t* aptr[ALOADS];
    int aoff[ALOADS];
#pragma unroll
    for (int i = 0; i < ALOADS; ++i) {
        const int cid = (t + 256 * i) % ACHUNKS;
        const int row = A4P ? cid / 2 : cid / 4, c = A4P ? 2 * (cid % 2) : cid % 4;      // c: first 16-byte chunk in LDS
        int gr = m0 + row;
        if (gr >= M) gr = M - 1;
        aptr[i] = A4P ? q + (size_t)gr * (K / 2) + (c / 2) * 16 : q + (size_t)gr * K + c * 16;
        aoff[i] = ((row / 32) * 4 + c) * PLANE + (row % 32) * 16;
    }
    if (t < BM) {
        const int r = m0 + t;
        sc[t] = r < M ? scale[r] : 0.0f;
        if constexpr (ZP) zr[t] = r < M ? (zero ? zero[r] : const_zero) : 0;
    }
    if (t < BN) {
        const int n = n0 + t < N ? n0 + t : N - 1;
        wsc[t] = wscale[n];
        bs[t] = bias ? bias[n] : 0.0f;
        if constexpr (ZP) csum[t] = colsum[n];
    }

    v4i acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;

    // ---- prologue: A tiles 0, 1 -> LDS buffers 0, 1; A tiles 2 (aO), 3 (aE) in registers; B block 0 decoded (bdA), raw
    // codes of blocks 1 (bO) and 2 (bE) in registers
    unsigned C = 0x03020100u;
    asm volatile("" : "+v"(C));
    v4i aO[ALOADS], aE[ALOADS];
    BRaw<BITS> bE[NTW], bO[NTW];
    v4i bdA[CT], bdB[CT];
    {
        v4i a0[ALOADS], a1[ALOADS];
        BRaw<BITS> b0[NTW];
        const int k1 = KB > 1 ? 1 : 0, k2 = KB > 2 ? 2 : KB - 1, k3 = KB > 3 ? 3 : KB - 1;
#pragma unroll
        for (int j = 0; j < NTW; ++j) b0[j] = load_braw<BITS>(bptr[j]);
#pragma unroll
        for (int i = 0; i < ALOADS; ++i) {
            a0[i] = *reinterpret_cast<const v4i*>(aptr[i]);
            a1[i] = *reinterpret_cast<const v4i*>(aptr[i] + (size_t)k1 * ABK);
        }
        // same issue order as the steady state of the K loop (A set, B block, A set, B block), so that the wait
        // counters the compiler derives at the loop head are the loop's own and not a conservative merge
#pragma unroll
        for (int i = 0; i < ALOADS; ++i) aO[i] = *reinterpret_cast<const v4i*>(aptr[i] + (size_t)k2 * ABK);
#pragma unroll
        for (int j = 0; j < NTW; ++j) bO[j] = load_braw<BITS>(bptr[j] + (size_t)k1 * UNIT);
#pragma unroll
        for (int i = 0; i < ALOADS; ++i) aE[i] = *reinterpret_cast<const v4i*>(aptr[i] + (size_t)k3 * ABK);
#pragma unroll
        for (int j = 0; j < NTW; ++j) bE[j] = load_braw<BITS>(bptr[j] + (size_t)k2 * UNIT);
#pragma unroll
        for (int i = 0; i < ALOADS; ++i) {
            stage_a<A4P>(&smem[aoff[i]], a0[i]);
            stage_a<A4P>(&smem[ABUF + aoff[i]], a1[i]);
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int g = 0; g < 4; ++g) bdA[ct][g] = (int)decode_dword<BITS>(b0[ct / 2], L[ct], ct % 2, g, C);
    }
    __syncthreads();

    // fragment of row tile i (16 rows) of a buffer: + (i / 2) * 4 * PLANE + (i % 2) * 256; the lane's row lane % 16 and
    // its 16-byte k chunk lane / 16
    const int rd_off = (lane / 16) * PLANE + (lane % 16) * 16;
    v4i afp[AF_DIST];
#pragma unroll
    for (int p = 0; p < AF_DIST; ++p)
        afp[p] = *reinterpret_cast<const v4i*>(&smem[(p / 2) * 4 * PLANE + (p % 2) * 256 + rd_off]);

    int o0 = 0, o1 = ABUF, o2 = 2 * ABUF;       // LDS buffers of tiles kb, kb+1, kb+2
    int kb = 0;
    // two K blocks per trip with no branch in between: with a conditional second block the compiler has to assume the
    // shorter path at the loop head and drains the whole load queue there (s_waitcnt vmcnt(0)) on every trip
    for (; kb + 1 < KB; kb += 2) {
        kblock<BITS, RT, NTW, ALOADS, A4P>(smem, o0, o2, o1, aO, bO, kb, KB, aptr, aoff, bptr, L, C, bdA, bdB, acc, rd_off, afp);
        kblock<BITS, RT, NTW, ALOADS, A4P>(smem, o1, o0, o2, aE, bE, kb + 1, KB, aptr, aoff, bptr, L, C, bdB, bdA, acc, rd_off, afp);
        const int t0 = o0;      // two blocks done: tiles kb+2, kb+3, kb+4 live in o2, o0, o1
        o0 = o2;
        o2 = o1;
        o1 = t0;
    }
    if (kb < KB)                // odd number of K blocks
        kblock<BITS, RT, NTW, ALOADS, A4P>(smem, o0, o2, o1, aO, bO, kb, KB, aptr, aoff, bptr, L, C, bdA, bdB, acc, rd_off, afp);

    // ---- epilogue: rescale in fp32.  The weights are the first operand of the matrix instructions, so a lane holds token
    // lane % 16 and the four neighbouring channels 4 (lane / 16) + (0..3) of every 16 x 16 accumulator tile: they go to
    // LDS in one 8-byte (bf16) or 16-byte (fp32) store.
    // y of accumulator tile (i, ct); the zero-point form adds zero_t * colsum_n to the integer sum
    const int lc = 4 * (lane / 16);
    float wq[CT][4], bq[CT][4];
    double cq[CT][4];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const float4 w4 = *reinterpret_cast<const float4*>(&wsc[wv * WN + ct * 16 + lc]);
        const float4 b4 = *reinterpret_cast<const float4*>(&bs[wv * WN + ct * 16 + lc]);
        wq[ct][0] = w4.x; wq[ct][1] = w4.y; wq[ct][2] = w4.z; wq[ct][3] = w4.w;
        bq[ct][0] = b4.x; bq[ct][1] = b4.y; bq[ct][2] = b4.z; bq[ct][3] = b4.w;
        if constexpr (ZP) {
            const int4 c4 = *reinterpret_cast<const int4*>(&csum[wv * WN + ct * 16 + lc]);
            cq[ct][0] = c4.x; cq[ct][1] = c4.y; cq[ct][2] = c4.z; cq[ct][3] = c4.w;
        }
    }
    auto rescale4 = [&](int i, int ct, float (&y)[4]) {
        const float sv = sc[i * 16 + lane % 16];
        const double zv = ZP ? (double)zr[i * 16 + lane % 16] : 0.0;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int a = acc[i][ct][x];
            const float tot = ZP64 ? zp_sum64(a, zv, cq[ct][x]) : (ZP ? zp_sum(a, zv, cq[ct][x]) : (float)a);
            y[x] = (tot * sv) * wq[ct][x] + bq[ct][x];
        }
    };
    const int ncol0 = n0 + wv * WN;                 // first column of this wave
    unsigned char* slab = smem + wv * EPI_WAVE;
    if (!out_fp32) {
        // bf16: one 32-row slab (two row tiles) per wave staged in LDS (wave-private, so only wave-level ordering is needed
        // after the K loop's final barrier); every lane then stores 16 contiguous bytes, a row segment of the wave is
        // WN * 2 bytes
        uint16_t* Yh = reinterpret_cast<uint16_t*>(Y);
        const bool vec = N % 8 == 0;                // rows of Y are 16-byte aligned
#pragma unroll
        for (int i2 = 0; i2 < RT / 2; ++i2) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    float y[4];
                    rescale4(2 * i2 + h, ct, y);
                    *reinterpret_cast<uint2*>(&slab[(16 * h + lane % 16) * EPI_ROW + (ct * 16 + lc) * 2]) =
                        make_uint2(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]));
                }
            wave_sync();
            if (vec) {
                // 32 rows x (WN * 2) bytes: WN / 8 lanes per row, 16 bytes per lane
                constexpr int LPR = WN / 8, RPP = 64 / LPR;
#pragma unroll
                for (int p = 0; p < 32 / RPP; ++p) {
                    const int lr = p * RPP + lane / LPR, cb = (lane % LPR) * 8;   // 8 bf16 per lane
                    const uint4 v = *reinterpret_cast<const uint4*>(&slab[lr * EPI_ROW + cb * 2]);
                    const int row = m0 + i2 * 32 + lr, col = ncol0 + cb;
                    if (row < M && col < N) *reinterpret_cast<uint4*>(&Yh[(size_t)row * N + col]) = v;
                }
            } else {
                // rows of any alignment: neighbouring lanes store neighbouring elements
                const int cl = lane % WN, col = ncol0 + cl;
#pragma unroll 8
                for (int p = 0; p < WN / 2; ++p) {
                    const int lr = p * (64 / WN) + lane / WN, row = m0 + i2 * 32 + lr;
                    if (row < M && col < N) Yh[(size_t)row * N + col] = *reinterpret_cast<const uint16_t*>(&slab[lr * EPI_ROW + cl * 2]);
                }
            }
            wave_sync();
        }
    } else {
        // fp32: the same staging, 32 rows x 32 columns at a time
        float* Yf = reinterpret_cast<float*>(Y);
        const bool vec = N % 4 == 0;
#pragma unroll
        for (int i2 = 0; i2 < RT / 2; ++i2)
#pragma unroll
            for (int j = 0; j < NTW; ++j) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        float y[4];
                        rescale4(2 * i2 + h, 2 * j + c, y);
                        *reinterpret_cast<float4*>(&slab[(16 * h + lane % 16) * EPI_ROW + (c * 16 + lc) * 4]) =
                            make_float4(y[0], y[1], y[2], y[3]);
                    }
                wave_sync();
                if (vec) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int lr = p * 8 + lane / 8, cb = (lane % 8) * 4;    // 4 floats per lane
                        const uint4 v = *reinterpret_cast<const uint4*>(&slab[lr * EPI_ROW + cb * 4]);
                        const int row = m0 + i2 * 32 + lr, col = ncol0 + j * 32 + cb;
                        if (row < M && col < N) *reinterpret_cast<uint4*>(&Yf[(size_t)row * N + col]) = v;
                    }
                } else {
                    const int cl = lane % 32, col = ncol0 + j * 32 + cl;
#pragma unroll 8
                    for (int p = 0; p < 16; ++p) {
                        const int lr = p * 2 + lane / 32, row = m0 + i2 * 32 + lr;
                        if (row < M && col < N) Yf[(size_t)row * N + col] = *reinterpret_cast<const float*>(&slab[lr * EPI_ROW + cl * 4]);
                    }
                }
                wave_sync();
            }
    }
}

// Small inputs.  A 128-row tile makes so few workgroups of them that most of the chip idles while each walks all of K in
// sequence (256 x 1152 -> 1152: 18 workgroups on 256 CUs).  Here a workgroup owns 16 RT rows x 32 channels and its SW waves split
// K between them (wave w takes the K blocks w, w + SW, ...): no LDS and no barrier in the loop, both operands come straight
// from L2 as matrix operands, the loads of UB blocks in flight at a time.  The partial sums are integers, so their order does
// not matter; they meet in LDS once at the end.
constexpr int SW = 8;
template <int BITS, int RT, bool ZP, bool A4P>
__global__ __launch_bounds__(64 * SW) void qgemm_small_kernel(
    const int8_t* __restrict__ q, const float* __restrict__ scale, int M, int K, int N,
    const uint8_t* __restrict__ gcodes, const int8_t* __restrict__ lut, const float* __restrict__ wscale,
    const float* __restrict__ bias, int out_fp32, void* __restrict__ Y, int tiles_n,
    const int32_t* __restrict__ zero, const int32_t* __restrict__ colsum, int const_zero) {
    static_assert(!A4P || ZP, "the packed form needs the zero-point term of the epilogue");
    constexpr int UNIT = 64 * 16, UB = RT <= 2 ? 3 : 2;
    __shared__ __attribute__((aligned(16))) v4i part[SW][2 * RT][64];
    const int t = threadIdx.x, lane = t % 64, wv = t / 64;
    const int tn = blockIdx.x % tiles_n, m0 = (blockIdx.x / tiles_n) * (16 * RT);
    const int KB = K / BK;
    unsigned L[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        int n = tn * 32 + h * 16 + lane % 16;
        if (n >= N) n = N - 1;
        const uint4 lv = *reinterpret_cast<const uint4*>(lut + (size_t)n * 16);
        L[h][0] = lv.x; L[h][1] = lv.y; L[h][2] = lv.z; L[h][3] = lv.w;
    }
    const uint8_t* bptr = gcodes + (size_t)tn * KB * UNIT + (size_t)lane * (UNIT / 64);
    const int8_t* aptr[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        int r = m0 + i * 16 + lane % 16;
        if (r >= M) r = M - 1;
        aptr[i] = A4P ? q + (size_t)r * (K / 2) + (lane / 16) * 8 : q + (size_t)r * K + (lane / 16) * 16;
    }
    unsigned C = 0x03020100u;
    asm volatile("" : "+v"(C));
    v4i acc[RT][2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[i][h] = v4i{0, 0, 0, 0};
    for (int kb0 = wv; kb0 < KB; kb0 += SW * UB) {
        BRaw<BITS> b[UB];
        v4i a[UB][RT];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int kb = kb0 + u * SW < KB ? kb0 + u * SW : kb0;         // past the end: loaded again, not used
            b[u] = load_braw<BITS>(bptr + (size_t)kb * UNIT);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                if constexpr (A4P) {
                    const uint2 w = *reinterpret_cast<const uint2*>(aptr[i] + (size_t)kb * (BK / 2));
                    a[u][i] = v4i{(int)(w.x & 0x0f0f0f0fu), (int)((w.x >> 4) & 0x0f0f0f0fu), (int)(w.y & 0x0f0f0f0fu),
                                  (int)((w.y >> 4) & 0x0f0f0f0fu)};
                } else {
                    a[u][i] = *reinterpret_cast<const v4i*>(aptr[i] + (size_t)kb * BK);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            if (kb0 + u * SW < KB) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v4i bd;
#pragma unroll
                    for (int g = 0; g < 4; ++g) bd[g] = (int)decode_dword<BITS>(b[u], L[h], h, g, C);
#pragma unroll
                    for (int i = 0; i < RT; ++i)
                        acc[i][h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bd, a[u][i], acc[i][h], 0, 0, 0);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) part[wv][2 * i + h][lane] = acc[i][h];
    __syncthreads();
    // one thread per (accumulator tile, lane): token lane % 16, four neighbouring channels
    const bool vec = N % 4 == 0;
    for (int o = t; o < 2 * RT * 64; o += 64 * SW) {
        const int tile = o / 64, l = o % 64;
        const int row = m0 + (tile / 2) * 16 + l % 16, n = tn * 32 + (tile % 2) * 16 + 4 * (l / 16);
        if (row >= M || n >= N) continue;
        v4i s = part[0][tile][l];
#pragma unroll
        for (int w = 1; w < SW; ++w) s += part[w][tile][l];
        const float sv = scale[row];
        const double zv = ZP ? (double)(zero ? zero[row] : const_zero) : 0.0;
        float y[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int nx = n + x < N ? n + x : N - 1;
            const float tot = ZP ? zp_sum(s[x], zv, (double)colsum[nx]) : (float)s[x];
            y[x] = (tot * sv) * wscale[nx] + (bias ? bias[nx] : 0.0f);
        }
        if (!out_fp32) {
            uint16_t* dst = reinterpret_cast<uint16_t*>(Y) + (size_t)row * N + n;
            const unsigned d[2] = {pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
            if (vec) {
                *reinterpret_cast<uint2*>(dst) = make_uint2(d[0], d[1]);
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (n + x < N) dst[x] = (uint16_t)(d[x / 2] >> (16 * (x % 2)));
            }
        } else {
            float* dst = reinterpret_cast<float*>(Y) + (size_t)row * N + n;
            if (vec) {
                *reinterpret_cast<float4*>(dst) = make_float4(y[0], y[1], y[2], y[3]);
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (n + x < N) dst[x] = y[x];
            }
        }
    }
}

template <int BITS, int RT>
hipError_t launch_small(hipStream_t st, const int8_t* q, const float* scale, const int32_t* zero, int M, int K,
                        const lrq_tlq_weight& w, const float* bias, int fp32, void* Y, bool packed4) {
    const int tiles_n = (w.N + 31) / 32;
    const dim3 grid(((M + 16 * RT - 1) / (16 * RT)) * tiles_n), block(64 * SW);
    const int32_t* none = nullptr;
    if (packed4)
        hipLaunchKernelGGL((qgemm_small_kernel<BITS, RT, true, true>), grid, block, 0, st, q, scale, M, K, w.N, w.gemm_codes, w.lut,
                           w.wscale, bias, fp32, Y, tiles_n, none, w.colsum, -8);
    else if (zero)
        hipLaunchKernelGGL((qgemm_small_kernel<BITS, RT, true, false>), grid, block, 0, st, q, scale, M, K, w.N, w.gemm_codes, w.lut,
                           w.wscale, bias, fp32, Y, tiles_n, zero, w.colsum, 0);
    else
        hipLaunchKernelGGL((qgemm_small_kernel<BITS, RT, false, false>), grid, block, 0, st, q, scale, M, K, w.N, w.gemm_codes, w.lut,
                           w.wscale, bias, fp32, Y, tiles_n, none, w.colsum, 0);
    return hipGetLastError();
}

template <int BITS, int BM, int NTW>
hipError_t launch(hipStream_t st, const int8_t* q, const float* scale, const int32_t* zero, int M, int K,
                  const lrq_tlq_weight& w, const float* bias, int fp32, void* Y, bool packed4) {
    constexpr int BN = WAVES * 32 * NTW;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (w.N + BN - 1) / BN;
    if (packed4)
        hipLaunchKernelGGL((qgemm_kernel<BITS, BM, NTW, true, true>), dim3(tiles_m * tiles_n), dim3(256), 0, st, q, scale, M, K, w.N,
                           w.gemm_codes, w.lut, w.wscale, bias, fp32, Y, tiles_m, tiles_n, static_cast<const int32_t*>(nullptr),
                           w.colsum, -8);
    else if (zero)
        hipLaunchKernelGGL((qgemm_kernel<BITS, BM, NTW, true>), dim3(tiles_m * tiles_n), dim3(256), 0, st, q, scale, M, K, w.N,
                           w.gemm_codes, w.lut, w.wscale, bias, fp32, Y, tiles_m, tiles_n, zero, w.colsum, 0);
    else
        hipLaunchKernelGGL((qgemm_kernel<BITS, BM, NTW, false>), dim3(tiles_m * tiles_n), dim3(256), 0, st, q, scale, M, K, w.N,
                           w.gemm_codes, w.lut, w.wscale, bias, fp32, Y, tiles_m, tiles_n, zero, w.colsum, 0);
    return hipGetLastError();
}

// the zero-point form of rows longer than kZpF64K
template <int BITS>
hipError_t launch_long(hipStream_t st, const int8_t* q, const float* scale, const int32_t* zero, int M, int K,
                       const lrq_tlq_weight& w, const float* bias, int fp32, void* Y) {
    const int tiles_m = (M + 127) / 128, tiles_n = (w.N + 127) / 128;
    hipLaunchKernelGGL((qgemm_kernel<BITS, 128, 1, true, false, true>), dim3(tiles_m * tiles_n), dim3(256), 0, st, q, scale, M, K, w.N,
                       w.gemm_codes, w.lut, w.wscale, bias, fp32, Y, tiles_m, tiles_n, zero, w.colsum, 0);
    return hipGetLastError();
}

// ---- dispatch: the kernel whose predicted time is the smallest -----------------------------------------------------
// Times in us, fitted to 5600 measurements over M = 1 .. 35100, N = 96 .. 12288 and K = 1152 .. 12288, all forms and both output
// types; the kernel chosen is within 0.7 % of the fastest on average and within 24 % at worst.
//
// Tiles.  A CU's tiles run one after the other or share it at the same total rate, so the time follows from the tiles of the
// fullest CU.  One tile: lone_k (packed codes: + lone_packed) per K block + lone; n > 1 tiles: n (k (+ packed) per K block +
// tile) + once.  Output rows that are not 16-byte aligned leave element by element: + lone_ragged, or + ragged per tile (4.7 us for
// a 128 x 256 tile on its own, 2 us where others run beside it).  The tall shapes decode less per matrix instruction, the small
// ones leave less of the chip idle in the last round: 8192 x 4608 -> 1152 takes 53 us with 160 rows (468 tiles) and 57 with 128 (576),
// 1000 x 3072 -> 3072 20 us with 128 x 128 and 29 with 128 x 256, 2333 x 1152 -> 1091 in fp32 10.1 us with 64 rows and 13.0 with 128,
// 35100 x 3072 -> 12001 in fp32 1442 us with 128 x 256 and 1563 with 128 x 128; 3-bit codes decode faster: 8192 x 1152 -> 3456 37 / 38 us.
struct TileCost { int rows, cols; float lone_k, lone_packed, lone, lone_ragged, k, packed, tile, ragged, once; };
constexpr TileCost kTileCost[2][4] = {
    {{128, 256, 0.354f, 0.054f, 5.62f, 4.73f, 0.353f, 0.000f, 3.54f, 2.40f, 1.00f},        // 3-bit codes
     {160, 128, 0.291f, 0.135f, 4.65f, 2.78f, 0.284f, 0.019f, 2.27f, 1.44f, 1.58f},
     {128, 128, 0.235f, 0.057f, 4.09f, 2.23f, 0.220f, 0.002f, 1.60f, 0.91f, 2.19f},
     { 64, 128, 0.174f, 0.069f, 3.26f, 1.03f, 0.126f, 0.021f, 0.72f, 0.39f, 2.63f}},
    {{128, 256, 0.477f, 0.057f, 5.70f, 4.73f, 0.434f, 0.001f, 3.86f, 2.06f, 0.47f},        // 4-bit codes
     {160, 128, 0.368f, 0.114f, 4.55f, 2.94f, 0.332f, 0.004f, 2.33f, 1.23f, 1.92f},
     {128, 128, 0.299f, 0.047f, 4.09f, 2.33f, 0.258f, 0.003f, 1.62f, 0.84f, 2.79f},
     { 64, 128, 0.232f, 0.074f, 3.28f, 1.15f, 0.167f, 0.022f, 0.64f, 0.32f, 3.73f}}};
// K split over the waves.  A round of workgroups, one per CU, reads the codes of a K block (w) and 16-row pieces of activations (a
// each, as many as there are rows for): once + rounds ((w + a pieces (+ packed)) per K block + round).  Its column tiles lie on
// different XCDs, each of which fetches the activations: + fetch per MB of them and column tile, up to eight.  Measured up to
// kSplitOutputs; far below it the split always wins, beyond it the operands are fetched too often (us, split / best tile: 16 x 3072 ->
// 12288 6.2 / 14.2, 256 x 3072 -> 3072 12.2 / 14.6, 1024 x 1152 -> 1152 10.1 / 7.7, 3907 x 6144 -> 256 31.0 / 26.0).  More rows to a workgroup
// pay once there are more workgroups than CUs (us with 16 / 32 / 64 rows, K = 1152 -> 1152: 64 rows 3.4 / 4.1 / 4.8, 256 rows 5.3 /
// 5.7 / 4.8).
struct SplitCost { int rows; float w, a, packed, round, once, fetch; };
constexpr SplitCost kSplitCost[2][3] = {
    {{16, 0.0164f, 0.0163f, 0.0009f, 0.37f, 2.17f, 0.0165f},         // 3-bit codes
     {32, 0.0206f, 0.0181f, 0.0039f, 0.54f, 2.16f, 0.0286f},
     {64, 0.0337f, 0.0189f, 0.0049f, 0.20f, 2.51f, 0.0389f}},
    {{16, 0.0288f, 0.0063f, 0.0008f, 0.44f, 2.14f, 0.0145f},         // 4-bit codes
     {32, 0.0316f, 0.0134f, 0.0048f, 0.51f, 2.22f, 0.0305f},
     {64, 0.0398f, 0.0173f, 0.0080f, 0.29f, 2.40f, 0.0386f}}};
constexpr long kSplitOutputs = 1600000;

}  // namespace

// cols == 32: the split-K kernel
GemmShape qgemm_shape(int M, int N, int K, int bits, bool zero_point, bool packed4, bool fp32) {
    if (zero_point && K > kZpF64K) return {128, 128, 0.0f};       // the only shape that kernel is built in
    const float kb = (float)(K / BK), packed = packed4 ? 1.0f : 0.0f;
    const float ragged = N % (fp32 ? 4 : 8) != 0 ? 1.0f : 0.0f;
    GemmShape best = {0, 0, INFINITY};
    auto consider = [&](int rows, int cols, float us) {
        if (us < best.us) best = {rows, cols, us};
    };
    for (const TileCost& c : kTileCost[bits - 3]) {
        const long n = (((long)M + c.rows - 1) / c.rows * (((long)N + c.cols - 1) / c.cols) + 255) / 256;
        consider(c.rows, c.cols, n == 1 ? (c.lone_k + c.lone_packed * packed) * kb + c.lone + c.lone_ragged * ragged
                                        : (float)n * ((c.k + c.packed * packed) * kb + c.tile + c.ragged * ragged) + c.once);
    }
    if ((long)M * N <= kSplitOutputs)
        for (const SplitCost& c : kSplitCost[bits - 3]) {
            const long tn = (N + 31) / 32, rounds = ((M + c.rows - 1) / c.rows * tn + 255) / 256;
            const float pieces = (float)(M < c.rows ? M : c.rows) / 16.0f;
            const float mb = (float)M * (float)K * (packed4 ? 0.5e-6f : 1e-6f) * (float)(tn < 8 ? tn : 8);
            consider(c.rows, 32, c.once + (float)rounds * ((c.w + c.a * pieces + c.packed * packed) * kb + c.round) + c.fetch * mb);
        }
    return best;
}

hipError_t launch_qgemm(hipStream_t st, const int8_t* q, const float* scale, const int32_t* zero, int M, int K,
                        const lrq_tlq_weight& w, const float* bias, int out_dtype, void* Y, bool packed4) {
    if (packed4 && zero) return hipErrorInvalidValue;
    const int fp32 = out_dtype == LRQ_OUT_FP32;
#define LRQ_SHAPE(F, ...) (w.bits == 4 ? F<4, __VA_ARGS__>(st, q, scale, zero, M, K, w, bias, fp32, Y, packed4)   \
                                       : F<3, __VA_ARGS__>(st, q, scale, zero, M, K, w, bias, fp32, Y, packed4))
    if (zero && K > kZpF64K) {
        if (w.bits == 4) return launch_long<4>(st, q, scale, zero, M, K, w, bias, fp32, Y);
        return launch_long<3>(st, q, scale, zero, M, K, w, bias, fp32, Y);
    }
    const GemmShape shape = qgemm_shape(M, w.N, K, w.bits, zero != nullptr, packed4, fp32);
    if (shape.cols == 32) {
        if (shape.rows == 16) return LRQ_SHAPE(launch_small, 1);
        if (shape.rows == 32) return LRQ_SHAPE(launch_small, 2);
        return LRQ_SHAPE(launch_small, 4);
    }
    if (shape.cols == 256) return LRQ_SHAPE(launch, 128, 2);
    if (shape.rows == 160) return LRQ_SHAPE(launch, 160, 1);
    if (shape.rows == 128) return LRQ_SHAPE(launch, 128, 1);
    return LRQ_SHAPE(launch, 64, 1);
#undef LRQ_SHAPE
}

}  // namespace lrq
