// int8 GEMM of large products, 4-bit weights: weights decoded once per call, tiles of up to 256 x 256 (gfx950).
//
// In qgemm.hip every tile decodes the codes of its channels again, M / 128 times over: that is, at 4 bits, 110 vector instructions beside
// 32 matrix instructions per wave and K block, more than the issue port takes in the matrix pipe's time.  Here a first
// kernel writes the int8 levels of all weights to the workspace, in the order in which the matrix instructions read
// them (35100 x 3072 -> 12288: 9 us), and the GEMM itself has next to no vector work in its loop: 1290 -> 1095 us there, with the same sums.
//
// GEMM: one workgroup of eight waves per CU, 256 x 256 outputs, a wave 128 x 64 (128 accumulator registers), K stages of 64.  Both
// operands go from global memory straight into LDS (global_load_lds, 16 bytes a lane) through four buffers of 32 KB, three stages
// ahead; a stage's fragments are read up to a stage before their matrix instructions.  The workgroups are persistent: the loads of a
// tile's last three stages already fetch the next tile, so that the pipeline does not drain between tiles.
// Timing-only builds say what the loop waits for (35100 x 3072 -> 12288): 1095 us as it is, 957 without its stores, 934 with operands that
// always hit L2 on top of that, 773 with no operand loads at all; two 128 x 256 workgroups per CU instead of this one take 1119, since they
// fetch twice as much through the fabric (3.7 against 2.3 GB).
#include "qgemm_common.h"
#include "weight_decode.h"

namespace lrq {
namespace {

constexpr int BK = kGemmBlockK;                      // 64
constexpr int BN = 256;
constexpr int BUF = 256 * BK;                        // bytes of one operand tile of a stage (256 rows at most)
constexpr int NBUF = 4;
constexpr int OFF_B = NBUF * BUF, OFF_S = 2 * NBUF * BUF;
constexpr int GROUP = kWideGroup;
// token scales, channel scales, biases; zero-point form: zero-points and level sums
constexpr int LDS_BYTES = OFF_S + (3 * 256 + 2 * 256) * 4;

// The decoding pass on its own, for rotations whose launch does not take it.  Bound by its writes: 37.7 MB in 9 us.
__global__ __launch_bounds__(256) void decode_weights_kernel(DecodeJob job) { decode_weights(job, blockIdx.x, gridDim.x, 4); }

// 64 lanes x 16 bytes from global memory into LDS: lane l's bytes land at lds + 16 l.  In assembly, with no register written, because
// the compiler would wait for every load of this kind before any later LDS read; the waits are the WAIT_LOADS below.
__device__ __forceinline__ void load_to_lds(unsigned lds, unsigned voff, const void* base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
// all but the wave's latest n vector-memory operations have finished
#define LRQ_WAIT_LOADS(n) asm volatile("s_waitcnt vmcnt(" #n ")" ::: "memory")

// Workgroup barrier without waits of its own (the callers wait for exactly what has to be visible).
__device__ __forceinline__ void raw_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// One K stage (index s of the tile) of a wave.  bc / ac: its fragments (columns, rows); rows 0-3 and all columns were read during the
// stage before, which is why the operands of stage s + 1 have to be complete when stage s begins.  Loads for stage s + 3 go to the buffer
// that stage s - 1 has left, one instruction per block of eight matrix instructions so that the eight waves do not queue up for them.
struct Source {                     // of the loads of one stage: A rows (two 16-row pieces), B pieces
    const int8_t* a;
    const uint8_t* b;
    unsigned va0, va1;
    int piece0, piece1;             // where in the stage's A tile the rows go
};
__device__ __forceinline__ void load_stage_piece(unsigned lds0, int buf, int wv, unsigned lvoff, const Source& x, int piece) {
    const unsigned dst = lds0 + buf * BUF;
    if (piece == 0) load_to_lds(dst + x.piece0 * 1024, x.va0, x.a);
    if (piece == 1) load_to_lds(dst + x.piece1 * 1024, x.va1, x.a);
    if (piece == 2) load_to_lds(dst + OFF_B + wv * 2048, lvoff, x.b);
    if (piece == 3) load_to_lds(dst + OFF_B + wv * 2048 + 1024, lvoff, x.b + 1024);
}
template <int RT>
__device__ __forceinline__ void stage(const unsigned char* smem, unsigned lds0, int buf, int wv, unsigned lvoff, const Source& x,
                                      int a_rd, int b_rd, const v4i (&bc)[4], v4i (&bn)[4], v4i (&ac)[RT], v4i (&an)[RT],
                                      v4i (&acc)[RT][4]) {
    constexpr int NP = (RT + 1) / 2;                 // blocks: row tiles in pairs, the last one alone where RT is odd
    static_assert(NP == 3 || NP == 4, "the fragments and loads are dealt to three or four blocks");
    const unsigned char* cur = smem + buf * BUF;
    const unsigned char* nxt = smem + ((buf + 1) % NBUF) * BUF;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (p < 2) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (2 * p + 4 + e < RT) ac[2 * p + 4 + e] = *reinterpret_cast<const v4i*>(cur + a_rd + (2 * p + 4 + e) * 1024);
                bn[2 * p + e] = *reinterpret_cast<const v4i*>(nxt + b_rd + (2 * p + e) * 1024);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)                  // rows 0-3 of the next stage, during the last two blocks
            if (p == NP - 2 + e / 2) an[e] = *reinterpret_cast<const v4i*>(nxt + a_rd + e * 1024);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int CT = 4;
        const int rows = 2 * p + 1 < RT ? 2 : 1;
#pragma unroll
        for (int c = 0; c < rows * CT; ++c) {
            const int ct = c / rows, i = 2 * p + (rows == 2 ? ((c + 1) / 2) % 2 : 0);        // one operand changes per instruction
            acc[i][ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bc[ct], ac[i], acc[i][ct], 0, 0, 0);
            if (c == 1) {
                __builtin_amdgcn_sched_barrier(0);
                load_stage_piece(lds0, (buf + 3) % NBUF, wv, lvoff, x, p);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (NP == 3 && p == 1 && c == 5) {
                __builtin_amdgcn_sched_barrier(0);
                load_stage_piece(lds0, (buf + 3) % NBUF, wv, lvoff, x, 3);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // the loads of the stage before this one, i.e. the operands of stage s + 2, have arrived; so have all fragments of stage s
    LRQ_WAIT_LOADS(4);
    raw_barrier();
}

// 32 RT rows x 256 columns per workgroup
template <int RT, bool ZP>
__global__ __launch_bounds__(512, 2) void qgemm_wide_kernel(
    const int8_t* __restrict__ q, const float* __restrict__ scale, int M, int K, int N, const uint8_t* __restrict__ wdec,
    const float* __restrict__ wscale, const float* __restrict__ bias, uint16_t* __restrict__ Y, int tiles_m, int tiles_n,
    const int32_t* __restrict__ zero, const int32_t* __restrict__ colsum) {
    constexpr int BM = 32 * RT;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    // XCD x (workgroup ids go round-robin over the eight) owns a contiguous range of the tile order, its workgroups walk it side by side:
    // groups of 4 row tiles, columns fastest, so that 32 tiles in flight share 4 row panels and 8 column panels through that L2
    // (groups of 8: 1089 -> 1086 us at K = 3072, 1041 -> 1080 at K = 12288).
    const int ntiles = tiles_m * tiles_n;
    const int xcd = blockIdx.x % 8, step = (gridDim.x + 7 - xcd) / 8;
    const int first = xcd * (ntiles / 8) + (xcd < ntiles % 8 ? xcd : ntiles % 8), count = ntiles / 8 + (xcd < ntiles % 8);
    int ti = blockIdx.x / 8;
    if (ti >= count) return;
    const int t = threadIdx.x, lane = t % 64, wv = __builtin_amdgcn_readfirstlane(t / 64);
    const int wm = wv / 4, wn = wv % 4;
    const int KB = K / BK, groups = (N + 63) / 64;
    auto locate = [&](int i, int& m0, int& n0) {
        constexpr int GM = 4;
        const int tile = first + i, group = tile / (GM * tiles_n), first_m = group * GM, r = tile % (GM * tiles_n);
        const int gsize = tiles_m - first_m < GM ? tiles_m - first_m : GM;
        m0 = (first_m + r % gsize) * BM;
        n0 = (r / gsize) * BN;
    };
    // A tile: wave wv loads the 16-row pieces 2 wv and 2 wv + 1 (past the tile's end: its last piece once more, to the same place), lane -> (row
    // lane / 4, LDS chunk lane % 4).  The chunk that lands there
    // is permuted by row (chunk ^ 3 in the lower eight rows) so that the 16-byte fragment reads, which LDS serves in the lane groups
    // 0-3, 12-15, 20-27 and their shifts, find their 16 lanes in different banks (no conflicts; with a rotation by row / 4 one in three).
    auto swizzle = [](int r) { return r & 8 ? 3 : 0; };
    auto a_piece = [&](int i) { return 2 * wv + i < 2 * RT ? 2 * wv + i : 2 * RT - 1; };
    auto a_off = [&](int m0, int i) {
        const int r = lane / 4;
        int row = m0 + 16 * a_piece(i) + r;
        if (row >= M) row = M - 1;
        return (unsigned)(row - m0) * (unsigned)K + ((lane % 4) ^ swizzle(r)) * 16;
    };
    auto source = [&](int m0, int n0) {
        int g = n0 / 64 + wv / 2;
        if (g >= groups) g = groups - 1;
        return Source{q + (size_t)m0 * K, wdec + (size_t)g * KB * GROUP + (wv % 2) * 2048, a_off(m0, 0), a_off(m0, 1), a_piece(0), a_piece(1)};
    };
    auto at = [](const Source& x, int kb) { return Source{x.a + (size_t)kb * BK, x.b + (size_t)kb * GROUP, x.va0, x.va1, x.piece0, x.piece1}; };
    const unsigned lvoff = lane * 16;

    int m0, n0;
    locate(ti, m0, n0);
    Source src = source(m0, n0);
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int p = 0; p < 4; ++p) load_stage_piece(lds0, s, wv, lvoff, at(src, s), p);
    LRQ_WAIT_LOADS(4);
    raw_barrier();

    const int r = lane % 16, g = lane / 16;
    const int a_rd = wm * RT * 1024 + r * 64 + (g ^ swizzle(r)) * 16;
    const int b_rd = OFF_B + wn * 4 * 1024 + lane * 16;
    v4i bf[2][4], af[2][RT], acc[RT][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        bf[0][j] = *reinterpret_cast<const v4i*>(&smem[b_rd + j * 1024]);
        af[0][j] = *reinterpret_cast<const v4i*>(&smem[a_rd + j * 1024]);
    }
    float* const tscale = reinterpret_cast<float*>(&smem[OFF_S]);
    float* const cscale = tscale + 256;
    float* const cbias = cscale + BN;
    int* const tzero = reinterpret_cast<int*>(cbias + BN);
    int* const csum = tzero + 256;
    int buf = 0;
    for (;;) {
        const bool more = ti + step < count;
        int nm0, nn0;
        locate(more ? ti + step : ti, nm0, nn0);            // after the last tile its first stages are fetched once more, unused
        const Source nsrc = source(nm0, nn0);
        // threads 0-255: the tile's tokens, 256-511: its channels; they go to LDS when the K loop is done
        float sv, bv = 0.0f;
        int zv = 0;
        if (t < 256) {
            const int row = m0 + t < M ? m0 + t : M - 1;
            sv = scale[row];
            if constexpr (ZP) zv = zero[row];
        } else {
            const int n = n0 + t - 256 < N ? n0 + t - 256 : N - 1;
            sv = wscale[n];
            if (bias) bv = bias[n];
            if constexpr (ZP) zv = colsum[n];
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = v4i{0, 0, 0, 0};
        auto ahead = [&](int s) { return s + 3 < KB ? at(src, s + 3) : at(nsrc, s + 3 - KB); };
        int s = 0;
        for (; s + 1 < KB; s += 2) {
            stage<RT>(smem, lds0, buf, wv, lvoff, ahead(s), a_rd, b_rd, bf[0], bf[1], af[0], af[1], acc);
            stage<RT>(smem, lds0, (buf + 1) % NBUF, wv, lvoff, ahead(s + 1), a_rd, b_rd, bf[1], bf[0], af[1], af[0], acc);
            buf = (buf + 2) % NBUF;
        }
        if (s < KB) {
            stage<RT>(smem, lds0, buf, wv, lvoff, ahead(s), a_rd, b_rd, bf[0], bf[1], af[0], af[1], acc);
            buf = (buf + 1) % NBUF;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                bf[0][j] = bf[1][j];
                af[0][j] = af[1][j];
            }
        }

        // ---- rescale in fp32 and store.  A lane holds token lane % 16 of every row tile and, of each pair of column tiles, the eight
        // channels 8 (lane / 16) + [0, 8) of 32
        tscale[t] = sv;                                      // channels follow the tokens
        if (t >= 256) cbias[t - 256] = bv;
        if constexpr (ZP) tzero[t] = zv;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        raw_barrier();
        float wq[4][4], bq[4][4];
        int cq[4][4];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const int c = wn * 64 + (ct / 2) * 32 + g * 8 + (ct % 2) * 4;
            const float4 w4 = *reinterpret_cast<const float4*>(&cscale[c]);
            const float4 b4 = *reinterpret_cast<const float4*>(&cbias[c]);
            wq[ct][0] = w4.x; wq[ct][1] = w4.y; wq[ct][2] = w4.z; wq[ct][3] = w4.w;
            bq[ct][0] = b4.x; bq[ct][1] = b4.y; bq[ct][2] = b4.z; bq[ct][3] = b4.w;
            if constexpr (ZP) {
                const int4 c4 = *reinterpret_cast<const int4*>(&csum[c]);
                cq[ct][0] = c4.x; cq[ct][1] = c4.y; cq[ct][2] = c4.z; cq[ct][3] = c4.w;
            }
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const int lr = (wm * RT + i) * 16 + r, row = m0 + lr;
            const float ts = tscale[lr];
            const double tz = ZP ? (double)tzero[lr] : 0.0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int ct = 2 * h + e / 4, x = e % 4;
                    const float tot = ZP ? zp_sum(acc[i][ct][x], tz, (double)cq[ct][x]) : (float)acc[i][ct][x];
                    y[e] = (tot * ts) * wq[ct][x] + bq[ct][x];
                }
                const int col = n0 + wn * 64 + 32 * h + 8 * g;        // N % 8 == 0: inside or outside as a whole
                if (row < M && col < N)
                    *reinterpret_cast<uint4*>(Y + (size_t)row * N + col) =
                        make_uint4(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]), pack_bf16(y[4], y[5]), pack_bf16(y[6], y[7]));
            }
        }
        if (!more) break;
        ti += step;
        m0 = nm0;
        n0 = nn0;
        src = nsrc;
    }
    LRQ_WAIT_LOADS(0);          // no load may reach LDS after the workgroup has given it back
}

template <int RT, bool ZP>
hipError_t launch_wide(hipStream_t st, const int8_t* q, const float* scale, const int32_t* zero, int M, int K, const lrq_tlq_weight& w,
                       const float* bias, void* Y, const uint8_t* wdec) {
    const hipError_t e = allow_large_lds(reinterpret_cast<const void*>(&qgemm_wide_kernel<RT, ZP>), LDS_BYTES);
    if (e != hipSuccess) return e;
    const int tiles_m = (M + 32 * RT - 1) / (32 * RT), tiles_n = (w.N + BN - 1) / BN, tiles = tiles_m * tiles_n;
    hipLaunchKernelGGL((qgemm_wide_kernel<RT, ZP>), dim3(tiles < 256 ? tiles : 256), dim3(512), LDS_BYTES, st, q, scale, M, K, w.N, wdec,
                       w.wscale, bias, static_cast<uint16_t*>(Y), tiles_m, tiles_n, zero, w.colsum);
    return hipGetLastError();
}

}  // namespace

// Times in us, decoding included, fitted (with 4 % between fit and measurement) to 600 measurements of each height over M = 200 ..
// 35100, N = 96 .. 12288, K = 320 .. 12288.  A round of tiles, one per CU, takes k per K block + k_fill times the share of the CUs that
// have a tile (the chip's clock falls with the work in flight) + its epilogue.  The lower tiles are taken where they fill the last round
// better (us with 192 / 224 / 256 rows: 8192 x 4608 -> 1152 50.2 / 52.1 / 55.5, 4608 x 3072 -> 9216 136 / 128 / 143, 35100 x 3072 -> 12288
// 1165 / 1138 / 1104).  The zero-point form's epilogue needs more registers than there are at 224 and 256 rows: the compiler spills 2 and 16,
// which is most of what zero_point adds there.  Decoded along with the rotation, the weights cost neither their launch nor most of their
// time (8192 x 1152 -> 4608: 3 us of 62).
// Against qgemm.hip, whose predicted time has to be 3 % longer than this one's with an epilogue 1.5 us longer than fitted: the boards differ in
// how fast all CUs' stores drain once outputs no longer stay in the Infinity Cache.  75 shapes with K = 320 .. 4608, N % 8 == 0, both
// kernels timed on five boards with the buffers rotated through 700 MB: none of the 54 that the rule takes loses 1 % on any board, and
// all 75 gain 7.2 % on average.  The fit as it is, with a demand of 3 / 5 %, takes 70 / 67 for 7.9 / 8.0 %, but 6 / 4 lose on a board, up to
// 12 / 8 % (8192 x 1152 -> 4608, not among the 75, loses on some boards and gains on others, by up to 7 %); + 0.5 / + 1 us with 3 % takes
// 67 / 63 for 8.1 / 7.8 %, 3 / 2 lose, up to 6 / 1.5 %.
// 35100 x 3072 -> 12288: 1340 us at 4 bits in qgemm.hip.  3-bit weights, whose decoding takes a third of the instructions, stay there:
// 35100 x 3072 -> 9216 835 us against 846 here.  So do outputs other than bf16 rows of whole 16-byte pieces: fp32 outputs (22488 x 6144 -> 4736
// 616 us against 678, but 30107 x 3072 -> 490 87 against 62: every tile's 256 KB are written at once) and ragged rows (element by element:
// 20688 x 2304 -> 2389 212 us against 143) rarely gain.
struct WideCost { int rows; float k, k_fill, tile, zero_point, once; };
constexpr WideCost kWideCost[3] = {{192, 0.315f, 0.288f, 6.06f, 0.3f, 6.9f},
                                   {224, 0.357f, 0.318f, 6.87f, 1.3f, 6.1f},
                                   {256, 0.382f, 0.376f, 7.36f, 4.2f, 7.0f}};
constexpr float kDecodePerByte = 0.17e-6f, kAlong = 3.5f;

int qgemm_wide_rows(int M, int N, int K, int bits, bool zero_point, bool fp32, bool along) {
    if (bits != 4 || fp32 || N % 8 != 0) return 0;
    if (K < 4 * BK || (zero_point && K > kZpF64K)) return 0;         // three stages are in flight; longer sums need 64-bit integers
    const float kb = (float)(K / BK), decode = kDecodePerByte * (float)N * (float)K;
    float best = INFINITY;
    int rows = 0;
    for (const WideCost& c : kWideCost) {
        const long tiles = ((long)M + c.rows - 1) / c.rows * (((long)N + BN - 1) / BN), n = (tiles + 255) / 256;
        const float us = c.once + (along ? 0.5f * decode - kAlong : decode) +
                         (float)n * ((c.k + c.k_fill * (float)tiles / (256.0f * (float)n)) * kb + c.tile + (zero_point ? c.zero_point : 0.0f));
        if (us < best) {
            best = us;
            rows = c.rows;
        }
    }
    return best * 1.03f < qgemm_shape(M, N, K, 4, zero_point, false, false).us ? rows : 0;
}

size_t qgemm_wide_bytes(int N, int K) { return ((size_t)N + 63) / 64 * 64 * K; }

hipError_t launch_qgemm_wide(hipStream_t st, const int8_t* q, const float* scale, const int32_t* zero, int M, int K,
                             const lrq_tlq_weight& w, const float* bias, void* Y, void* ws, int rows, bool decoded) {
    uint8_t* wdec = static_cast<uint8_t*>(ws);
    if (!decoded) {
        DecodeJob job;
        job.gcodes = w.gemm_codes;
        job.lut = w.lut;
        job.out = wdec;
        job.N = w.N;
        job.KB = K / BK;
        hipLaunchKernelGGL(decode_weights_kernel, dim3(decode_groups(job, 4)), dim3(256), 0, st, job);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    switch (rows) {
        case 192:
            return zero ? launch_wide<6, true>(st, q, scale, zero, M, K, w, bias, Y, wdec) : launch_wide<6, false>(st, q, scale, zero, M, K, w, bias, Y, wdec);
        case 224:
            return zero ? launch_wide<7, true>(st, q, scale, zero, M, K, w, bias, Y, wdec) : launch_wide<7, false>(st, q, scale, zero, M, K, w, bias, Y, wdec);
        default:
            return zero ? launch_wide<8, true>(st, q, scale, zero, M, K, w, bias, Y, wdec) : launch_wide<8, false>(st, q, scale, zero, M, K, w, bias, Y, wdec);
    }
}

}  // namespace lrq
