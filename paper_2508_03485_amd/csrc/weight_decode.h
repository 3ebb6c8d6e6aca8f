// Decoding of 4-bit weight codes to int8 levels in the operand order of the wide GEMM.
#pragma once
#include "lrq_internal.h"

namespace lrq {
namespace {

constexpr int kWideGroup = 64 * kGemmBlockK;         // bytes of a 64-channel group of decoded weights in one K block

// int8 levels of four 4-bit codes, one in the low nibble of each byte of w (level table of the codes' channel: entries 0-7 in L[0..1],
// 8-15, the negative twin, in L[2..3])
__device__ __forceinline__ unsigned decode_codes4(unsigned w, const unsigned (&L)[4]) {
    const unsigned idx = w & 0x07070707u;
    const unsigned lo = __builtin_amdgcn_perm(L[1], L[0], idx), hi = __builtin_amdgcn_perm(L[3], L[2], idx);
    return __builtin_amdgcn_perm(hi, lo, ((w >> 1) & 0x04040404u) | 0x03020100u);
}

// Decoded weights: [64-channel group][K block][16-column tile ct 0..3][k chunk 0..3][column i 0..15] of 16 bytes (k = 16 chunk +
// [0, 16) of the block): 1 KB a tile, the order of a wave's operand registers.  Column i of tile ct is channel
// 32 (ct / 2) + 8 (i / 4) + 4 (ct % 2) + i % 4 of the group, so that a lane's accumulators of two neighbouring tiles are eight
// neighbouring channels: 16 bytes of bf16, and the four lanes of a token store 64 contiguous bytes without a pass through LDS.
// One wave per (32-channel tile, K block) unit of the code tiling; lane = its slot (lrq_internal.h).  Workgroup `id` of the job: tile id % tiles,
// its waves every (workgroups per tile x waves)-th K block.
__device__ __forceinline__ void decode_weights(const DecodeJob& job, int id, int groups, int waves) {
    const int tiles = (job.N + 31) / 32, tl = id % tiles, lane = threadIdx.x % 64, c = lane % 16;
    unsigned L[2][4];
    int off[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        int n = tl * 32 + h * 16 + c;
        if (n >= job.N) n = job.N - 1;
        const uint4 lv = *reinterpret_cast<const uint4*>(job.lut + (size_t)n * 16);
        L[h][0] = lv.x; L[h][1] = lv.y; L[h][2] = lv.z; L[h][3] = lv.w;
        const int m = h * 16 + c;
        off[h] = ((tl % 2) * 2 + (m / 4) % 2) * 1024 + ((m / 8) * 4 + m % 4) * 16;
    }
    const uint8_t* src = job.gcodes + (size_t)tl * job.KB * 1024 + lane * 16;
    uint8_t* dst = job.out + (size_t)(tl / 2) * job.KB * kWideGroup + (lane / 16) * 256;
    for (int kb = id / tiles * waves + threadIdx.x / 64; kb < job.KB; kb += groups / tiles * waves) {
        const uint4 raw = *reinterpret_cast<const uint4*>(src + (size_t)kb * 1024);
        const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint4 o;
            o.x = decode_codes4(w[2 * h], L[h]);
            o.y = decode_codes4(w[2 * h] >> 4, L[h]);
            o.z = decode_codes4(w[2 * h + 1], L[h]);
            o.w = decode_codes4(w[2 * h + 1] >> 4, L[h]);
            *reinterpret_cast<uint4*>(dst + (size_t)kb * kWideGroup + off[h]) = o;
        }
    }
}

// workgroups for a job: a multiple of its tiles, about four K blocks to a wave
inline unsigned decode_groups(const DecodeJob& job, int waves) {
    const int parts = (job.KB + 4 * waves - 1) / (4 * waves);
    return (unsigned)((job.N + 31) / 32 * parts);
}

}  // namespace
}  // namespace lrq
