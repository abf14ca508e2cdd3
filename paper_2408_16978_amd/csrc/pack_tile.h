// One 32-row block of one head of a row-major [rows, H, D] bf16 tensor into MFMA fragment order (fpdt_internal.h), by NT threads.
#pragma once
#include "fpdt_internal.h"

namespace fpdt {

struct PackJobs {
    PackJob job[PACK_MAX_JOBS];
};

// Block rb of head h, counted over the heads of all jobs
template <int D, int NT>
__device__ __forceinline__ void pack_tile(const PackJobs& jobs, int64_t head_stride_blocks, int64_t rb, int h)
{
    constexpr int DT = D / 16, DP = (D + 31) / 32 * 32, DB = DP / 32;
    constexpr int LD = DP + 2;  // padded row (in bf16) to spread LDS banks on column reads
    __shared__ uint16_t tile[32 * LD];
    int which = 0;
#pragma unroll
    for (int i = 0; i < PACK_MAX_JOBS - 1; ++i)
        if (which == i && h >= jobs.job[i].H) { h -= jobs.job[i].H; ++which; }
    const PackJob job = jobs.job[which];
    const uint16_t* __restrict__ X = static_cast<const uint16_t*>(job.X);
    uint4* __restrict__ nat = static_cast<uint4*>(job.nat);
    uint4* __restrict__ tr = static_cast<uint4*>(job.tr);
    const int H = job.H;
    const int tid = threadIdx.x;
    // load 32 rows x D (8 bf16 = 16 B per thread per step)
    constexpr int VEC_PER_ROW = D / 8;
    for (int i = tid; i < 32 * VEC_PER_ROW; i += NT) {
        const int r = i / VEC_PER_ROW, c = (i % VEC_PER_ROW) * 8;
        const uint4 v = *reinterpret_cast<const uint4*>(X + ((size_t)(rb * 32 + r) * H + h) * D + c);
        const uint16_t* e = reinterpret_cast<const uint16_t*>(&v);
#pragma unroll
        for (int k = 0; k < 8; ++k) tile[r * LD + c + k] = e[k];
    }
    if (DP != D) {
        for (int i = tid; i < 32 * (DP - D); i += NT) {
            const int r = i / (DP - D), c = D + i % (DP - D);
            tile[r * LD + c] = 0;
        }
    }
    __syncthreads();
    const size_t blk = (size_t)h * head_stride_blocks + rb;
    if (nat) {
        uint4* out = nat + blk * (DT * 64);
        for (int i = tid; i < DT * 64; i += NT) {
            const int t = i >> 6, lane = i & 63;
            const int r = lane & 31, hh = lane >> 5;
            uint16_t e[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) e[k] = tile[r * LD + 16 * t + 8 * hh + k];
            out[i] = *reinterpret_cast<const uint4*>(e);
        }
    }
    if (tr) {
        uint4* out = tr + blk * (2 * DB * 64);
        for (int i = tid; i < 2 * DB * 64; i += NT) {
            const int lane = i & 63, db = (i >> 6) % DB, s = (i >> 6) / DB;
            const int c = lane & 31, hh = lane >> 5;
            uint16_t e[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                e[k] = tile[(8 * (2 * s + (k >> 2)) + 4 * hh + (k & 3)) * LD + 32 * db + c];
            out[i] = *reinterpret_cast<const uint4*>(e);
        }
    }
}

}  // namespace fpdt
