// Re-layout of [rows, H, D] bf16 tensors into MFMA fragment order (see fpdt_internal.h).
// HBM-bound streaming kernel: each workgroup stages one 32-row x D tile of one head in
// LDS and writes it back as NAT and/or TR fragments, 16 bytes per lane, fully coalesced.  The
// tensors of a call that have the same rows share a launch (at 2K tokens a launch costs as much as
// its work: forward 29.4 -> 27.4 us).
#include "fpdt_internal.h"
#include "mfma_tiles.h"

namespace fpdt {

struct PackJobs {
    PackJob job[PACK_MAX_JOBS];
};

template <int D>
__global__ __launch_bounds__(256) void pack_kernel(PackJobs jobs, int64_t head_stride_blocks)
{
    constexpr int DT = D / 16, DP = (D + 31) / 32 * 32, DB = DP / 32;
    constexpr int LD = DP + 2;  // padded row (in bf16) to spread LDS banks on column reads
    __shared__ uint16_t tile[32 * LD];
    const int64_t rb = blockIdx.x;
    int h = blockIdx.y, which = 0;  // blockIdx.y counts the heads of all jobs
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
    for (int i = tid; i < 32 * VEC_PER_ROW; i += 256) {
        const int r = i / VEC_PER_ROW, c = (i % VEC_PER_ROW) * 8;
        const uint4 v = *reinterpret_cast<const uint4*>(X + ((size_t)(rb * 32 + r) * H + h) * D + c);
        const uint16_t* e = reinterpret_cast<const uint16_t*>(&v);
#pragma unroll
        for (int k = 0; k < 8; ++k) tile[r * LD + c + k] = e[k];
    }
    if (DP != D) {
        for (int i = tid; i < 32 * (DP - D); i += 256) {
            const int r = i / (DP - D), c = D + i % (DP - D);
            tile[r * LD + c] = 0;
        }
    }
    __syncthreads();
    const size_t blk = (size_t)h * head_stride_blocks + rb;
    if (nat) {
        uint4* out = nat + blk * (DT * 64);
        for (int i = tid; i < DT * 64; i += 256) {
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
        for (int i = tid; i < 2 * DB * 64; i += 256) {
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

void launch_pack(std::initializer_list<PackJob> tensors, int64_t rows, int D, int64_t head_stride_blocks, hipStream_t st)
{
    if (rows <= 0) return;
    PackJobs jobs = {};
    unsigned heads = 0;
    int n = 0;
    for (const PackJob& j : tensors) {
        jobs.job[n++] = j;
        heads += (unsigned)j.H;
    }
    if (heads > 65535 && n > 1) {  // the grid's second dimension
        for (const PackJob& j : tensors) launch_pack({j}, rows, D, head_stride_blocks, st);
        return;
    }
    dim3 grid((unsigned)(rows / 32), heads);
    if (D == 128) pack_kernel<128><<<grid, 256, 0, st>>>(jobs, head_stride_blocks);
    else if (D == 80) pack_kernel<80><<<grid, 256, 0, st>>>(jobs, head_stride_blocks);
    else pack_kernel<64><<<grid, 256, 0, st>>>(jobs, head_stride_blocks);
}

}  // namespace fpdt
