// Re-layout of [rows, H, D] bf16 tensors into MFMA fragment order (see fpdt_internal.h).
// HBM-bound streaming kernel: each workgroup stages one 32-row x D tile of one head in
// LDS and writes it back as NAT and/or TR fragments, 16 bytes per lane, fully coalesced.  The
// tensors of a call that have the same rows share a launch (at 2K tokens a launch costs as much as
// its work: forward 29.4 -> 27.4 us).
#include "fpdt_internal.h"
#include "pack_tile.h"

namespace fpdt {

template <int D>
__global__ __launch_bounds__(256) void pack_kernel(PackJobs jobs, int64_t head_stride_blocks)
{
    pack_tile<D, 256>(jobs, head_stride_blocks, blockIdx.x, (int)blockIdx.y);
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
