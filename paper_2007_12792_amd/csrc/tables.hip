// gfx950 kernel that fills a tree's ghost table on the device, coarser neighbours as virtual blocks.  Made on the host, the table
// (540 bytes per block, twice) took most of the time of a regrid, in page faults, scattered reads and the copy over PCIe; its source is
// 30 bytes per block.  (Tree of 27,756 blocks: upload 0.62 -> 0.15 ms; the regrid to
// it with 24 fields, from seeds to fields on the new tree, 7.3 -> 2.5.)
#include "kernels.hpp"

namespace octfd {
namespace {

__global__ __launch_bounds__(256) void k_ghost_table(TableSource t, int64_t entries, int32_t* __restrict__ out)
{
    const int64_t n = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (n >= entries) return;
    int32_t e[kEntry];
    table_entry(t, n / kDirs, static_cast<int>(n % kDirs), true, e);
#pragma unroll
    for (int m = 0; m < kEntry; ++m) out[n * kEntry + m] = e[m];
}

}  // namespace

hipError_t launch_ghost_table(const TableSource& t, int64_t nb, int32_t* ghost_v, hipStream_t s)
{
    int64_t entries = nb * kDirs;
    // the launch's own status: hipGetLastError() may return one that an earlier call of the program has left, and the caller is uploading a tree
    TableSource source = t;
    void* args[] = {&source, &entries, &ghost_v};
    return hipLaunchKernel(reinterpret_cast<const void*>(k_ghost_table), dim3(static_cast<unsigned>((entries + 255) / 256)), dim3(256), args, 0, s);
}

}  // namespace octfd
