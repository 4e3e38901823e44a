// Field update of the 3-D patch-PIC step (the block bodies are in
// maxwell3d.h): the fused Yee kernel and the three passes of the sixth-order
// solver.
#include "kernels.h"
#include "maxwell3d.h"

namespace pic {

namespace {

template <typename T, int PASS>
__global__ __launch_bounds__(kMB) void k_maxwell3d_b(const SimDev<T> *__restrict__ sims, int nsims,
                                                     const int *__restrict__ tile_prefix, int total)
{
    hi3d_b_tiles<T, PASS>(sims, nsims, tile_prefix, total, blockIdx.x, gridDim.x);
}

template <typename T>
__global__ __launch_bounds__(kMB) void k_maxwell3d_e(const SimDev<T> *__restrict__ sims, int nsims,
                                                     const int *__restrict__ tile_prefix, int total)
{
    hi3d_e_tiles<T>(sims, nsims, tile_prefix, total, blockIdx.x, gridDim.x);
}

template <typename T>
__global__ __launch_bounds__(kYT) void k_maxwell3d_yee(const SimDev<T> *__restrict__ sims, int nsims,
                                                       const int *__restrict__ tile_prefix, int total)
{
    yee3d_blocks<T>(sims, nsims, tile_prefix, total, blockIdx.x, gridDim.x);
}

}  // namespace

template <typename T>
void launch_maxwell3d(const SimDev<T> *sims, int nsims, const int *tile_prefix, int total_tiles,
                      int grid, bool yee, bool hi_order, hipStream_t st, Ev2 ev)
{
    if (yee)
        hipExtLaunchKernelGGL((k_maxwell3d_yee<T>), dim3(grid), dim3(kYT), 0, st, ev.start,
                              hi_order ? nullptr : ev.stop, 0, sims, nsims, tile_prefix, total_tiles);
    if (!hi_order) return;
    hipExtLaunchKernelGGL((k_maxwell3d_b<T, 0>), dim3(grid), dim3(kMB), 0, st, yee ? nullptr : ev.start,
                          nullptr, 0, sims, nsims, tile_prefix, total_tiles);
    hipLaunchKernelGGL((k_maxwell3d_e<T>), dim3(grid), dim3(kMB), 0, st, sims, nsims, tile_prefix,
                       total_tiles);
    hipExtLaunchKernelGGL((k_maxwell3d_b<T, 2>), dim3(grid), dim3(kMB), 0, st, nullptr, ev.stop, 0,
                          sims, nsims, tile_prefix, total_tiles);
}

template void launch_maxwell3d<float>(const SimDev<float> *, int, const int *, int, int, bool, bool,
                                      hipStream_t, Ev2);
template void launch_maxwell3d<double>(const SimDev<double> *, int, const int *, int, int, bool, bool,
                                       hipStream_t, Ev2);

}  // namespace pic
