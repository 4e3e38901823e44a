// Field update of the 2-D patch-PIC step (the bodies are in maxwell2d.h):
// the Yee kernels and the three passes of the sixth-order solver.
#include "kernels.h"
#include "maxwell2d.h"

namespace pic {

namespace {

template <typename T, int TX, int TY>
__global__ __launch_bounds__(256) void k_maxwell2d(const SimDev<T> *__restrict__ sims, int nsims,
                                                   const int *__restrict__ tile_prefix, int total)
{
    yee2d_tiles<T, TX, TY>(sims, nsims, tile_prefix, total, blockIdx.x, gridDim.x);
}

template <typename T>
__global__ __launch_bounds__(256) void k_maxwell2d_march(const SimDev<T> *__restrict__ sims, int nsims,
                                                         const int *__restrict__ tile_prefix, int total)
{
    yee2d_march<T>(sims, nsims, tile_prefix, total, blockIdx.x, gridDim.x);
}

template <typename T, int PASS>
__global__ __launch_bounds__(256) void k_maxwell2d_hi(const SimDev<T> *__restrict__ sims, int nsims,
                                                      const int *__restrict__ tile_prefix, int total,
                                                      int TX, int TY)
{
    hi2d_tiles<T, PASS>(sims, nsims, tile_prefix, total, TX, TY, blockIdx.x, gridDim.x);
}

}  // namespace

// Tile shapes (TX x TY nodes per workgroup) the tuner can choose from.
// (0: the sixth-order solver only, Yee takes strips).  FP32 tiles hold 9 x (TX+3)(TY+3) floats of LDS, FP64 tiles doubles.
namespace {
constexpr int kTiles32[6][2] = {{64, 16}, {64, 8}, {128, 8}, {32, 16}, {32, 32}, {128, 4}};
constexpr int kTiles64[6][2] = {{64, 8}, {32, 16}, {32, 8}, {16, 16}, {64, 4}, {128, 4}};
}  // namespace

template <typename T>
void maxwell_tile(int preset, int &tx, int &ty)
{
    const int p = (preset >= 0 && preset < 6) ? preset : 0;
    tx = sizeof(T) == 4 ? kTiles32[p][0] : kTiles64[p][0];
    ty = sizeof(T) == 4 ? kTiles32[p][1] : kTiles64[p][1];
}

template <typename T>
void launch_maxwell(const SimDev<T> *sims, int nsims, const int *tile_prefix, int total_tiles,
                    int grid, int preset, bool yee, bool hi_order, hipStream_t st, Ev2 ev)
{
    hipEvent_t stop1 = hi_order ? nullptr : ev.stop;
#define PIC_MW(TX, TY)                                                                          \
    hipExtLaunchKernelGGL((k_maxwell2d<T, TX, TY>), dim3(grid), dim3(256), 0, st, ev.start,    \
                          stop1, 0, sims, nsims, tile_prefix, total_tiles)
    const int p = (preset >= 0 && preset < 6) ? preset : 0;
    if (!yee) {
        // every simulation of the batch uses the sixth-order solver
    } else if (p == 0) {
        hipExtLaunchKernelGGL((k_maxwell2d_march<T>), dim3((total_tiles + kStripsPerWg - 1) / kStripsPerWg), dim3(256),
                              0, st, ev.start, stop1, 0, sims, nsims, tile_prefix, total_tiles);
    } else if constexpr (sizeof(T) == 4) {
        switch (p) {
        case 1: PIC_MW(64, 8); break;
        case 2: PIC_MW(128, 8); break;
        case 3: PIC_MW(32, 16); break;
        case 4: PIC_MW(32, 32); break;
        default: PIC_MW(128, 4); break;
        }
    } else {
        switch (p) {
        case 1: PIC_MW(32, 16); break;
        case 2: PIC_MW(32, 8); break;
        case 3: PIC_MW(16, 16); break;
        case 4: PIC_MW(64, 4); break;
        default: PIC_MW(128, 4); break;
        }
    }
#undef PIC_MW
    if (hi_order) {
        // the sixth-order simulations of the batch (the Yee kernel skipped their tiles)
        int tx, ty;
        maxwell_tile<T>(preset, tx, ty);
        hipExtLaunchKernelGGL((k_maxwell2d_hi<T, 0>), dim3(grid), dim3(256), 0, st, yee ? nullptr : ev.start,
                              nullptr, 0, sims, nsims, tile_prefix, total_tiles, tx, ty);
        hipLaunchKernelGGL((k_maxwell2d_hi<T, 1>), dim3(grid), dim3(256), 0, st, sims, nsims, tile_prefix,
                           total_tiles, tx, ty);
        hipExtLaunchKernelGGL((k_maxwell2d_hi<T, 2>), dim3(grid), dim3(256), 0, st, nullptr, ev.stop, 0,
                              sims, nsims, tile_prefix, total_tiles, tx, ty);
    }
}

template void maxwell_tile<float>(int, int &, int &);
template void maxwell_tile<double>(int, int &, int &);
template void launch_maxwell<float>(const SimDev<float> *, int, const int *, int, int, int, bool, bool,
                                    hipStream_t, Ev2);
template void launch_maxwell<double>(const SimDev<double> *, int, const int *, int, int, int, bool, bool,
                                     hipStream_t, Ev2);

}  // namespace pic
