// Field update and re-binning side by side in one launch, for small batches:
// the first workgroups take the field strips or tiles, the others a pass of the
// re-binning (the two share no data).  On two streams the fork and the join
// cost about 7 us per step, as much as the passes of a small box themselves
// (128 x 128 box: field update 6 us and the three launches of the re-binning 20 us
// by themselves, 18 us together here); here they cost nothing.  Yee: one launch
// with the count pass; sixth order: its three passes go with the count, check and
// scatter passes.
#include <algorithm>

#include "kernels.h"
#include "maxwell2d.h"
#include "maxwell3d.h"
#include "rebin_common.h"

namespace pic {

namespace {

constexpr int kNT = 256;
static_assert(kMB == kNT && kYT == kNT && kRC == kNT, "one workgroup size for both parts");

// PASS 0: Yee and count; 1, 2, 3: the sixth-order passes with count, check
// and scatter.  The first field_wgs workgroups take the fields.
template <typename T, int ND, int PASS>
__global__ __launch_bounds__(kNT) void k_fields_rebin(const SimDev<T> *__restrict__ sims, int nsims,
                                                      const int *__restrict__ tile_prefix, int tiles,
                                                      int field_wgs, const int *__restrict__ patch_prefix,
                                                      int patches, int TX, int TY)
{
    const int b = blockIdx.x;
    if (b < field_wgs) {
        if constexpr (ND == kNDir3) {
            if constexpr (PASS == 0) yee3d_blocks<T>(sims, nsims, tile_prefix, tiles, b, field_wgs);
            if constexpr (PASS == 1) hi3d_b_tiles<T, 0>(sims, nsims, tile_prefix, tiles, b, field_wgs);
            if constexpr (PASS == 2) hi3d_e_tiles<T>(sims, nsims, tile_prefix, tiles, b, field_wgs);
            if constexpr (PASS == 3) hi3d_b_tiles<T, 2>(sims, nsims, tile_prefix, tiles, b, field_wgs);
        } else {
            if constexpr (PASS == 0)
                yee2d_march<T>(sims, nsims, tile_prefix, tiles, b, field_wgs);
            else
                hi2d_tiles<T, PASS - 1>(sims, nsims, tile_prefix, tiles, TX, TY, b, field_wgs);
        }
        return;
    }
    const int wg = b - field_wgs, nwg = (int)gridDim.x - field_wgs;
    if constexpr (PASS <= 1) rebin_count_patches<T, ND, kNT>(sims, nsims, patch_prefix, patches, wg, nwg);
    if constexpr (PASS == 2) rebin_check_patches<T, ND>(sims, nsims, patch_prefix, patches, wg);
    if constexpr (PASS == 3) rebin_scatter_patches<T, ND, kNT>(sims, nsims, patch_prefix, patches, wg, nwg);
}

template <typename T, int ND>
void launch_nd(const SimDev<T> *sims, int nsims, const int *tile_prefix, int tiles, int field_wgs,
               const int *patch_prefix, int patches, int rebin_grid, bool hi_order, hipStream_t st)
{
    int tx, ty;
    maxwell_tile<T>(0, tx, ty);
    if (ND == kNDir2 && !hi_order) field_wgs = (tiles + kStripsPerWg - 1) / kStripsPerWg;
    const int check_wgs = (int)(((int64_t)patches * kCheckLanes<ND> + kNT - 1) / kNT);
#define PIC_FR(PASS, N)                                                                                     \
    hipLaunchKernelGGL((k_fields_rebin<T, ND, PASS>), dim3(field_wgs + (N)), dim3(kNT), 0, st, sims, nsims, \
                       tile_prefix, tiles, field_wgs, patch_prefix, patches, tx, ty)
    if (hi_order) {
        PIC_FR(1, patches);
        PIC_FR(2, check_wgs);
        PIC_FR(3, rebin_grid);
    } else {
        PIC_FR(0, patches);
        launch_rebin_rest<T>(sims, nsims, patch_prefix, patches, rebin_grid, ND == kNDir3 ? 3 : 2, st);
    }
#undef PIC_FR
}

}  // namespace

template <typename T>
void launch_fields_rebin(const SimDev<T> *sims, int nsims, const int *tile_prefix, int tiles, int field_wgs,
                         const int *patch_prefix, int patches, int rebin_grid, int ndim, bool hi_order,
                         hipStream_t st)
{
    if (ndim == 3)
        launch_nd<T, kNDir3>(sims, nsims, tile_prefix, tiles, field_wgs, patch_prefix, patches, rebin_grid,
                             hi_order, st);
    else
        launch_nd<T, kNDir2>(sims, nsims, tile_prefix, tiles, field_wgs, patch_prefix, patches, rebin_grid,
                             hi_order, st);
}

template void launch_fields_rebin<float>(const SimDev<float> *, int, const int *, int, int, const int *, int,
                                         int, int, bool, hipStream_t);
template void launch_fields_rebin<double>(const SimDev<double> *, int, const int *, int, int, const int *, int,
                                          int, int, bool, hipStream_t);

}  // namespace pic
