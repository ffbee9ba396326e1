// What the two forms of the SSIM kernel share: the window and the reciprocal.
#ifndef GM_SSIM_CORE_H
#define GM_SSIM_CORE_H
#include "gm_internal.h"

namespace ssimcore {

constexpr int R = 5, WN = 2 * R + 1;               // the window's half width and taps
constexpr int MAX_PARTS = GM_REDUCE_WORKSPACE_BYTES / 8;    // one FP64 sum a block

// 1/d from the hardware reciprocal refined by two Newton steps (error ~1 ulp); here
// d = b1 b2 lies in [C1 C2, 4.1]
__device__ __forceinline__ double recip(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    return fma(r, fma(-d, r, 1.0), r);
}

}  // namespace ssimcore

// The form in 32 x 32 tiles (ssim_tiles.hip): columns and rows of a tile, and the launch over a's
// tiles (tiles_x, tiles_y, tile_begin), whose sums go to part; returns the sums written.
constexpr int SSIM_TILE = 32;
int launch_ssim_tiles(const SsimArgs& a, double* part, hipStream_t s);
#endif
