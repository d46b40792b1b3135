// cvo_device.hpp -- device helpers shared by the planner and the pair pass.
#pragma once
#include "cvo_internal.hpp"

namespace cvo {

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Inclusive scans over the 64 lanes of a wave with DPP row shifts and row
// broadcasts (no LDS traffic): within each row of 16 lanes a Hillis-Steele
// scan over shifts 1, 2, 4, 8 (lanes shifted in from outside the row add
// the identity 0), then row 0's last lane is added to row 1 and row 2's to
// row 3, then lane 31 to rows 2 and 3.  The max scan needs values >= 0.
__device__ __forceinline__ int wave_scan_add(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

__device__ __forceinline__ int wave_scan_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));
    return v;
}

// Cells [i0, i1] along one axis covering [c - R, c + R]; false if none.
// Uses the same floor((p - o) * inv_h) as the binning.
__device__ __forceinline__ bool axis_range(double c, double R, double o, double inv_h, int n, int &i0, int &i1)
{
    const double f0 = floor(((c - R) - o) * inv_h);
    const double f1 = floor(((c + R) - o) * inv_h);
    if (!(f1 >= 0.0) || !(f0 <= (double)(n - 1))) return false;
    i0 = (int)fmax(f0, 0.0);
    i1 = (int)fmin(f1, (double)(n - 1));
    return true;
}

// Geometry shared by the planner and the pass: the cluster centre in the
// reference frame, the cull radius, and the cell ranges of its neighbourhood.
struct Neighbourhood {
    double cx, cy, cz, Rm;
    int ix0, ix1, iy0, iy1, iz0, iz1;
    bool any;
};

__device__ __forceinline__ Neighbourhood neighbourhood(const double *Pm, const double4 g, double rc, bool cut,
                                                       const GridDesc &gd)
{
    Neighbourhood nb;
    nb.cx = Pm[0] * g.x + Pm[1] * g.y + Pm[2] * g.z + Pm[3];
    nb.cy = Pm[4] * g.x + Pm[5] * g.y + Pm[6] * g.z + Pm[7];
    nb.cz = Pm[8] * g.x + Pm[9] * g.y + Pm[10] * g.z + Pm[11];
    nb.Rm = cut ? (rc + g.w) * (1.0 + 1e-5) : INFINITY;
    nb.ix0 = 0; nb.ix1 = gd.nx - 1; nb.iy0 = 0; nb.iy1 = gd.ny - 1; nb.iz0 = 0; nb.iz1 = gd.nz - 1;
    nb.any = gd.n > 0;
    if (cut && nb.any)
        nb.any = axis_range(nb.cx, nb.Rm, gd.ox, gd.inv_h, gd.nx, nb.ix0, nb.ix1) &&
                 axis_range(nb.cy, nb.Rm, gd.oy, gd.inv_h, gd.ny, nb.iy0, nb.iy1) &&
                 axis_range(nb.cz, nb.Rm, gd.oz, gd.inv_h, gd.nz, nb.iz0, nb.iz1);
    return nb;
}

}  // namespace cvo
