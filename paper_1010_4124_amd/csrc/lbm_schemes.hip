// lbm_schemes.hip -- the comparison convection schemes of Sec. III.B of
// arXiv:1010.4124 (Fig. 2): first- and second-order upwind fluxes in the same
// forward-Euler step (Eq. (47)) as the WENO5 path, by the whole-tile kernel
// (lbm_tile.h) with their faces in place of the WENO5 ones. The face at I+1/2
// from the upwind-ordered samples (b, c) = (f_{I-1}, f_I) (or their mirror
// images for v < 0) is c (first order) or c + (c - b)/2 (second order), times v.
//
// Bound by the latency of a tile on small grids (400 x 4 shock tube, second
// order: 6.1 us a step, against 54 with one thread per cell that took the 18
// velocities in turn in 7 workgroups) and by moving the planes on large ones
// (2048^2: 275 us, 4.6 TB/s of the 304 B per cell, against 1405).
#include "lbm_device.h"
#include "lbm_internal.h"
#include "lbm_stage.h"
#include "lbm_step.h"
#include "lbm_tile.h"

namespace lbmd {

template <int R, int SCHEME>
__global__ __launch_bounds__((64 * tile_waves(R))) __attribute__((amdgpu_waves_per_eu(6)))
void k_step_lo(TileArgs a)
{
    __shared__ double lds[TileWg<R>::LDS];
    tile_block<R, false, SCHEME>(a, lds);
}

hipError_t launch_step_lo(int scheme, int R, const double* fin, double* fout, const Consts& k,
                          double* ke_part, int nx, int ny, const int bc[4], double cx, double cy,
                          double ct, int ke_axis, const double* const gb[4], hipStream_t st)
{
    StepGrid s;
    s.fin = fin;
    s.fout = fout;
    s.nx = nx;
    s.ny = ny;
    s.ke_axis = ke_axis;
    for (int j = 0; j < 4; ++j) {
        s.bc[j] = bc[j];
        s.gb[j] = gb ? gb[j] : nullptr;
    }
    s.cx = cx;
    s.cy = cy;
    s.ct = ct;
    void (*const kernels[3][2])(TileArgs) = {{k_step_lo<1, 1>, k_step_lo<1, 2>},
                                             {k_step_lo<2, 1>, k_step_lo<2, 2>},
                                             {k_step_lo<4, 1>, k_step_lo<4, 2>}};
    return launch_tiles(kernels[R >> 1][scheme == 1 ? 0 : 1], tile_args(s, k, ke_part, R), R, st);
}

}  // namespace lbmd
