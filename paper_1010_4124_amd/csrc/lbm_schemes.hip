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
// (2048^2: 270 us, 4.7 TB/s of the 304 B per cell, against 1405). Temporal
// stores at all sizes; non-temporal ones, with plain wave priority around the
// loads, take 250 us there and 68 against 72 at 1024^2, but 92 against 86 on
// 14 x 32000.
//
// On grids of a few columns a tile is mostly idle lanes: a step takes 10.5 ns per
// tile however few cells it holds. The tall ones of them have one thread per
// cell instead (k_step_lo_cell), which resolves ghost cells per neighbour.
#include "lbm_device.h"
#include "lbm_internal.h"
#include "lbm_stage.h"
#include "lbm_step.h"
#include "lbm_tile.h"

namespace lbmd {

struct LoArgs {
    StepGrid s;
    double* __restrict__ ke_part;  // per 256-cell block (sum, max) or null
    Consts k;
};

// f_i at (x, y) with x or y (not both) possibly in the three ghost layers.
__device__ __forceinline__ double lo_value(const StepGrid& a, const Consts& k, int i, int x, int y)
{
    const int64_t n = (int64_t)a.nx * a.ny;
    if (x < 0 || x >= a.nx) {
        const bool lo = x < 0;
        const int m = lo ? -1 - x : x - a.nx;
        const int bc = a.bc[lo ? XLO : XHI];
        if (bc == PERIODIC) return a.fin[i * n + (int64_t)y * a.nx + wrap_index(x, a.nx)];
        if (bc == REFLECT)
            return a.fin[k.mirx[i] * n + (int64_t)y * a.nx + (lo ? m : a.nx - 1 - m)];
        if (bc == OUTFLOW) return (lo ? a.gb[XLO] : a.gb[XHI])[(int64_t)i * a.ny + y];
        return k.side_eq[lo ? XLO : XHI][i];
    }
    if (y < 0 || y >= a.ny) {
        const bool lo = y < 0;
        const int m = lo ? -1 - y : y - a.ny;
        const int bc = a.bc[lo ? YLO : YHI];
        if (bc == PERIODIC) return a.fin[i * n + (int64_t)wrap_index(y, a.ny) * a.nx + x];
        if (bc == REFLECT)
            return a.fin[k.miry[i] * n + (int64_t)(lo ? m : a.ny - 1 - m) * a.nx + x];
        if (bc == OUTFLOW) return (lo ? a.gb[YLO] : a.gb[YHI])[(int64_t)i * a.nx + x];
        return k.side_eq[lo ? YLO : YHI][i];
    }
    return a.fin[i * n + (int64_t)y * a.nx + x];
}

template <int SCHEME>
__device__ __forceinline__ double lo_face(double b, double c)
{
    return SCHEME == 1 ? c : __builtin_fma(0.5, c - b, c);
}

// h_{I+1/2} - h_{I-1/2} along one axis for velocity component v, from the
// samples F(-2..2) = v f at offsets -2..2 of the cell.
template <int SCHEME>
__device__ __forceinline__ double lo_diff(double v, const double (&F)[5])
{
    if (v >= 0.0) return lo_face<SCHEME>(F[1], F[2]) - lo_face<SCHEME>(F[0], F[1]);
    // mirror image: face I+1/2 from (F_{I+2}, F_{I+1}), face I-1/2 from (F_{I+1}, F_I)
    return lo_face<SCHEME>(F[4], F[3]) - lo_face<SCHEME>(F[3], F[2]);
}

template <int SCHEME>
__global__ __launch_bounds__(256) void k_step_lo_cell(LoArgs a)
{
    __shared__ double sr[8];
    const StepGrid& g = a.s;
    const Consts& k = a.k;
    const int64_t n = (int64_t)g.nx * g.ny;
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double e = 0.0;
    if (c < n) {
        const int y = (int)(c / g.nx), x = (int)(c - (int64_t)y * g.nx);
        double r = 0.0, jx = 0.0, jy = 0.0, E = 0.0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const double fi = g.fin[i * n + c];
            r += fi;
            jx = __builtin_fma(fi, k.vx[i], jx);
            jy = __builtin_fma(fi, k.vy[i], jy);
            E = __builtin_fma(fi, k.hv2[i], E);
        }
        const CellEq q = cell_eq_from_sums(r, jx, jy, E);
        const double un = (g.ke_axis ? jx : jy) / r;
        e = 0.5 * r * un * un;
        const double F1 = weight_c(k, 0, q.T), F2 = weight_c(k, 1, q.T), F3 = weight_c(k, 2, q.T);
        const double omct = 1.0 - g.ct;
        // rest particle: no convection
        const double f0 = g.fin[c];
        const double fe0 = q.rho * (1.0 - 6.0 * (F1 + F2 + F3)) * q.t0;
        g.fout[c] = __builtin_fma(-g.ct, f0 - fe0, f0);
        for (int i = 1; i < NV; ++i) {
            const double vx = k.vx[i], vy = k.vy[i];
            double Fx[5], Fy[5];
#pragma unroll
            for (int o = 0; o < 5; ++o) {
                Fx[o] = vx == 0.0 ? 0.0 : vx * lo_value(g, k, i, x - 2 + o, y);
                Fy[o] = vy == 0.0 ? 0.0 : vy * lo_value(g, k, i, x, y - 2 + o);
            }
            const double dhx = lo_diff<SCHEME>(vx, Fx);
            const double dhy = lo_diff<SCHEME>(vy, Fy);
            const double A = (g.ct * q.rho) * (i < 7 ? F1 : i < 13 ? F2 : F3);
            const double eta = __builtin_fma(vx, q.uxt, vy * q.uyt);
            double fn = __builtin_fma(omct, g.fin[i * n + c], A * feq_poly(eta, q.t0));
            fn = __builtin_fma(-g.cx, dhx, fn);
            fn = __builtin_fma(-g.cy, dhy, fn);
            g.fout[i * n + c] = fn;
        }
    }
    if (!a.ke_part) return;
    const double s = wave_sum(e), mx = wave_max(e);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sr[2 * w] = s;
        sr[2 * w + 1] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.ke_part[2 * blockIdx.x] = sr[0] + sr[2] + sr[4] + sr[6];
        a.ke_part[2 * blockIdx.x + 1] = fmax(fmax(sr[1], sr[3]), fmax(sr[5], sr[7]));
    }
}

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
    if (R == 0) {
        s.tiles_x = 0;
        const LoArgs a{s, ke_part, k};
        hipLaunchKernelGGL(scheme == 1 ? k_step_lo_cell<1> : k_step_lo_cell<2>,
                           dim3((unsigned)(((int64_t)nx * ny + 255) / 256)), dim3(256), 0, st, a);
        return hipGetLastError();
    }
    void (*const kernels[3][2])(TileArgs) = {{k_step_lo<1, 1>, k_step_lo<1, 2>},
                                             {k_step_lo<2, 1>, k_step_lo<2, 2>},
                                             {k_step_lo<4, 1>, k_step_lo<4, 2>}};
    return launch_tiles(kernels[R >> 1][scheme == 1 ? 0 : 1], tile_args(s, k, ke_part, R), R, st);
}

}  // namespace lbmd
