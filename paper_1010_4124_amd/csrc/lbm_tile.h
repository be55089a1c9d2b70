// lbm_tile.h -- one forward-Euler D2V19 FDLB step (Eq. (47) of
// arXiv:1010.4124) of one 64 x R tile by one workgroup of 12 wavefronts that
// holds all 18 moving planes of the tile at once: the device body of the
// whole-tile step variants (PH_TILE).
//
// Every plane is loaded once: the rows a velocity's y faces need go to
// registers, their R centre rows and the x halo to LDS. The moments of Eq. (10)
// are summed over the staged planes, so the step needs neither a pass over f
// that forms them first nor sums carried from step to step: 19 planes read
// (plus halo rows, found in L2) and 19 written, in one launch.
//
// Wave w takes one velocity with v_y != 0 (shell w / 4; the four directions
// off the x axis). Waves 0-5 take one velocity on the x axis as well (no y
// faces), waves 6 .. 5+R one row of cells: moments, equilibrium data, rest
// particle and energy. A workgroup's waves go to the four SIMDs of a CU in
// turn, so 12 waves of about equal work keep them level.
//
//   load     plane rows and the rest plane, all in flight at once
//   stage    centre rows and x halo to LDS                           | barrier
//   phase A  the cell rows; y and x faces of the wave's planes       | barrier
//   phase B  the x flux differences replace the planes in LDS to get from the
//            strips' lanes to the columns'; update, store
//
// Velocities are handled in a canonical frame: a plane with v_x < 0 is staged
// with its columns reversed, one with v_y < 0 with its rows reversed (each
// axis on its own), so that every velocity moves towards larger indices and
// one code path serves all 18; the reversal is in addresses and the sign of
// a flux difference in the Courant factor, so the arithmetic is exactly that
// of the M = 1 kernel, in its order (results equal to its bit for bit).
//
// What bounds it: on small grids the latency of one tile (launch, loads,
// faces, stores in sequence), hence the many waves and the low R; on large
// ones the phases of the two workgroups that fit a CU (LDS 53 KB and 24 waves
// at R = 4) overlap incompletely: VALU busy 62% of the time at 2048^2, with
// HBM traffic of 314 B per cell of the 304 it cannot do without (the
// fast-tile kernel: 416, but 78% of the issue slots used, 320 us against 390
// there). Measured per step, against the state pass and plane kernel it
// replaces: 400 x 4 7.5 us (12.6), 256^2 11.5 (17.0), 512^2 27.4 (37.0),
// 1101 x 605 67 (101), four outflow grids of 600 x 200 in a batch 59 (76).
#pragma once

#include "lbm_device.h"
#include "lbm_stage.h"
#include "lbm_step.h"

namespace lbmd {

// What the kernel needs of one speed shell, side by side: |v_x| of the
// directions off and on the x axis, |v_y|, |v|^2 / 2, the WENO regularisers
// eps / v^2 of the same three components, and the weight's coefficients.
struct TileShell {
    double vh, vk, vs, h2;
    double eh, ek, ey;
    double Fc4, Fbc, Fden, Frden;
    double pad;
};

struct TileConsts {
    TileShell s[3];
    double side_eq[4][NV];  // f^eq of each fixed-equilibrium side (single grid)
};

inline TileConsts tile_consts(const Consts& k)
{
    TileConsts t;
    for (int s = 0; s < 3; ++s) {
        const int h = 1 + 6 * s, x = 6 + 6 * s;  // directions pi/3 and 2 pi
        t.s[s] = TileShell{k.vx[h],  k.vx[x],  k.vy[h],   k.hv2[h],  k.epsx[h], k.epsx[x],
                           k.epsy[h], k.Fc4[s], k.Fbc[s], k.Fden[s], k.Frden[s], 0.0};
    }
    for (int q = 0; q < 4; ++q)
        for (int i = 0; i < NV; ++i) t.side_eq[q][i] = k.side_eq[q][i];
    return t;
}

// weight_c of a shell
__device__ __forceinline__ double weight_t(const TileShell& k, double T)
{
    const double P = T * __builtin_fma(T, __builtin_fma(T, 24.0, -k.Fc4), k.Fbc);
    const double q = P * k.Frden;
    return __builtin_fma(__builtin_fma(-k.Fden, q, P), k.Frden, q);
}

constexpr int TILE_WAVES = 12;
template <int R>
struct TileWg {
    static constexpr int PL = R * PITCH;        // one staged plane, later its x flux differences
    static constexpr int ST = 18 * PL;          // cell state [6][R][64]
    static constexpr int KE = ST + 6 * R * 64;  // energy partials of the cell rows
    static constexpr int LDS = KE + 2 * R;
    static_assert(R <= 4, "one cell row for each of the waves 6 .. 9 at most");
    static_assert(5 * R <= 64, "the x halo of a plane must fit one 64-lane load");
    static_assert(XPITCH <= PITCH, "the x flux differences must fit the staged plane");
};

// A plane's rows through raw buffer accesses: the row goes in the scalar
// offset (always inside the descriptor's range), the lane's column in the
// vector offset, and a lane that must not touch memory gets a vector offset
// beyond the range (such a read gives 0, such a write is dropped). Fast tiles
// have one descriptor per plane, over the tile's rows, whose offsets stay below
// 2^31 on grids up to TILE_MAX_NX cells wide; boundary tiles, and every tile of
// a wider grid, one per row, over the tile's columns.
constexpr int TILE_MAX_NX = 1 << 24;
constexpr unsigned TILE_SKIP = 0x80000000u;

__device__ __forceinline__ unsigned uniform(int v)
{
    return (unsigned)__builtin_amdgcn_readfirstlane(v);
}
// (p and bytes are the same for all lanes; saying so keeps the compiler, which
// may hold them in vector registers, from looping over their values)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const double* p, int bytes)
{
    const unsigned long long u = (unsigned long long)p;
    const unsigned lo = uniform((int)(unsigned)u), hi = uniform((int)(unsigned)(u >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)((unsigned long long)hi << 32 | lo), 0,
                                             (int)uniform(bytes), 0x00020000);
}
__device__ __forceinline__ double row_load(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
}
template <bool NT>
__device__ __forceinline__ void row_store(double x, __amdgpu_buffer_rsrc_t r, unsigned v,
                                          unsigned s)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, x), r, v, s, NT ? 2 : 0);
}

// The lane, opaque to the compiler: the addresses derived from it are then
// formed where they are used, instead of all being kept in registers around
// the loop over tiles.
__device__ __forceinline__ int tile_lane()
{
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    return l;
}

// The velocities and the cell row of a wave.
struct TileWave {
    int sy, iy, sn, in, m;  // shells and planes off and on the x axis, cell row
    bool ynegx, negy, hasn, nnegx;
};

__device__ __forceinline__ TileWave tile_wave(int wave)
{
    TileWave v;
    const int t = wave & 3;  // directions 0, 1, 3, 4
    v.sy = wave >> 2;
    v.ynegx = t == 1 || t == 2;
    v.negy = t >= 2;
    v.iy = 1 + 6 * v.sy + t + (v.negy ? 1 : 0);
    v.hasn = wave < 6;
    v.sn = v.hasn ? wave >> 1 : 0;
    v.nnegx = (wave & 1) == 0;  // directions 2 and 5
    v.in = 1 + 6 * v.sn + (v.nnegx ? 2 : 5);
    v.m = wave - 6;
    return v;
}

// Halo lanes (lane < 5 R): row lane / 5 (canonical) and one of five columns,
// counted from the tile's first cell: -3, -2, -1, w, w+1 for v_x > 0 (the
// reach of its upwind stencils), the mirrored w+2, w+1, w, -1, -2 for v_x < 0.
__device__ __forceinline__ int halo_col(int hq, bool negx, int w)
{
    const int c = hq < 3 ? hq - 3 : w + hq - 3;
    return negx ? w - 1 - c : c;
}

// What a wave loads of a tile.
template <int R>
struct TileRegs {
    double p[R + 5], h;  // velocity off the axis: canonical rows, halo value
    double pn[R], hn;    // velocity on it
    double f0;           // rest plane, the wave's cell row
};

// Request the wave's rows of tile g (FAST: a fast tile). Canonical row j of the
// velocity off the axis is row y0-3 + j, or y0+R+2 - j for v_y < 0; cell row m
// is j = m + 3.
template <int R, bool FAST, class Grid>
__device__ __forceinline__ void tile_load(const Grid& g, const TileConsts& k, const TileWave& v,
                                          int lane, TileRegs<R>& L)
{
    const int x0 = g.x0, y0 = g.y0;
    constexpr int ROWS = R + 5;
    const int nx = g.nx(), ny = g.ny(), rb = 8 * nx;
    const int64_t plane = (int64_t)nx * ny;
    const double* fin = g.fin();
    const int w = FAST ? 64 : min(64, nx - x0);
    const unsigned l8 = 8u * (unsigned)lane, vx8 = l8 + 8u * (unsigned)x0;  // (vx8: fast tiles)
    const bool hl = lane < 5 * R;
    const int hr = lane / 5, hq = lane - 5 * hr;
    const int yhx = x0 + halo_col(hq, v.ynegx, w), nhx = x0 + halo_col(hq, v.nnegx, w);
    const int yhm = v.negy ? R - 1 - hr : hr;
    const bool hasm = v.m >= 0 && v.m < R;
    if constexpr (FAST) {
        const __amdgpu_buffer_rsrc_t ry =
            rows_rsrc(fin + v.iy * plane + (int64_t)(y0 - HALO) * nx, (R + 2 * HALO) * rb);
        const int s0 = v.negy ? (R + 5) * rb : 0, sd = v.negy ? -rb : rb;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) L.p[j] = row_load(ry, vx8, uniform(s0 + j * sd));
        L.h = row_load(ry, hl ? (unsigned)((yhm + HALO) * rb + 8 * wrap_once(yhx, nx)) : TILE_SKIP,
                       0);
        if (v.hasn) {
            const __amdgpu_buffer_rsrc_t rn =
                rows_rsrc(fin + v.in * plane + (int64_t)y0 * nx, R * rb);
            L.hn = row_load(rn, hl ? (unsigned)(hr * rb + 8 * wrap_once(nhx, nx)) : TILE_SKIP, 0);
#pragma unroll
            for (int j = 0; j < R; ++j) L.pn[j] = row_load(rn, vx8, uniform(j * rb));
        }
    } else {
        const GridBC b = g.bc();
        // mirror partners of directions 0, 1, 3, 4: (1, 0, 4, 3) and (4, 3, 1, 0)
        const int s6 = 1 + 6 * v.sy, d = v.iy - s6;
        const int ix = s6 + (d == 0 ? 1 : d == 1 ? 0 : d == 3 ? 4 : 3), im = s6 + 4 - d;
        // a row's source is the same for all lanes
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const RowDesc rd = row_desc_g<false>(b, v.negy ? y0 + R + 2 - j : y0 - HALO + j);
            const double* src = fin + (rd.mode == RM_MIRY ? im : v.iy) * plane +
                                (int64_t)rd.src * nx;
            if (rd.mode == RM_OUT)
                src = (rd.side == YLO ? b.gb[YLO] : b.gb[YHI]) + (int64_t)v.iy * nx;
            const bool ld = rd.mode != RM_CONST && rd.mode != RM_NONE;
            L.p[j] = row_load(rows_rsrc(src + x0, ld ? 8 * w : 0), l8, 0);
        }
        // halo values of the rows inside the domain
        auto halo = [&](int i, int imx, int hx, int hy) {
            int col = 0, kind = CK_NONE;
            if (hl && hy < ny) x_source_g<false>(b, hx, col, kind);
            const bool out = kind == CK_OUTLO || kind == CK_OUTHI;
            const int64_t off = out ? (int64_t)i * ny + hy
                                    : (kind == CK_MIRX ? imx : i) * plane + (int64_t)hy * nx + col;
            const double* base = kind == CK_OUTLO ? b.gb[XLO] : kind == CK_OUTHI ? b.gb[XHI] : fin;
            const bool ld = kind == CK_NORM || kind == CK_MIRX || out;
            const double x = base[ld ? off : 0];
            const double c = kind == CK_CXLO ? g.side_eq(k, XLO, i) : g.side_eq(k, XHI, i);
            return ld ? x : kind == CK_NONE ? 0.0 : c;
        };
        L.h = halo(v.iy, ix, yhx, y0 + yhm);
        if (v.hasn) {
#pragma unroll
            for (int j = 0; j < R; ++j)
                L.pn[j] = row_load(
                    rows_rsrc(fin + v.in * plane + (int64_t)min(y0 + j, ny - 1) * nx + x0, 8 * w),
                    l8, 0);
            L.hn = halo(v.in, 1 + 6 * v.sn + (v.nnegx ? 5 : 2), nhx, y0 + hr);
        }
        // rows of a fixed-equilibrium side
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const RowDesc rd = row_desc_g<false>(b, v.negy ? y0 + R + 2 - j : y0 - HALO + j);
            if (rd.mode == RM_CONST) L.p[j] = g.side_eq(k, rd.side, v.iy);
        }
    }
    if (hasm)
        L.f0 = row_load(rows_rsrc(fin + (int64_t)(y0 + v.m) * nx + x0,
                                  FAST || y0 + v.m < ny ? 8 * w : 0), l8, 0);
}

// Flux differences of f along a strip of R cells from its upwind-ordered
// samples P (P[m+3] is cell m): WENO5, or the upwind schemes, whose face
// downstream of a cell c with upstream neighbour b takes c (first order) or
// c + (c - b) / 2 (second order).
template <int R, int SCHEME>
__device__ __forceinline__ void strip_diff(const double (&P)[R + 5], double eps, double (&dh)[R])
{
    if constexpr (SCHEME == 0) {
        weno_strip<R, false>(P, eps, [&](int m, double d) { dh[m] = d; });
    } else {
        auto face = [&](int j) {
            return SCHEME == 1 ? P[j + 2] : __builtin_fma(0.5, P[j + 2] - P[j + 1], P[j + 2]);
        };
        double hp = face(0);
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const double h = face(m + 1);
            dh[m] = h - hp;
            hp = h;
        }
    }
}

// Tile g (FAST: a fast tile) by one workgroup. g is a Grid (the accessors used
// below) with the tile's origin x0, y0 and its energy partial ke (null: none
// wanted). lds holds TileWg<R>::LDS doubles.
// SCHEME: the convection flux (lbm_params.scheme).
template <int R, bool NT, bool FAST, int SCHEME, class Grid>
__device__ __forceinline__ void tile_step(const Grid& g, const TileConsts& k, double* lds)
{
    using S = TileWg<R>;
    constexpr int ROWS = R + 5;
    const TileWave v = tile_wave(__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)));
    const bool hasm = v.m >= 0 && v.m < R;
    const TileShell& ky = k.s[v.sy];
    const TileShell& kn = k.s[v.sn];
    double* const s_y = lds + (v.iy - 1) * S::PL;
    double* const s_n = lds + (v.in - 1) * S::PL;
    double* const st = lds + S::ST;

    TileRegs<R> L;
    tile_load<R, FAST>(g, k, v, tile_lane(), L);
    // the constants' lines into the scalar cache while the planes are on their way
    asm volatile("" ::"s"(k.s[0].vh), "s"(k.s[0].Fbc), "s"(k.s[1].ek), "s"(k.s[2].vh),
                 "s"(k.s[2].Fc4));
    int lane = tile_lane();
    const int nx = g.nx(), ny = g.ny(), rb = 8 * nx;
    const int64_t plane = (int64_t)nx * ny;
    const int y0 = g.y0, wd = FAST ? 64 : min(64, nx - g.x0);
    // ---- stage
    if (FAST || lane < wd) {
        const int ylc = v.ynegx ? 63 - lane : lane, nlc = v.nnegx ? 63 - lane : lane;
#pragma unroll
        for (int j = 0; j < R; ++j) s_y[j * PITCH + HALO + ylc] = L.p[j + HALO];
        if (v.hasn) {
#pragma unroll
            for (int j = 0; j < R; ++j) s_n[j * PITCH + HALO + nlc] = L.pn[j];
        }
    }
    if (lane < 5 * R) {
        const int hr = lane / 5, hq = lane - 5 * hr;
        const int cy = halo_col(hq, v.ynegx, wd), cn = halo_col(hq, v.nnegx, wd);
        s_y[hr * PITCH + HALO + (v.ynegx ? 63 - cy : cy)] = L.h;
        if (v.hasn) s_n[hr * PITCH + HALO + (v.nnegx ? 63 - cn : cn)] = L.hn;
    }
    __syncthreads();

    // ---- phase A
    if (hasm) {
        const int m = v.m;
        lane = tile_lane();
        const bool inx = FAST || lane < wd, act = FAST || (inx && y0 + m < ny);
        const double f0 = L.f0;
        // the sums of k_sums, in its order
        double r = 0.0, jx = 0.0, jy = 0.0, E = 0.0;
        r += f0;
        jx = __builtin_fma(f0, 0.0, jx);
        jy = __builtin_fma(f0, 0.0, jy);
        E = __builtin_fma(f0, 0.0, E);
#pragma unroll
        for (int i = 1; i < NV; ++i) {
            const int d = (i - 1) % 6;
            const TileShell& s = k.s[(i - 1) / 6];
            const bool nx_ = dir_cos(d) < 0.0;
            const int row = dir_sin_sign(d) < 0 ? R - 1 - m : m;
            const double fi =
                lds[(i - 1) * S::PL + row * PITCH + HALO + (nx_ ? 63 - lane : lane)];
            const double vx = d == 2 || d == 5 ? s.vk : s.vh;
            r += fi;
            jx = __builtin_fma(fi, nx_ ? -vx : vx, jx);
            jy = __builtin_fma(
                fi, dir_sin_sign(d) > 0 ? s.vs : dir_sin_sign(d) < 0 ? -s.vs : 0.0, jy);
            E = __builtin_fma(fi, s.h2, E);
        }
        if (!act) {  // idle lanes: unit state
            r = E = 1.0;
            jx = jy = 0.0;
        }
        const CellEq c = cell_eq_from_sums(r, jx, jy, E);
        const double ct = g.ct(), rho = ct * c.rho;
        const double F1 = weight_t(k.s[0], c.T), F2 = weight_t(k.s[1], c.T),
                     F3 = weight_t(k.s[2], c.T);
        double* sc = st + m * 64 + lane;
        sc[0 * R * 64] = rho * F1;
        sc[1 * R * 64] = rho * F2;
        sc[2 * R * 64] = rho * F3;
        sc[3 * R * 64] = c.uxt;
        sc[4 * R * 64] = c.uyt;
        sc[5 * R * 64] =
            __builtin_fma(-0.5 * c.T, __builtin_fma(c.uxt, c.uxt, c.uyt * c.uyt), 1.0);
        // rest particle: no convection, f^eq_0 = rho F_0 (1 - u^2/2T)
        const double F0 = 1.0 - 6.0 * (F1 + F2 + F3);
        const double fe = c.rho * F0 * c.t0;
        row_store<false>(__builtin_fma(-ct, f0 - fe, f0),
                         rows_rsrc(g.fout() + (int64_t)(y0 + m) * nx + g.x0,
                                   FAST || y0 + m < ny ? 8 * wd : 0), 8u * (unsigned)lane, 0);
        if (g.ke) {
            const double un = (g.ke_axis() ? jx : jy) / r;
            const double e = act ? 0.5 * r * un * un : 0.0;
            const double ke_s = wave_sum(e), ke_m = wave_max(e);
            if (lane == 0) {
                lds[S::KE + 2 * m] = ke_s;
                lds[S::KE + 2 * m + 1] = ke_m;
            }
        }
    }
    lane = tile_lane();
    const int xr = lane % R, xs = lane / R;  // x strips: row, strip of R cells (x_pass)
    // The faces, one strip after the other: each result is pinned where it
    // is computed, as the compiler would otherwise interleave the strips
    // (and spill) or move them past the barrier, behind the cell rows.
    double dhx[R], dhy[R], dhn[R];
    auto pin = [](double(&x)[R]) {
#pragma unroll
        for (int q = 0; q < R; ++q) asm volatile("" : "+v"(x[q]));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto x_strip = [&](const double* s_pl, double eps, double(&dh)[R]) {
        double P[ROWS];
        const double* b = s_pl + xr * PITCH + xs * R;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) P[j] = b[j];
        strip_diff<R, SCHEME>(P, eps, dh);
        pin(dh);
    };
    strip_diff<R, SCHEME>(L.p, ky.ey, dhy);
    pin(dhy);
    x_strip(s_y, ky.eh, dhx);
    if (v.hasn) x_strip(s_n, kn.ek, dhn);
    __syncthreads();
    if (g.ke && threadIdx.x == 0) {
        double s = lds[S::KE], mx = lds[S::KE + 1];
#pragma unroll
        for (int j = 1; j < R; ++j) {
            s += lds[S::KE + 2 * j];
            mx = fmax(mx, lds[S::KE + 2 * j + 1]);
        }
        g.ke[0] = s;
        g.ke[1] = mx;
    }

    // ---- phase B: the cells' values, left to the staged planes so far,
    // then the x flux differences in their place
    double fy[R], fn_[R];
    lane = tile_lane();
    const int ylc = v.ynegx ? 63 - lane : lane, nlc = v.nnegx ? 63 - lane : lane;
#pragma unroll
    for (int j = 0; j < R; ++j) fy[j] = s_y[j * PITCH + HALO + ylc];
    if (v.hasn) {
#pragma unroll
        for (int j = 0; j < R; ++j) fn_[j] = s_n[j * PITCH + HALO + nlc];
    }
    plane_sync<2>();
#pragma unroll
    for (int q = 0; q < R; ++q) s_y[(lane % R) * XPITCH + lane / R * R + q] = dhx[q];
    if (v.hasn) {
#pragma unroll
        for (int q = 0; q < R; ++q) s_n[(lane % R) * XPITCH + lane / R * R + q] = dhn[q];
    }
    plane_sync<2>();
    const double omct = 1.0 - g.ct();
    // f' of plane i in the lane's column of row m of the tile
    auto put = [&](int i, int m, double x) {
        double* row = g.fout() + i * plane + (int64_t)y0 * nx + g.x0;
        if constexpr (FAST)
            row_store<NT>(x, rows_rsrc(row, R * rb), 8u * (unsigned)lane, uniform(m * rb));
        else
            row_store<NT>(x, rows_rsrc(row + (int64_t)m * nx, y0 + m < ny ? 8 * wd : 0),
                          8u * (unsigned)lane, 0);
    };
    {
        const double vx = v.ynegx ? -ky.vh : ky.vh, vy = v.negy ? -ky.vs : ky.vs;
        const double ncx = -(g.cx() * ky.vh), ncy = -(g.cy() * ky.vs);
#pragma unroll
        for (int mc = 0; mc < R; ++mc) {
            const int mr = v.negy ? R - 1 - mc : mc;
            const double* sc = st + mr * 64 + lane;
            const double eta = __builtin_fma(vx, sc[3 * R * 64], vy * sc[4 * R * 64]);
            double fn = __builtin_fma(omct, fy[mc],
                                      sc[v.sy * R * 64] * feq_poly(eta, sc[5 * R * 64]));
            fn = __builtin_fma(ncx, s_y[mc * XPITCH + ylc], fn);
            fn = __builtin_fma(ncy, dhy[mc], fn);
            put(v.iy, mr, fn);
        }
    }
    if (v.hasn) {
        const double vx = v.nnegx ? -kn.vk : kn.vk, ncx = -(g.cx() * kn.vk);
#pragma unroll
        for (int mc = 0; mc < R; ++mc) {
            const double* sc = st + mc * 64 + lane;
            // v_y = 0: eta = fma(v_x, u_x/T, 0 u_y/T)
            const double eta = __builtin_fma(vx, sc[3 * R * 64], 0.0 * sc[4 * R * 64]);
            double fn = __builtin_fma(omct, fn_[mc],
                                      sc[v.sn * R * 64] * feq_poly(eta, sc[5 * R * 64]));
            fn = __builtin_fma(ncx, s_n[mc * XPITCH + nlc], fn);
            put(v.in, mc, fn);
        }
    }
}

// Tile g of either kind.
template <int R, bool NT, int SCHEME, class Grid>
__device__ __forceinline__ void tile_any(const Grid& g, const TileConsts& k, double* lds)
{
    if (g.nx() <= TILE_MAX_NX && fast_tile(g.bc(), g.x0, g.y0, TX, R, HALO))
        tile_step<R, NT, true, SCHEME>(g, k, lds);
    else
        tile_step<R, NT, false, SCHEME>(g, k, lds);
}

// A launch over one grid: one workgroup per tile, XCD-major over the strip walk
// as in k_step.
struct TileArgs {
    StepGrid s;
    double* __restrict__ ke_part;  // [ntiles][2] or null
    int tiles_y, nwork, per_xcd;
    TileConsts k;
};

// One tile of the grid, as tile_step sees it.
struct TileOfGrid {
    const TileArgs& a;
    int x0, y0;
    double* ke;
    __device__ int nx() const { return a.s.nx; }
    __device__ int ny() const { return a.s.ny; }
    __device__ const double* fin() const { return a.s.fin; }
    __device__ double* fout() const { return a.s.fout; }
    __device__ double cx() const { return a.s.cx; }
    __device__ double cy() const { return a.s.cy; }
    __device__ double ct() const { return a.s.ct; }
    __device__ int ke_axis() const { return a.s.ke_axis; }
    __device__ GridBC bc() const { return grid_bc(a.s); }
    __device__ double side_eq(const TileConsts& k, int side, int i) const
    {
        return k.side_eq[side][i];
    }
};

inline TileArgs tile_args(const StepGrid& s, const Consts& k, double* ke_part, int R)
{
    TileArgs t;
    t.s = s;
    t.s.tiles_x = (s.nx + TX - 1) / TX;
    t.ke_part = ke_part;
    t.tiles_y = (s.ny + R - 1) / R;
    t.nwork = t.s.tiles_x * t.tiles_y;
    t.per_xcd = (t.nwork + 7) / 8;
    t.k = tile_consts(k);
    return t;
}

// Workgroup blockIdx.x of such a launch.
template <int R, bool NT, int SCHEME>
__device__ __forceinline__ void tile_block(const TileArgs& a, double* lds)
{
    const int b = blockIdx.x;
    const int work = (b & 7) * a.per_xcd + (b >> 3);
    if (work >= a.nwork) return;
    const TileXY t = strip_walk_xy(work, a.s.tiles_x, a.tiles_y);
    tile_any<R, NT, SCHEME>(
        TileOfGrid{a, t.tx * TX, t.ty * R,
                   a.ke_part ? a.ke_part + 2 * (t.ty * a.s.tiles_x + t.tx) : nullptr}, a.k, lds);
}

}  // namespace lbmd
