// lbm_tile.h -- one forward-Euler D2V19 FDLB step (Eq. (47) of
// arXiv:1010.4124) of one 64 x R tile by one workgroup of 12 (R = 4: 8)
// wavefronts that holds all 18 moving planes of the tile at once: the device
// body of the whole-tile step variants (PH_TILE).
//
// Every plane is loaded once: the rows a velocity's y faces need go to
// registers, their R centre rows and the x halo to LDS. The moments of Eq. (10)
// are summed over the staged planes, so the step needs neither a pass over f
// that forms them first nor sums carried from step to step: 19 planes read
// (plus halo rows, found in L2) and 19 written, in one launch.
//
// With 12 waves, wave w takes one velocity with v_y != 0 (shell w / 4; the four
// directions off the x axis). Waves 0-5 take one velocity on the x axis as well (no y
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
// ones the phases of the workgroups that fit a CU overlap incompletely: with
// the three of tile8_step (R = 4) VALU issues 63 to 68% of the time at 2048^2, with
// HBM traffic of 313 B per cell of the 304 it cannot do without (the fast-tile
// kernel: 60% and 399). Measured per step, against the state pass and plane kernel it
// replaces: 400 x 4 6.1 us (12.6), 256^2 10.4 (17.0), 512^2 25.2 (37.0),
// 1101 x 605 60 (101), four outflow grids of 600 x 200 in a batch 54 (76).
#pragma once

#include "lbm_device.h"
#include "lbm_internal.h"
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
// wavefronts of a tile's workgroup (tile_step, tile8_step)
constexpr int tile_waves(int R) { return R == 4 ? 8 : TILE_WAVES; }
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

// v around a periodic axis of n, without the division of x_source_g and
// row_desc_g where the tile and its halo reach less than a period beyond it.
__device__ __forceinline__ int wrap_near(int v, int n, int lo, int hi)
{
    return lo == PERIODIC && hi == PERIODIC && n >= 12 ? wrap_once(v, n) : v;
}

// Sources of the rows of one plane of a boundary tile, row j in lane j: one
// evaluation of row_desc_g for all of them (row by row, with all lanes alike,
// these were most of the instructions of such a tile, which took 4 times the
// others' time: 400 x 4 6.9 us per step, 6.1 so; 1101 x 605 66.6 and 60.4).
struct RowSources {
    unsigned long long at;     // address of the row's first column in the tile
    int bytes;                 // its length, 0: reads as zero
    unsigned long long fixed;  // rows of a fixed-equilibrium side (all lanes)
    __device__ __forceinline__ double load(int j, unsigned v) const
    {
        const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)at, j);
        const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(at >> 32), j);
        return row_load(rows_rsrc((const double*)((unsigned long long)hi << 32 | lo),
                                  __builtin_amdgcn_readlane(bytes, j)), v, 0);
    }
};
// Plane i of the grid b's field (im: its mirror partner in y), w columns from
// x0, rows row(0 .. n-1); ZG: zero outside the domain.
template <bool ZG, class Row>
__device__ __forceinline__ RowSources row_sources(const GridBC& b, const double* field, int i,
                                                  int im, int x0, int w, Row&& row, int n, int lane)
{
    const int64_t plane = (int64_t)b.nx * b.ny;
    const int y = row(min(lane, n - 1));
    const RowDesc rd = row_desc_g<ZG>(b, wrap_near(y, b.ny, b.bc[YLO], b.bc[YHI]));
    const double* src = rd.mode == RM_OUT
                            ? (rd.side == YLO ? b.gb[YLO] : b.gb[YHI]) + (int64_t)i * b.nx
                            : field + (rd.mode == RM_MIRY ? im : i) * plane + (int64_t)rd.src * b.nx;
    return RowSources{(unsigned long long)(src + x0),
                      rd.mode == RM_CONST || rd.mode == RM_NONE ? 0 : 8 * w,
                      __ballot(lane < n && rd.mode == RM_CONST)};
}

// Halo lanes (lane < 5 R): row lane / 5 (canonical) and one of five columns,
// counted from the tile's first cell: -3, -2, -1, w, w+1 for v_x > 0 (the
// reach of its upwind stencils), the mirrored w+2, w+1, w, -1, -2 for v_x < 0.
__device__ __forceinline__ int halo_col(int hq, bool negx, int w)
{
    const int c = hq < 3 ? hq - 3 : w + hq - 3;
    return negx ? w - 1 - c : c;
}

// One moving velocity: its plane, shell and sense on each axis (hasy: v_y != 0).
struct TileVel {
    int i, s;
    bool negx, negy, hasy;
};
// direction t of {0, 1, 3, 4} of shell s; velocity j of the six on the x axis
__device__ __forceinline__ TileVel vel_y(int s, int t)
{
    return TileVel{1 + 6 * s + t + (t >= 2 ? 1 : 0), s, t == 1 || t == 2, t >= 2, true};
}
__device__ __forceinline__ TileVel vel_x(int j)
{
    const bool neg = (j & 1) == 0;  // directions 2 and 5
    return TileVel{1 + 6 * (j >> 1) + (neg ? 2 : 5), j >> 1, neg, false, false};
}

// Request a velocity's rows p and halo value h of tile g (FAST: a fast tile).
// Canonical row j is row y0-3 + j, or y0+R+2 - j for v_y < 0; cell row m is
// j = m + 3. Without y faces only the R cell rows are read.
template <int R, bool FAST, class Grid>
__device__ __forceinline__ void vel_load(const Grid& g, const TileConsts& k, const TileVel& v,
                                         int lane, double (&p)[R + 5], double& h)
{
    const int x0 = g.x0, y0 = g.y0;
    constexpr int ROWS = R + 5;
    const int nx = g.nx(), ny = g.ny(), rb = 8 * nx;
    const int64_t plane = (int64_t)nx * ny;
    const double* fin = g.fin();
    const int w = FAST ? 64 : min(64, nx - x0);
    const unsigned l8 = 8u * (unsigned)lane, vx8 = l8 + 8u * (unsigned)x0;
    const bool hl = lane < 5 * R;
    const int hr = lane / 5, hq = lane - 5 * hr;
    const int hx = x0 + halo_col(hq, v.negx, w), hm = v.negy ? R - 1 - hr : hr;
    if constexpr (FAST) {
        const __amdgpu_buffer_rsrc_t ry =
            rows_rsrc(fin + v.i * plane + (int64_t)(y0 - HALO) * nx, (R + 2 * HALO) * rb);
        const int s0 = v.negy ? (R + 5) * rb : 0, sd = v.negy ? -rb : rb;
        if (v.hasy) {
#pragma unroll
            for (int j = 0; j < ROWS; ++j) p[j] = row_load(ry, vx8, uniform(s0 + j * sd));
        } else {
#pragma unroll
            for (int j = HALO; j < HALO + R; ++j) p[j] = row_load(ry, vx8, uniform(s0 + j * sd));
        }
        h = row_load(ry, hl ? (unsigned)((hm + HALO) * rb + 8 * wrap_once(hx, nx)) : TILE_SKIP, 0);
    } else {
        const GridBC b = g.bc();
        const int s6 = 1 + 6 * v.s, d = v.i - s6;
        // mirror partners: directions 0 .. 5 in x (1, 0, 5, 4, 3, 2); in y (4, 3, -, 1, 0, -)
        const int ix = s6 + (d == 0 ? 1 : d == 1 ? 0 : d == 2 ? 5 : d == 3 ? 4 : d == 4 ? 3 : 2);
        const int im = s6 + 4 - d;
        // halo values of the rows inside the domain
        int col = 0, kind = CK_NONE;
        const int hy = y0 + hm;
        if (hl && hy < ny) x_source_g<false>(b, wrap_near(hx, nx, b.bc[XLO], b.bc[XHI]), col, kind);
        const bool out = kind == CK_OUTLO || kind == CK_OUTHI;
        const int64_t off = out ? (int64_t)v.i * ny + hy
                                : (kind == CK_MIRX ? ix : v.i) * plane + (int64_t)hy * nx + col;
        const double* base = kind == CK_OUTLO ? b.gb[XLO] : kind == CK_OUTHI ? b.gb[XHI] : fin;
        const bool ld = kind == CK_NORM || kind == CK_MIRX || out;
        const double x = base[ld ? off : 0];
        const double c = kind == CK_CXLO ? g.side_eq(k, XLO, v.i) : g.side_eq(k, XHI, v.i);
        h = ld ? x : kind == CK_NONE ? 0.0 : c;
        if (v.hasy) {
            const RowSources rs = row_sources<false>(b, fin, v.i, im, x0, w, [&](int j) {
                return v.negy ? y0 + R + 2 - j : y0 - HALO + j;
            }, ROWS, lane);
#pragma unroll
            for (int j = 0; j < ROWS; ++j) p[j] = rs.load(j, l8);
            if (rs.fixed) {  // rows of a fixed-equilibrium side
#pragma unroll
                for (int j = 0; j < ROWS; ++j) {
                    const bool low = (v.negy ? y0 + R + 2 - j : y0 - HALO + j) < 0;
                    if (rs.fixed >> j & 1)
                        p[j] = low ? g.side_eq(k, YLO, v.i) : g.side_eq(k, YHI, v.i);
                }
            }
        } else {
#pragma unroll
            for (int j = HALO; j < HALO + R; ++j)
                p[j] = row_load(rows_rsrc(fin + v.i * plane +
                                              (int64_t)min(y0 + j - HALO, ny - 1) * nx + x0, 8 * w),
                                l8, 0);
        }
    }
}

// A velocity's R centre rows and x halo into its plane in LDS (w columns).
template <int R, bool FAST>
__device__ __forceinline__ void vel_stage(const TileVel& v, int w, int lane,
                                          const double (&p)[R + 5], double h, double* lds)
{
    double* s = lds + (v.i - 1) * TileWg<R>::PL + HALO;
    if (FAST || lane < w) {
        const int c = v.negx ? 63 - lane : lane;
#pragma unroll
        for (int j = 0; j < R; ++j) s[j * PITCH + c] = p[j + HALO];
    }
    if (lane < 5 * R) {
        const int hr = lane / 5, hq = lane - 5 * hr;
        const int c = halo_col(hq, v.negx, w);
        s[hr * PITCH + (v.negx ? 63 - c : c)] = h;
    }
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

// The rest plane in the wave's cell row m.
template <bool FAST, class Grid>
__device__ __forceinline__ double rest_load(const Grid& g, int m, int w, int lane)
{
    const int nx = g.nx();
    return row_load(rows_rsrc(g.fin() + (int64_t)(g.y0 + m) * nx + g.x0,
                              FAST || g.y0 + m < g.ny() ? 8 * w : 0), 8u * (unsigned)lane, 0);
}

// The constants' lines into the scalar cache, while the planes are on their way.
__device__ __forceinline__ void warm_consts(const TileConsts& k)
{
    asm volatile("" ::"s"(k.s[0].vh), "s"(k.s[0].Fbc), "s"(k.s[1].ek), "s"(k.s[2].vh),
                 "s"(k.s[2].Fc4));
}

// Cell row m of the staged tile: moments, equilibrium data for the update,
// rest particle, energy partial.
template <int R, bool FAST, class Grid>
__device__ __forceinline__ void tile_cells(const Grid& g, const TileConsts& k, int m, int wd,
                                           double f0, double* lds)
{
    using S = TileWg<R>;
    double* const st = lds + S::ST;
    const int lane = tile_lane(), nx = g.nx(), ny = g.ny(), y0 = g.y0;
    const bool inx = FAST || lane < wd, act = FAST || (inx && y0 + m < ny);
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

// The tile's energy partial from those of its cell rows.
template <int R, class Grid>
__device__ __forceinline__ void tile_energy(const Grid& g, const double* lds)
{
    using S = TileWg<R>;
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

    const TileVel vy{v.iy, v.sy, v.ynegx, v.negy, true}, vn{v.in, v.sn, v.nnegx, false, false};
    double p[ROWS], f0 = 0.0;
    int lane = tile_lane();
    const int nx = g.nx(), ny = g.ny(), rb = 8 * nx;
    const int64_t plane = (int64_t)nx * ny;
    const int y0 = g.y0, wd = FAST ? 64 : min(64, nx - g.x0);
    {
        double h, pn[ROWS], hn;
        vel_load<R, FAST>(g, k, vy, lane, p, h);
        if (v.hasn) vel_load<R, FAST>(g, k, vn, lane, pn, hn);
        if (hasm) f0 = rest_load<FAST>(g, v.m, wd, lane);
        warm_consts(k);
        lane = tile_lane();
        vel_stage<R, FAST>(vy, wd, lane, p, h, lds);
        if (v.hasn) vel_stage<R, FAST>(vn, wd, lane, pn, hn, lds);
    }
    __syncthreads();

    // ---- phase A
    if (hasm) tile_cells<R, FAST>(g, k, v.m, wd, f0, lds);
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
    strip_diff<R, SCHEME>(p, ky.ey, dhy);
    pin(dhy);
    x_strip(s_y, ky.eh, dhx);
    if (v.hasn) x_strip(s_n, kn.ek, dhn);
    __syncthreads();
    tile_energy<R>(g, lds);

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

// The same by 8 wavefronts, for R = 4. Three such workgroups fit a CU (3 x 53 KB
// of LDS, 24 waves at 80 registers) where 12 waves let two: one more tile's
// loads and stores behind the others' faces. Waves 0-3 take two velocities off
// the x axis, waves 4-7 one, one or two on it and a cell row; both kinds have
// three plane loads, and a wave of each kind shares a SIMD. The x faces come
// after the second barrier, one velocity at a time, to stay within 80
// registers. Per step against 12 waves: 512^2 25.9 us (27.1), 1101 x 605 62.4
// (66.4), 1024^2 86 (100), 1448^2 175 (196), 2048^2 309 (358), a
// batch of 1.45 M cells 167 (180); below one round, where only a tile's latency
// counts, 600 x 200 24.1-24.7 (24.3).
// Raised wave priority around the loads gives 6% at 1101 x 605 (66.2 to 62.4)
// and 5% on four grids of 600 x 200, but costs as much on the states beyond the
// cache (2048^2 309 to 325), which are the ones stored non-temporally.
// Workgroups that stay and loop over tiles: 348 at 2048^2 (the next tile's loads
// wait behind the last one's stores, as both are counted in order).
template <int R, bool NT, bool FAST, int SCHEME, class Grid>
__device__ __forceinline__ void tile8_step(const Grid& g, const TileConsts& k, double* lds)
{
    using S = TileWg<R>;
    constexpr int ROWS = R + 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const TileVel va = vel_y(wave < 4 ? 0 : 2, wave & 3);
    const int jn = wave == 5 ? 2 : wave == 6 ? 4 : wave == 7 ? 5 : 0;
    const TileVel yb = vel_y(1, wave & 3), nb = vel_x(jn), vb = wave < 4 ? yb : nb;
    const TileVel vc = vel_x(jn + 1);
    const bool hasc = wave == 4 || wave == 5;
    const int m = wave - 4;
    double* const st = lds + S::ST;
    const int nx = g.nx(), ny = g.ny(), rb = 8 * nx;
    const int64_t plane = (int64_t)nx * ny;
    const int y0 = g.y0, wd = FAST ? 64 : min(64, nx - g.x0);

    // ---- load, stage, y faces
    double f0 = 0.0, dya[R], dyb[R];
    {
        double pa[ROWS], pb[ROWS], ha, hb;
        // the loads of a tile ahead of the faces of the CU's other two
        if (!NT) __builtin_amdgcn_s_setprio(3);
        const int lane = tile_lane();
        vel_load<R, FAST>(g, k, va, lane, pa, ha);
        if (m >= 0) f0 = rest_load<FAST>(g, m, wd, lane);
        if (wave < 4) {
            vel_load<R, FAST>(g, k, yb, lane, pb, hb);
        } else {
            double pn[ROWS], hn, pc[ROWS], hc = 0.0;
            vel_load<R, FAST>(g, k, nb, lane, pn, hn);
            if (hasc) vel_load<R, FAST>(g, k, vc, lane, pc, hc);
            vel_stage<R, FAST>(nb, wd, lane, pn, hn, lds);
            if (hasc) vel_stage<R, FAST>(vc, wd, lane, pc, hc, lds);
        }
        warm_consts(k);
        vel_stage<R, FAST>(va, wd, lane, pa, ha, lds);
        if (wave < 4) vel_stage<R, FAST>(yb, wd, lane, pb, hb, lds);
        if (!NT) __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        strip_diff<R, SCHEME>(pa, k.s[va.s].ey, dya);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            asm volatile("" : "+v"(dya[q]));
            dyb[q] = 0.0;
        }
        __builtin_amdgcn_sched_barrier(0);
        if (wave < 4) strip_diff<R, SCHEME>(pb, k.s[1].ey, dyb);
#pragma unroll
        for (int q = 0; q < R; ++q) asm volatile("" : "+v"(dyb[q]));
        __builtin_amdgcn_sched_barrier(0);
    }
    if (m >= 0) tile_cells<R, FAST>(g, k, m, wd, f0, lds);
    __syncthreads();
    tile_energy<R>(g, lds);

    // ---- a velocity's x faces, update and stores
    const double omct = 1.0 - g.ct();
    auto finish = [&](const TileVel& v, const double (&dhy)[R]) {
        const int lane = tile_lane();
        const TileShell& ks = k.s[v.s];
        double* s_p = lds + (v.i - 1) * S::PL;
        const int lc = v.negx ? 63 - lane : lane;
        double fc[R], P[ROWS], dh[R];
#pragma unroll
        for (int j = 0; j < R; ++j) fc[j] = s_p[j * PITCH + HALO + lc];
        const double* b = s_p + (lane % R) * PITCH + lane / R * R;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) P[j] = b[j];
        strip_diff<R, SCHEME>(P, v.hasy ? ks.eh : ks.ek, dh);
        plane_sync<2>();
#pragma unroll
        for (int q = 0; q < R; ++q) s_p[(lane % R) * XPITCH + lane / R * R + q] = dh[q];
        plane_sync<2>();
        const double ax = v.hasy ? ks.vh : ks.vk, ay = v.hasy ? ks.vs : 0.0;
        const double vx = v.negx ? -ax : ax, vy = v.negy ? -ay : ay;
        const double ncx = -(g.cx() * ax), ncy = -(g.cy() * ay);
#pragma unroll
        for (int mc = 0; mc < R; ++mc) {
            const int mr = v.negy ? R - 1 - mc : mc;
            const double* sc = st + mr * 64 + lane;
            const double eta = __builtin_fma(vx, sc[3 * R * 64], vy * sc[4 * R * 64]);
            double fn = __builtin_fma(omct, fc[mc],
                                      sc[v.s * R * 64] * feq_poly(eta, sc[5 * R * 64]));
            fn = __builtin_fma(ncx, s_p[mc * XPITCH + lc], fn);
            fn = __builtin_fma(ncy, dhy[mc], fn);
            double* row = g.fout() + v.i * plane + (int64_t)y0 * nx + g.x0;
            if constexpr (FAST)
                row_store<NT>(fn, rows_rsrc(row, R * rb), 8u * (unsigned)lane, uniform(mr * rb));
            else
                row_store<NT>(fn, rows_rsrc(row + (int64_t)mr * nx, y0 + mr < ny ? 8 * wd : 0),
                              8u * (unsigned)lane, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    finish(va, dya);
    finish(vb, dyb);
    if (hasc) {
        double z[R];
#pragma unroll
        for (int q = 0; q < R; ++q) z[q] = 0.0;
        finish(vc, z);
    }
}

template <int R, bool NT, bool FAST, int SCHEME, class Grid>
__device__ __forceinline__ void tile_step_any(const Grid& g, const TileConsts& k, double* lds)
{
    if constexpr (tile_waves(R) == 8)
        tile8_step<R, NT, FAST, SCHEME>(g, k, lds);
    else
        tile_step<R, NT, FAST, SCHEME>(g, k, lds);
}

// Tile g of either kind.
template <int R, bool NT, int SCHEME, class Grid>
__device__ __forceinline__ void tile_any(const Grid& g, const TileConsts& k, double* lds)
{
    if (g.nx() <= TILE_MAX_NX && fast_tile(g.bc(), g.x0, g.y0, TX, R, HALO))
        tile_step_any<R, NT, true, SCHEME>(g, k, lds);
    else
        tile_step_any<R, NT, false, SCHEME>(g, k, lds);
}

// A launch over one grid: one workgroup per tile, XCD-major over the strip walk
// as in k_step.
struct TileArgs {
    StepGrid s;
    double* __restrict__ ke_part;  // [ntiles][2] or null
    int tiles_y, nwork, per_xcd;
    int first;  // workgroup number of the launch's first (launch_spans)
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
    t.first = 0;
    t.k = tile_consts(k);
    return t;
}

// Launches `kernel` over all tiles of t in tiles of R rows.
inline hipError_t launch_tiles(void (*kernel)(TileArgs), TileArgs t, int R, hipStream_t st)
{
    const int threads = 64 * tile_waves(R);
    return launch_spans(8ll * t.per_xcd, threads, [&](int first, unsigned count) {
        t.first = first;
        hipLaunchKernelGGL(kernel, dim3(count), dim3(threads), 0, st, t);
    });
}

// Workgroup blockIdx.x of such a launch.
template <int R, bool NT, int SCHEME>
__device__ __forceinline__ void tile_block(const TileArgs& a, double* lds)
{
    const int b = a.first + (int)blockIdx.x;
    const int work = (b & 7) * a.per_xcd + (b >> 3);
    if (work >= a.nwork) return;
    const TileXY t = strip_walk_xy(work, a.s.tiles_x, a.tiles_y);
    tile_any<R, NT, SCHEME>(
        TileOfGrid{a, t.tx * TX, t.ty * R,
                   a.ke_part ? a.ke_part + 2 * (t.ty * a.s.tiles_x + t.tx) : nullptr}, a.k, lds);
}

}  // namespace lbmd
