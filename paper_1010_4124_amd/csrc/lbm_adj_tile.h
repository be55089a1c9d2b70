// lbm_adj_tile.h -- the reverse step (see lbm_adjoint.hip) of one 64 x R tile
// by one workgroup of 12 wavefronts that holds f^n and lambda^{n+1} of all 18
// moving planes at once: the device body of the whole-tile reverse variants.
//
// The waves share the velocities and cell rows as in lbm_tile.h, in the same
// canonical frame (columns and rows counted along v_x and v_y). A row of cells
// forms its K's from the staged planes, so that f and lambda are read once and
// no pass over them comes first.
//   load     rows of f (R + 8) and lambda (R + 6) for the y faces to registers
//   stage    their R centre rows with the x halo to LDS; the strip's R + 4 y
//            faces, from the registers                               | barrier
//   phase A  the cell rows' K's and rest plane; x faces row by row, one per
//            lane, whose five contributions go through LDS to the cells; the
//            four faces beyond a row's ends on 4 R lanes at once     | barrier
//   phase B  output rows
// Reflecting walls in y: the ghost rows of plane j hold rows of its mirror i,
// so what plane j's wall faces give those ghosts belongs to i. The wave of j has
// it in its strip already and hands it over through LDS. The terms of walls in x
// are added by a second kernel (k_adj_wall).
//
// What bounds it: one workgroup per CU (142 KB of LDS, 168 registers), whose
// phases do not overlap: VALU issues 41% of the time at 256^2 (9 of 22 us, most of
// it the 3.25 faces per cell and velocity) and 52% at 2048^2, with HBM traffic
// of 498 and 476 B per cell of the 456 it cannot do without. Measured per reverse
// step, against the state pass and one workgroup per tile and velocity:
// 128^2 19 us (27), 256^2 21 us (40), 600 x 200 37 us (68).
#pragma once

#include "lbm_tile.h"

namespace lbmd {

template <int R>
struct AdjTile {
    static constexpr int FC = 4;            // halo columns on each side
    static constexpr int P = 64 + 2 * FC;   // row pitch of a staged plane
    static constexpr int PL = R * P;
    static constexpr int LAM = 18 * PL;     // lambda planes after the f planes
    static constexpr int K = 2 * 18 * PL;   // [4][R][64]
    static constexpr int G = K + 4 * R * 64;  // per wave [4][68]: face contributions of a row
    static constexpr int GW = 4 * 68;
    static constexpr int W = G + TILE_WAVES * GW;  // per wave [R][64]: wall sums
    static constexpr int LDS = W + TILE_WAVES * R * 64;
    static_assert(R >= 3, "the rows next to a wall in y lie in one tile");
    static_assert(13 * R <= 64, "both halos of a plane take one 64-lane load");
};

// Loads of one plane's halo columns (lanes below 13 R): 8 of f for each row, then
// 5 of lambda. Columns are counted from the tile's first cell of w; canonical
// columns -4..-1, 64..67 of f and -2, -1, 64, 65, 66 of lambda.
struct AdjHalo {
    bool any, lam;
    int row, col;
};
template <int R>
__device__ __forceinline__ AdjHalo adj_halo(int lane, bool negx, int w)
{
    AdjHalo h;
    h.any = lane < 13 * R;
    h.lam = lane >= 8 * R;
    const int l = h.lam ? lane - 8 * R : lane;
    h.row = h.lam ? l / 5 : l >> 3;
    const int q = h.lam ? l - 5 * h.row : l & 7;
    const int c = h.lam ? (q < 2 ? q - 2 : w + q - 2) : (q < 4 ? q - 4 : w + q - 4);
    h.col = negx ? w - 1 - c : c;
    return h;
}

// Sums over the faces of one row of canonical cells, one cell per lane: s_f and
// s_l are the staged row's canonical column 0; eg holds, in lanes 4 r + e, the
// contributions of the edge faces -2, -1, 64, 65 of row r.
__device__ __forceinline__ double adj_x_row(const double* s_f, const double* s_l, double* G, int r,
                                            int lane, double vx, double cnx, double eps,
                                            const double (&eg)[5])
{
    const double* f = s_f + lane;
    double Gx[5];
    face_g5(vx * f[-2], vx * f[-1], vx * f[0], vx * f[1], vx * f[2], eps,
            cnx * (s_l[lane + 1] - s_l[lane]), Gx);
    plane_sync<2>();  // (the previous row's contributions have been read)
    G[lane + 2] = Gx[0];
    G[68 + lane + 2] = Gx[1];
    G[2 * 68 + lane + 2] = Gx[3];
    G[3 * 68 + lane + 2] = Gx[4];
    if ((lane >> 2) == r) {
        const int s = (lane & 3) < 2 ? (lane & 3) : 64 + (lane & 3);
        G[s] = eg[0];
        G[68 + s] = eg[1];
        G[2 * 68 + s] = eg[3];
        G[3 * 68 + s] = eg[4];
    }
    plane_sync<2>();
    return ((G[lane + 4] + G[68 + lane + 3]) + Gx[2]) + (G[2 * 68 + lane + 1] + G[3 * 68 + lane]);
}

template <int R, bool FAST>
__device__ __forceinline__ void adj_tile_step(const AdjArgs& a, int x0, int y0, double* lds)
{
    using S = AdjTile<R>;
    constexpr int FR = R + 8, LR = R + 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const TileWave v = tile_wave(wave);
    const int nx = a.nx, ny = a.ny, rb = 8 * nx;
    const int64_t plane = (int64_t)nx * ny;
    const int w = FAST ? 64 : min(64, nx - x0);
    const bool hasm = v.m >= 0 && v.m < R;
    const GridBC b = grid_of(a);
    const Consts& k = a.k;
    // (uniform: the compiler would keep them in vector registers, and spill)
    double* const s_fy = lds + (int)uniform((v.iy - 1) * S::PL) + S::FC;
    double* const s_fn = lds + (int)uniform((v.in - 1) * S::PL) + S::FC;

    double f0 = 0.0, l0 = 0.0;
    // the rest plane of the wave's cell row (boundary tiles: asked for after the
    // y faces, for want of registers)
    auto rest_rows = [&]() {
        if (!hasm) return;
        const int64_t c = (int64_t)(FAST ? y0 + v.m : min(y0 + v.m, ny - 1)) * nx + x0;
        const unsigned l8 = 8u * (unsigned)tile_lane();
        f0 = row_load(rows_rsrc(a.f + c, 8 * w), l8, 0);
        l0 = row_load(rows_rsrc(a.lam1 + c, 8 * w), l8, 0);
    };

    // ---- load
    double f[FR], L[LR], h, fn[R], ln[R], hn = 0.0;
    {
        const int lane = tile_lane();
        const unsigned l8 = 8u * (unsigned)lane;
        const AdjHalo hy = adj_halo<R>(lane, v.ynegx, w), hq = adj_halo<R>(lane, v.nnegx, w);
        const int hym = v.negy ? R - 1 - hy.row : hy.row;
        // the value of plane i at halo position (col, row m), of lambda or of f
        auto halo = [&](const AdjHalo& q, int m, int i) {
            if constexpr (FAST) {
                const double* base = (q.lam ? a.lam1 : a.f) + i * plane;
                return base[q.any ? (int64_t)(y0 + m) * nx + wrap_once(x0 + q.col, nx) : 0];
            } else {
                int col = 0, kind = CK_NONE;
                const bool in = q.any && y0 + m < ny;
                if (in)
                    x_source_g<false>(b, wrap_near(x0 + q.col, nx, b.bc[XLO], b.bc[XHI]), col, kind);
                if (q.lam && kind != CK_NORM) kind = CK_NONE;  // (lambda is zero outside)
                const bool ld = kind == CK_NORM || kind == CK_MIRX;
                const double* base = (q.lam ? a.lam1 : a.f) + (kind == CK_MIRX ? k.mirx[i] : i) * plane;
                const double x = base[ld ? (int64_t)(y0 + m) * nx + col : 0];
                const double c = kind == CK_CXLO ? k.side_eq[XLO][i]
                                 : kind == CK_CXHI ? k.side_eq[XHI][i] : 0.0;
                return ld ? x : c;
            }
        };
        {
            // (waves without such a velocity skip its rows by their range)
            auto nrow = [&](const double* base, int y) {
                return row_load(rows_rsrc(base + v.in * plane + (int64_t)y * nx + x0,
                                          v.hasn ? 8 * w : 0), l8, 0);
            };
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int y = FAST ? y0 + j : min(y0 + j, ny - 1);
                fn[j] = nrow(a.f, y);
                ln[j] = nrow(a.lam1, y);
            }
        }
        if (v.hasn) hn = halo(hq, hq.row, v.in);
        auto stage_n = [&]() {
            if (!v.hasn) return;
            const int nc = v.nnegx ? 63 - lane : lane;
            if (FAST || lane < w) {
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    s_fn[j * S::P + nc] = fn[j];
                    s_fn[S::LAM + j * S::P + nc] = ln[j];
                }
            }
            if (hq.any)
                s_fn[(hq.lam ? S::LAM : 0) + hq.row * S::P + (v.nnegx ? 63 - hq.col : hq.col)] = hn;
        };
        // (boundary tiles: at once, for want of registers)
        if constexpr (!FAST) stage_n();
        h = halo(hy, hym, v.iy);
        if constexpr (!FAST) __builtin_amdgcn_sched_barrier(0);
        if constexpr (FAST) {
            // canonical row j of f is row y0-4 + j or y0+R+3 - j, of lambda y0-3 + j
            // or y0+R+2 - j
            const __amdgpu_buffer_rsrc_t rf =
                rows_rsrc(a.f + v.iy * plane + (int64_t)(y0 - 4) * nx + x0, (R + 8) * rb);
            const __amdgpu_buffer_rsrc_t rl =
                rows_rsrc(a.lam1 + v.iy * plane + (int64_t)(y0 - 3) * nx + x0, (R + 6) * rb);
            const int sd = v.negy ? -rb : rb;
            const int sf = v.negy ? (R + 7) * rb : 0, sl = v.negy ? (R + 5) * rb : 0;
#pragma unroll
            for (int j = 0; j < FR; ++j) f[j] = row_load(rf, l8, uniform(sf + j * sd));
#pragma unroll
            for (int j = 0; j < LR; ++j) L[j] = row_load(rl, l8, uniform(sl + j * sd));
        } else {
            const RowSources rf = row_sources<false>(b, a.f, v.iy, k.miry[v.iy], x0, w, [&](int j) {
                return v.negy ? y0 + R + 3 - j : y0 - 4 + j;
            }, FR, lane);
            const RowSources rl = row_sources<true>(b, a.lam1, v.iy, k.miry[v.iy], x0, w, [&](int j) {
                return v.negy ? y0 + R + 2 - j : y0 - 3 + j;
            }, LR, lane);
#pragma unroll
            for (int j = 0; j < FR; ++j) f[j] = rf.load(j, l8);
#pragma unroll
            for (int j = 0; j < LR; ++j) L[j] = rl.load(j, l8);
            if (rf.fixed) {  // rows of a fixed-equilibrium side
#pragma unroll
                for (int j = 0; j < FR; ++j) {
                    const bool low = (v.negy ? y0 + R + 3 - j : y0 - 4 + j) < 0;
                    if (rf.fixed >> j & 1) f[j] = k.side_eq[low ? YLO : YHI][v.iy];
                }
            }
        }
        if constexpr (FAST) rest_rows();
        // ---- stage
        if (FAST || lane < w) {
            const int yc = v.ynegx ? 63 - lane : lane;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                s_fy[j * S::P + yc] = f[j + 4];
                s_fy[S::LAM + j * S::P + yc] = L[j + 3];
            }
        }
        if constexpr (FAST) stage_n();
        if (hy.any) {
            s_fy[(hy.lam ? S::LAM : 0) + hy.row * S::P + (v.ynegx ? 63 - hy.col : hy.col)] = h;
        }
    }
    const double vx = k.vx[v.iy], vy = k.vy[v.iy], vn = k.vx[v.in], eps = k.eps;
    // ---- y faces of the strip, from the registers; Gp: what they give the canonical rows -4 .. R+3
    double accy[R];
    const int H = ny - y0;  // rows from the tile's first to the end
    const bool wlo = !FAST && b.bc[YLO] == REFLECT && y0 == 0;
    const bool whi = !FAST && b.bc[YHI] == REFLECT && H <= R + 2;
    {
        double Gp[FR];
#pragma unroll
        for (int q = 0; q < FR; ++q) Gp[q] = 0.0;
        __builtin_amdgcn_sched_barrier(0);
        gather_faces<R, !FAST>(f, L, vy, v.negy ? -a.cy : a.cy, eps, Gp);
#pragma unroll
        for (int m = 0; m < R; ++m) accy[m] = vy * Gp[m + 4];
        if (wlo || whi) {
            // what the ghosts of the tile's rows received: the ghost of row m is
            // at strip position -1 - m, or 2 H - 1 - m beyond the upper wall
            double* W = lds + S::W + wave * R * 64 + tile_lane();
#pragma unroll
            for (int m = 0; m < R; ++m) W[m * 64] = 0.0;
#pragma unroll
            for (int q = 0; q < FR; ++q) {
                const int pos = v.negy ? R + 3 - q : q - 4;
                const int lo = -1 - pos, hi = 2 * H - 1 - pos;
                if (wlo && lo >= 0 && lo < HALO) W[lo * 64] += vy * Gp[q];
                if (whi && hi >= max(0, H - HALO) && hi < min(H, R)) W[hi * 64] += vy * Gp[q];
            }
        }
    }
#pragma unroll
    for (int m = 0; m < R; ++m) asm volatile("" : "+v"(accy[m]));
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!FAST) rest_rows();
    __syncthreads();

    // ---- phase A
    if (hasm) {
        const int lane = tile_lane(), m = v.m;
        const bool act = FAST || (lane < w && y0 + m < ny);
        // shell by shell (the velocities of a shell side by side: all 18 at once
        // do not fit the registers); LDS offsets of direction d of the first shell
        int at[6];
#pragma unroll
        for (int d = 0; d < 6; ++d)
            at[d] = d * S::PL + (dir_sin_sign(d) < 0 ? R - 1 - m : m) * S::P + S::FC +
                    (dir_cos(d) < 0.0 ? 63 - lane : lane);
        // the sums of k_sums, in its order
        double r = 0.0, jx = 0.0, jy = 0.0, E = 0.0;
        r += f0;
        jx = __builtin_fma(f0, k.vx[0], jx);
        jy = __builtin_fma(f0, k.vy[0], jy);
        E = __builtin_fma(f0, k.hv2[0], E);
#pragma unroll 1
        for (int s = 0; s < 3; ++s) {
#pragma unroll
            for (int d = 0; d < 6; ++d) {
                const int i = 1 + 6 * s + d;
                const double fi = lds[6 * S::PL * s + at[d]];
                r += fi;
                jx = __builtin_fma(fi, k.vx[i], jx);
                jy = __builtin_fma(fi, k.vy[i], jy);
                E = __builtin_fma(fi, k.hv2[i], E);
            }
        }
        if (!act) {
            r = E = 1.0;
            jx = jy = 0.0;
        }
        AdjSums q(r, jx, jy, E);
        {
            const double F0 = 1.0 - 6.0 * (weight_c(k, 0, q.T) + weight_c(k, 1, q.T) +
                                           weight_c(k, 2, q.T));
            const double d0 = -6.0 * (dweight_c(k, 0, q.T) + dweight_c(k, 1, q.T) +
                                      dweight_c(k, 2, q.T));
            q.add(l0, k.vx[0], k.vy[0], F0, d0);
        }
#pragma unroll 1
        for (int s = 0; s < 3; ++s) {
            const double Fs = weight_c(k, s, q.T), dFs = dweight_c(k, s, q.T);
#pragma unroll
            for (int d = 0; d < 6; ++d) {
                const int i = 1 + 6 * s + d;
                q.add(lds[S::LAM + 6 * S::PL * s + at[d]], k.vx[i], k.vy[i], Fs, dFs);
            }
        }
        const AdjCell c = q.finish(l0, a.ct, a.wdxdy);
        double* sk = lds + S::K + m * 64 + lane;
        sk[0] = c.K0;
        sk[R * 64] = c.Kx;
        sk[2 * R * 64] = c.Ky;
        sk[3 * R * 64] = c.KE;
        row_store<false>(c.rest, rows_rsrc(a.lam0 + (int64_t)(y0 + m) * nx + x0,
                                           FAST || y0 + m < ny ? 8 * w : 0),
                         8u * (unsigned)lane, 0);
    }
    // x faces of a plane's rows
    auto x_plane = [&](const double* s_f, double vv, bool neg, double(&xs)[R]) {
        const int lane = tile_lane();
        double* G = lds + S::G + wave * S::GW;
        const double cnx = neg ? -a.cx : a.cx;
        double eg[5];
        {
            // lanes 4 r + e: face -2, -1, 64 or 65 of row r
            const int er = min(lane >> 2, R - 1), e = lane & 3, c = e < 2 ? e - 2 : 62 + e;
            const double* p = s_f + er * S::P + c;
            face_g5(vv * p[-2], vv * p[-1], vv * p[0], vv * p[1], vv * p[2], eps,
                    cnx * (p[S::LAM + 1] - p[S::LAM]), eg);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            xs[r] = adj_x_row(s_f + r * S::P, s_f + S::LAM + r * S::P, G, r, lane, vv, cnx, eps, eg);
            asm volatile("" : "+v"(xs[r]));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    double xy[R], xn[R];
    x_plane(s_fy, vx, v.ynegx, xy);
    if (v.hasn) x_plane(s_fn, vn, v.nnegx, xn);
    // the sums are by canonical column; each goes to the lane of its cell
    const int lane = tile_lane();
    if (v.ynegx) {
#pragma unroll
        for (int r = 0; r < R; ++r) xy[r] = __shfl(xy[r], 63 - lane, 64);
    }
    if (v.hasn && v.nnegx) {
#pragma unroll
        for (int r = 0; r < R; ++r) xn[r] = __shfl(xn[r], 63 - lane, 64);
    }
    double lc[R], lq[R];
#pragma unroll
    for (int j = 0; j < R; ++j) lc[j] = s_fy[S::LAM + j * S::P + (v.ynegx ? 63 - lane : lane)];
    if (v.hasn) {
#pragma unroll
        for (int j = 0; j < R; ++j) lq[j] = s_fn[S::LAM + j * S::P + (v.nnegx ? 63 - lane : lane)];
    }
    __syncthreads();
    // The third ghost row beyond a wall in y whose last tile has two rows is past
    // the strip of the tile below it: its one face that reaches row ny - 3, for
    // the velocities towards the wall. It waits in the place of the lambda plane.
    const bool past = !FAST && whi && H == R + 2 && !v.negy;
    if constexpr (!FAST) {
        if (past) {
            const int i = (int)uniform(v.iy), j = k.miry[i];
            const unsigned l8 = 8u * (unsigned)tile_lane();
            int last = ny - 1;
            asm volatile("" : "+s"(last));  // (no addresses kept from the tile's loads)
            auto at = [&](const double* base, int pl, int up) {
                return row_load(rows_rsrc(base + pl * plane + (int64_t)(last - up) * nx + x0, 8 * w),
                                l8, 0);
            };
            double F[5] = {at(a.f, i, 2), at(a.f, i, 1), at(a.f, i, 0), at(a.f, j, 0),
                           at(a.f, j, 1)};
            const double mu = a.cy * at(a.lam1, j, 0);
#pragma unroll
            for (int q = 0; q < 5; ++q) F[q] *= vy;
            double G[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
            weno_face_bar(F, eps, mu, G);
            s_fy[S::LAM + lane] = vy * G[0];
        }
    }

    // ---- phase B
    const double omct = 1.0 - a.ct;
    auto put = [&](int plane_i, int m_, double l, double x, double y, double ux, double uy) {
        const int i = (int)uniform(plane_i), m = (int)uniform(m_);
        const double* sk = lds + S::K + m * 64 + lane;
        double out = __builtin_fma(omct, l, sk[0]);
        out = __builtin_fma(sk[R * 64], ux, out);
        out = __builtin_fma(sk[2 * R * 64], uy, out);
        out = __builtin_fma(sk[3 * R * 64], k.hv2[i], out);
        out += __builtin_fma(ux, x, y);
        if (past && i == v.iy && m == R - 1) out += s_fy[S::LAM + lane];
        row_store<false>(out, rows_rsrc(a.lam0 + i * plane + (int64_t)(y0 + m) * nx + x0,
                                        FAST || y0 + m < ny ? 8 * w : 0),
                         8u * (unsigned)lane, 0);
    };
#pragma unroll
    for (int mc = 0; mc < R; ++mc) {
        const int m = v.negy ? R - 1 - mc : mc;
        double y = accy[mc];
        // (from the wave of the velocity mirrored in y)
        if (wlo || whi) y += lds[S::W + (wave ^ 3) * R * 64 + m * 64 + lane];
        put(v.iy, m, lc[mc], xy[mc], y, vx, vy);
    }
    if (v.hasn) {
#pragma unroll
        for (int m = 0; m < R; ++m) put(v.in, m, lq[m], xn[m], 0.0, vn, 0.0);
    }
}

template <int R>
__global__ __launch_bounds__((64 * TILE_WAVES)) __attribute__((amdgpu_waves_per_eu(3)))
void k_adj_tile(AdjArgs a)
{
    __shared__ double lds[AdjTile<R>::LDS];
    const int b = blockIdx.x;
    const int work = (b & 7) * a.per_xcd + (b >> 3);
    if (work >= a.nwork) return;
    const int tile = strip_walk(work, a.tiles_x, a.tiles_y);
    const int ty = tile / a.tiles_x, tx = tile - ty * a.tiles_x;
    if (a.nx <= TILE_MAX_NX && fast_tile(grid_of(a), tx * TX, ty * R, TX, R, FH))
        adj_tile_step<R, true>(a, tx * TX, ty * R, lds);
    else
        adj_tile_step<R, false>(a, tx * TX, ty * R, lds);
}

// The wall terms of reflecting walls in x, which no strip of k_adj_tile has, added
// to lam0: the three columns next to each, a thread per cell (plane, row, column).
// Inside the tile kernel, as its last chain of loads and faces, these took 88 of
// the 107 us of a 64 x 64 box; so the two kernels take 26 (256 x 195: 48, 29).
// Columns next to the walls of a grid that has any.
__host__ __device__ inline int adj_wall_columns(int nx, int bc_xlo, int bc_xhi)
{
    const bool lo = bc_xlo == REFLECT, hi = bc_xhi == REFLECT;
    return lo && hi ? min(2 * HALO, nx) : lo || hi ? HALO : 0;
}

__global__ __launch_bounds__(64) void k_adj_wall(AdjArgs a)
{
    const bool lo = a.bc[XLO] == REFLECT, hi = a.bc[XHI] == REFLECT;
    const int nc = adj_wall_columns(a.nx, a.bc[XLO], a.bc[XHI]);
    const int64_t t = (int64_t)blockIdx.x * 64 + threadIdx.x, rows = t / nc;
    if (rows >= (int64_t)(NV - 1) * a.ny) return;
    const int i = 1 + (int)(rows / a.ny), y = (int)(rows - (int64_t)(i - 1) * a.ny);
    const int c = (int)(t - rows * nc), x = lo && c < HALO ? c : a.nx - nc + c;
    const int j = a.k.mirx[i];
    double e = 0.0;  // (a cell may be near both walls)
    if (lo && x < HALO) e += wall_term(a, j, 0, y, 1, 0, x, a.k.vx[j], a.cx);
    if (hi && x >= a.nx - HALO)
        e += wall_term(a, j, a.nx - 1, y, -1, 0, a.nx - 1 - x, -a.k.vx[j], a.cx);
    a.lam0[((int64_t)i * a.ny + y) * a.nx + x] += e;
}

}  // namespace lbmd
