// window_kernel.hpp -- one or more time steps of a 2D window of a plate per block.
//
// A block owns a rectangle of output nodes and keeps a window around it, WW
// columns by WH rows, one column and K rows per thread: a site's own state
// (u, j, f and the intermediates of the step) stays in its thread's
// registers, and LDS only carries what neighbours read. The stages of a
// step run on the whole window at once, each valid one ring further in:
//   u_n -> K = P + Pbar (ring 1) -> source, collision (2) -> pull streaming,
//   moments, predictor u^p (3) -> K of u^p (4) -> corrector (5);
// the explicit scheme ends at ring 3. One barrier separates two stages (five
// per step), and nothing waits for another block. Further steps of the same
// launch run on the registers the last one left, another 5 (3) rings further
// in, so `nsteps` steps read and write the state once.
//
// Walls (any edge) and holes: the thread of the node next to a wall writes
// the ghost values of the displacement beyond it, and a value a wall returns
// into direction i of a node is written to the LDS slot the pull reads for it
// (direction i of the ghost or hole site the link comes from: no site but
// that node reads it), so the streaming stage itself has no wall code.
//
// The arithmetic of a site is the fused step kernel's, expression by
// expression (y walls included), so both give the same bits; plates with x
// walls or holes keep one arithmetic too, whatever shape and split runs them.
//
// Bound: on small plates the latency of a launch, of the load and of five
// stages (about 400 vector instructions a site on periodic plates, walls three
// times that); on larger ones the issue of those instructions, with the rings
// computed twice. Per step against the fused kernel's plan, which marches 12
// or more dependent rows: 64^2 FP64 4.2 us (12.3), 256^2 FP32_U64 5.1 (16.4),
// 512^2 FP32_U64 9.5 (19.5), between y walls 11.3 (23.7); 80^2 FP64 with a
// hole 8.2 (17.0 with the 2D tiles, which spent 1500 of 2500 vector
// instructions on index arithmetic).
#pragma once

#include <algorithm>
#include <cmath>

#include "../../include/lbm_solid.h"
#include "general_kernels.hpp"

namespace lbm {

constexpr int kWinMaxSteps = 2;  // steps per launch at most

// Geometry of a launch: output rectangle of a block, blocks per row, blocks,
// steps; the momentum walls' displacement at steps n .. n + nsteps.
struct WinGrid {
    int out_w, out_h, nbx, nb, nsteps;
    double uw[kWinMaxSteps + 1][4][2];
};

// Keeps code that depends on v where it is written (the wall code of a site
// would otherwise be prepared, in registers, for every stage at once).
__device__ __forceinline__ unsigned opaque(unsigned v)
{
    asm("" : "+v"(v));
    return v;
}

// Rings a step of a scheme (MODE 0: explicit, 1: predictor-corrector or
// extrapolation) takes.
template <int MODE>
constexpr int win_reach()
{
    return MODE ? 5 : 3;
}

// Edges a window is built for: periodic plates; y walls between periodic x
// edges, in the fused kernel's arithmetic; walls on any edge, holes and the
// extrapolation variant beside walls, in the general rules' arithmetic.
enum : int { WIN_PERIODIC = 0, WIN_YWALLS = 1, WIN_GENERAL = 2 };

template <class PR, int MODE, int WW, int WH, int K, int GEN>
struct Window {
    using TF = typename PR::TF;
    using TU = typename PR::TU;
    using TJ = typename PR::TJ;
    using TC = typename PR::TC;
    using FS = FStore<TF>;
    static constexpr bool DEV = FS::kDeviation;
    static constexpr int N = WW * WH, BLOCK = N / K, RS = BLOCK / WW;  // RS: rows between a thread's sites
    static constexpr int HS = win_reach<MODE>();
    static_assert((WW & (WW - 1)) == 0 && BLOCK % WW == 0 && RS * K == WH, "window shape");
    struct Lds {
        TU u[2][N];
        TC k[4][N];
        TC f[8][N];  // directions 1..8
        unsigned char hole[GEN == WIN_GENERAL ? N : 1];
    };

    // bits of a site's flags
    enum : unsigned { NODE = 1u, GHOST = 2u, XL = 4u, XH = 8u, YL = 16u, YH = 32u, EDGE = XL | XH | YL | YH, HOLE = 64u,
                      BOTTOM = 128u /* ghost row below the bottom wall */, NEAR = 256u /* << direction: hole there */ };

    const GenParams &p;
    Lds &L;
    const TC lam, mu;

    __device__ __forceinline__ Window(const GenParams &p_, Lds &l) : p(p_), L(l), lam(TC(p_.lam)), mu(TC(p_.mu)) {}

    __device__ __forceinline__ static int wrap(int v, int n)
    {
        v = v < 0 ? v + n : (v >= n ? v - n : v);
        if ((unsigned)v >= (unsigned)n) {  // a plate narrower than the window
            v %= n;
            if (v < 0) v += n;
        }
        return v;
    }

    // The displacement of node i (LDS index) and, at an edge with a wall, the
    // ghost values beyond it (uw: wall displacements of the step).
    __device__ __forceinline__ void put_u(int i, int lx, int ly, unsigned fl, TU u0, TU u1, const double uw[4][2])
    {
        if (GEN && !(fl & NODE)) return;
        L.u[0][i] = u0;
        L.u[1][i] = u1;
        if (!GEN || !(fl & EDGE)) return;
        fl = opaque(fl);
        const bool lo_y = fl & YL, on_y = fl & (YL | YH);
        const bool lo_x = GEN == WIN_GENERAL && (fl & XL), on_x = GEN == WIN_GENERAL && (fl & (XL | XH));
        const int dx = lo_x ? -1 : 1, dy = lo_y ? -1 : 1;
        const int bcx = lo_x ? p.bc[EDGE_XMIN] : p.bc[EDGE_XMAX], bcy = lo_y ? p.bc[EDGE_YMIN] : p.bc[EDGE_YMAX];
        const bool x1 = (unsigned)(lx + dx) < (unsigned)WW, x2 = (unsigned)(lx + 2 * dx) < (unsigned)WW;
        const bool y1 = (unsigned)(ly + dy) < (unsigned)WH, y2 = (unsigned)(ly + 2 * dy) < (unsigned)WH;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            TU *r = L.u[a] + i;
            const TU v = a ? u1 : u0;
            const TU uwx = TU(lo_x ? uw[EDGE_XMIN][a] : uw[EDGE_XMAX][a]);
            const TU uwy = TU(lo_y ? uw[EDGE_YMIN][a] : uw[EDGE_YMAX][a]);
            if (on_y) {
                const TU g = gen_ghost<TU>(bcy, uwy, v, 1);
                if (y1) r[dy * WW] = g;
                if (y2) r[2 * dy * WW] = gen_ghost<TU>(bcy, uwy, v, 2);
                // beyond a corner only the nearest ghost is read
                if (on_x && x1 && y1) r[dy * WW + dx] = gen_ghost<TU>(bcx, uwx, g, 1);
            }
            if (on_x) {
                if (x1) r[dx] = gen_ghost<TU>(bcx, uwx, v, 1);
                if (x2) r[2 * dx] = gen_ghost<TU>(bcx, uwx, v, 2);
            }
        }
    }

    __device__ __forceinline__ static bool near(unsigned fl, int dir) { return (fl >> (8 + dir)) & 1u; }

    // Central-difference gradient of the displacement in LDS at site i (a
    // hole neighbour takes the node's own value). With y walls alone the
    // ghost row below the bottom wall takes the fused kernel's form: the row's x-derivatives from
    // row 0, negated beyond a momentum wall, whose ghosts 2 uw - u0 and
    // 4 uw - 3 u0 give the y-difference 2 (u0 - uw).
    __device__ __forceinline__ void grad(int i, unsigned fl, const double uw[4][2], TC H[4]) const
    {
        if (GEN == WIN_YWALLS && (fl & BOTTOM)) {
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const TU *r = L.u[a] + i + WW;
                const TC hx = TC((r[1] - r[-1]) * TU(0.5));
                if (p.bc[EDGE_YMIN] == BC_NEUMANN) {
                    H[2 * a] = hx;
                    H[2 * a + 1] = TC(0);
                } else {
                    H[2 * a] = -hx;
                    H[2 * a + 1] = TC(TU(2) * (r[0] - TU(uw[EDGE_YMIN][a])));
                }
            }
            return;
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const TU *r = L.u[a] + i;
            TU xp = r[1], xm = r[-1], yp = r[WW], ym = r[-WW];
            if (GEN == WIN_GENERAL && (fl >> 8)) {
                const TU c = r[0];
                if (near(fl, 1)) xp = c;
                if (near(fl, 3)) xm = c;
                if (near(fl, 2)) yp = c;
                if (near(fl, 4)) ym = c;
            }
            H[2 * a] = TC((xp - xm) * TU(0.5));
            H[2 * a + 1] = TC((yp - ym) * TU(0.5));
        }
    }

    // K at the hole neighbour across axis n as a node with gradient H sees it
    __device__ __forceinline__ void k_hole(const TC H[4], int n, TC Kh[4]) const
    {
        TC Hn[4] = {H[0], H[1], H[2], H[3]};
        Hn[n] = TC(0);
        Hn[2 + n] = TC(0);
        stress_sum(Hn, lam, mu, Kh);
    }

    __device__ __forceinline__ void source(int i, unsigned fl, const TC H[4], TC S[2]) const
    {
        TC xp0 = L.k[0][i + 1], xm0 = L.k[0][i - 1], xp2 = L.k[2][i + 1], xm2 = L.k[2][i - 1];
        TC yp1 = L.k[1][i + WW], ym1 = L.k[1][i - WW], yp3 = L.k[3][i + WW], ym3 = L.k[3][i - WW];
        if (GEN == WIN_GENERAL && (fl >> 8)) {
            TC kh[4];
            if (near(fl, 1) || near(fl, 3)) {
                k_hole(H, 0, kh);
                if (near(fl, 1)) xp0 = kh[0], xp2 = kh[2];
                if (near(fl, 3)) xm0 = kh[0], xm2 = kh[2];
            }
            if (near(fl, 2) || near(fl, 4)) {
                k_hole(H, 1, kh);
                if (near(fl, 2)) yp1 = kh[1], yp3 = kh[3];
                if (near(fl, 4)) ym1 = kh[1], ym3 = kh[3];
            }
        }
        S[0] = TC(p.bx) + TC(0.5) * (xp0 - xm0) + TC(0.5) * (yp1 - ym1);
        S[1] = TC(p.by) + TC(0.5) * (xp2 - xm2) + TC(0.5) * (yp3 - ym3);
    }

    // slot of the value pulled in direction d at site i
    __device__ __forceinline__ static int slot(int i, int d) { return i - kGy[d] * WW - kGx[d]; }

    // Whether the diagonal link (ox, oy) of a node crosses walls, and which:
    // bit 0 the x side's, bit 1 the y side's. A link into a hole crosses the
    // wall its axis step enters, or both through a hole corner.
    __device__ __forceinline__ static int crossed(unsigned fl, int o, int ox, int oy)
    {
        const bool hole = near(fl, o);
        const bool hx = near(fl, ox > 0 ? 1 : 3), hy = near(fl, oy > 0 ? 2 : 4);
        const bool bx = hole ? (hx || !hy) : (fl & (ox < 0 ? XL : XH)) != 0;
        const bool by = hole ? (hy || !hx) : (fl & (oy < 0 ? YL : YH)) != 0;
        return (bx ? 1 : 0) | (by ? 2 : 0);
    }

    // One wall of WIN_GENERAL on side S (-1: low, 1: high) of axis A of node i:
    // the values it returns for the axis link and for the two diagonals that
    // cross this wall alone, into the slots the pull reads. m: r, Pxx, Pyy,
    // Pxy of the node's populations, whose values after the collision are in
    // the LDS. eq. (25), (26) with r_bd and the tangential moments at the
    // node; K at the wall is the mean of the node's and the one beyond it (a
    // ghost node, or at a hole, T* = 0, the hole K the node sees).
    template <int A, int S>
    __device__ __forceinline__ void side(int i, unsigned fl, const TC H[4], const TC m[4])
    {
        constexpr int o0 = A ? (S > 0 ? 2 : 4) : (S > 0 ? 1 : 3);
        const bool hole = near(fl, o0);
        if (!hole && !(fl & (A ? (S > 0 ? YH : YL) : (S > 0 ? XH : XL)))) return;
        constexpr int e = A ? (S > 0 ? EDGE_YMAX : EDGE_YMIN) : (S > 0 ? EDGE_XMAX : EDGE_XMIN);
        constexpr int o1 = A ? (S > 0 ? 5 : 8) : (S > 0 ? 5 : 6);  // diagonals: e_t = 1, then -1 along the wall
        constexpr int o2 = A ? (S > 0 ? 6 : 7) : (S > 0 ? 8 : 7);
        const TC f0 = L.f[o0 - 1][i], f1 = L.f[o1 - 1][i], f2 = L.f[o2 - 1][i];
        const TC s = TC(S), w1 = TC(1.0 / 9.0), w5 = TC(1.0 / 36.0);
        const double t0 = hole ? 0.0 : p.val[e][0], t1 = hole ? 0.0 : p.val[e][1];
        TC v0, v1, v2;
        if (!hole && p.bc[e] == BC_DIRICHLET) {
            const TC jn = TC(A ? t1 : t0), jt = TC(A ? t0 : t1);
            v0 = f0 - TC(6) * w1 * (s * jn);
            v1 = f1 - TC(6) * w5 * (s * jn + jt);
            v2 = f2 - TC(6) * w5 * (s * jn - jt);
        } else {
            const int g = A ? i + S * WW : i + S;
            TC ka = L.k[A][g], kb = L.k[2 + A][g];
            if (hole) {
                TC kh[4];
                k_hole(H, A, kh);
                ka = kh[A];
                kb = kh[2 + A];
            }
            // the wall's column of Pbar*
            const TC q0 = -s * TC(t0) + TC(0.5) * (L.k[A][i] + ka), q1 = -s * TC(t1) + TC(0.5) * (L.k[2 + A][i] + kb);
            const TC Pxx = A ? m[1] : q0, Pyy = A ? q1 : m[2], Pxy = A ? q0 : q1;
            const TC r = m[0], third = TC(1) / TC(3);
            const TC axx = Pxx - r * third, ayy = Pyy - r * third;
            const TC tr = axx + ayy, an = A ? ayy : axx;
            const TC d1 = (axx + TC(2) * (s * Pxy)) + ayy, d2 = (axx - TC(2) * (s * Pxy)) + ayy;
            v0 = -f0 + TC(2) * w1 * (r + TC(4.5) * (an - tr * third));
            v1 = -f1 + TC(2) * w5 * (r + TC(4.5) * (d1 - tr * third));
            v2 = -f2 + TC(2) * w5 * (r + TC(4.5) * (d2 - tr * third));
        }
        constexpr int only = A ? 2 : 1;
        L.f[kGopp[o0] - 1][i + kGy[o0] * WW + kGx[o0]] = v0;
        if (crossed(fl, o1, kGx[o1], kGy[o1]) == only) L.f[kGopp[o1] - 1][i + kGy[o1] * WW + kGx[o1]] = v1;
        if (crossed(fl, o2, kGx[o2], kGy[o2]) == only) L.f[kGopp[o2] - 1][i + kGy[o2] * WW + kGx[o2]] = v2;
    }

    // Values the walls return to node i, into the slots its pull reads (m, H:
    // as side). y walls alone take the fused kernel's form. The general form
    // goes one side at a time, three links each, then over the diagonals that
    // cross two walls: the off-diagonal entry of Pbar* is the mean of both
    // walls' values, a momentum wall (the mean j* of two) bounces back. (A
    // rolled loop over eight links with the two-wall rule for each: 8.8 us per
    // step on the 64 x 64 plate with a hole in FP64 with 16 x 16 windows,
    // against 8.2.)
    __device__ __forceinline__ void walls(int i, unsigned fl, const TC H[4], const TC m[4])
    {
        fl = opaque(fl);
        if constexpr (GEN == WIN_YWALLS) {
            const bool top = fl & YH;
            const int g = top ? i + WW : i - WW;
            const double val[2] = {top ? p.val[EDGE_YMAX][0] : p.val[EDGE_YMIN][0],
                                   top ? p.val[EDGE_YMAX][1] : p.val[EDGE_YMIN][1]};
            const TC fco[3] = {L.f[top ? 1 : 3][i], L.f[top ? 4 : 6][i], L.f[top ? 5 : 7][i]};
            TC w[3];
            wall_populations(top, top ? p.bc[EDGE_YMAX] : p.bc[EDGE_YMIN], fco, val, m[0], m[1],
                             TC(0.5) * (L.k[1][i] + L.k[1][g]), TC(0.5) * (L.k[3][i] + L.k[3][g]), w);
            // returned as 4, 7, 8 (top) or 2, 5, 6
            L.f[top ? 3 : 1][g] = w[0];
            L.f[top ? 6 : 4][top ? g + 1 : g - 1] = w[1];
            L.f[top ? 7 : 5][top ? g - 1 : g + 1] = w[2];
            return;
        }
        side<0, -1>(i, fl, H, m);
        side<0, 1>(i, fl, H, m);
        side<1, -1>(i, fl, H, m);
        side<1, 1>(i, fl, H, m);
#pragma unroll 1
        for (int o = 5; o < 9; ++o) {
            const int ox = o == 5 || o == 8 ? 1 : -1, oy = o < 7 ? 1 : -1;
            if (crossed(fl, o, ox, oy) != 3) continue;
            const bool hole = near(fl, o);
            const int ex = ox < 0 ? EDGE_XMIN : EDGE_XMAX, ey = oy < 0 ? EDGE_YMIN : EDGE_YMAX;
            const bool ddx = !hole && p.bc[ex] == BC_DIRICHLET, ddy = !hole && p.bc[ey] == BC_DIRICHLET;
            const TC w = TC(1.0 / 36.0), cx = TC(ox), cy = TC(oy), fco = L.f[o - 1][i];
            TC val;
            if (ddx || ddy) {
                const double sc = ddx && ddy ? 0.5 : 1.0;
                const TC jx = TC(sc * ((ddx ? p.val[ex][0] : 0.0) + (ddy ? p.val[ey][0] : 0.0)));
                const TC jy = TC(sc * ((ddx ? p.val[ex][1] : 0.0) + (ddy ? p.val[ey][1] : 0.0)));
                val = fco - TC(6) * w * (cx * jx + cy * jy);
            } else {
                TC kx0 = L.k[0][i + ox], kx2 = L.k[2][i + ox], ky1 = L.k[1][i + oy * WW], ky3 = L.k[3][i + oy * WW];
                TC kh[4];
                if (near(fl, ox > 0 ? 1 : 3)) {
                    k_hole(H, 0, kh);
                    kx0 = kh[0];
                    kx2 = kh[2];
                }
                if (near(fl, oy > 0 ? 2 : 4)) {
                    k_hole(H, 1, kh);
                    ky1 = kh[1];
                    ky3 = kh[3];
                }
                const TC Pxx = -cx * TC(hole ? 0.0 : p.val[ex][0]) + TC(0.5) * (L.k[0][i] + kx0);
                const TC qx1 = -cx * TC(hole ? 0.0 : p.val[ex][1]) + TC(0.5) * (L.k[2][i] + kx2);
                const TC qy0 = -cy * TC(hole ? 0.0 : p.val[ey][0]) + TC(0.5) * (L.k[1][i] + ky1);
                const TC Pyy = -cy * TC(hole ? 0.0 : p.val[ey][1]) + TC(0.5) * (L.k[3][i] + ky3);
                const TC Pxy = TC(0.5) * (qx1 + qy0);
                const TC third = TC(1) / TC(3);
                const TC axx = Pxx - m[0] * third, ayy = Pyy - m[0] * third;
                const TC d = (axx + TC(2) * (cx * cy * Pxy)) + ayy;
                val = -fco + TC(2) * w * (m[0] + TC(4.5) * (d - (axx + ayy) * third));
            }
            L.f[o < 7 ? o + 1 : o - 3][i + oy * WW + ox] = val;
        }
    }

    __device__ __forceinline__ void run(const WinGrid &g, int x0, int y0)
    {
        const size_t pl = (size_t)p.plane;
        const TF *__restrict__ fin = static_cast<const TF *>(p.f_in);
        const TU *__restrict__ uin = static_cast<const TU *>(p.u_in);
        const TJ *__restrict__ jin = static_cast<const TJ *>(p.j_in);
        const int nx = p.nx, ny = p.ny;
        const int h = g.nsteps * HS + (DEV ? 1 : 0);
        const int ow = min(g.out_w, nx - x0), oh = min(g.out_h, ny - y0);
        const int rows = oh + 2 * h, cols = ow + 2 * h;  // of the window that are used
        const bool perx = p.bc[EDGE_XMIN] == BC_PERIODIC, pery = p.bc[EDGE_YMIN] == BC_PERIODIC;
        const TC omega = TC(p.omega), inv = TC(p.f_inv_scale), scale = TC(p.f_scale);
        const bool sr = FS::kStochastic && p.sr;
        const int lx = (int)threadIdx.x % WW, r0 = (int)threadIdx.x / WW;
        bool bad = false;

        TC f[K][9];
        TU u[K][2];
        TC j[K][2];
        uint32_t site[K];
        unsigned fl[K];
        bool out[K];
        auto row_in = [&](int k, int d) { return r0 + k * RS >= d && r0 + k * RS < rows - d; };

        const int ux = x0 - h + lx;
        int x = ux, bx = 0;
        if (GEN != WIN_GENERAL || perx) {
            x = wrap(ux, nx);
        } else if (ux < 0) {
            x = 0, bx = -ux;
        } else if (ux >= nx) {
            x = nx - 1, bx = ux - (nx - 1);
        }
        // every load of the state is issued before the first barrier
        TF lf[K][9];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int ly = r0 + k * RS, uy = y0 - h + ly;
            int y = uy, by = 0;
            if (!GEN || pery) {
                y = wrap(uy, ny);
            } else if (uy < 0) {
                y = 0, by = -uy;
            } else if (uy >= ny) {
                y = ny - 1, by = uy - (ny - 1);
            }
            site[k] = (uint32_t)y * (uint32_t)nx + (uint32_t)x;
            out[k] = lx >= h && lx < h + ow && ly >= h && ly < h + oh;
            fl[k] = NODE;
            if (GEN) {
                if (bx | by) {
                    fl[k] = bx + by == 1 ? (unsigned)GHOST : 0u;
                    if (GEN == WIN_YWALLS && uy == -1) fl[k] |= BOTTOM;
                } else {
                    if (GEN == WIN_GENERAL && !perx) fl[k] |= (ux == 0 ? XL : 0u) | (ux == nx - 1 ? XH : 0u);
                    if (!pery) fl[k] |= (uy == 0 ? YL : 0u) | (uy == ny - 1 ? YH : 0u);
                }
            }
            u[k][0] = u[k][1] = TU(0);
            j[k][0] = j[k][1] = TC(0);
#pragma unroll
            for (int i = 0; i < 9; ++i) lf[k][i] = TF(0);
            if (row_in(k, 0) && lx < cols && (!GEN || (fl[k] & NODE))) {
                u[k][0] = gload(uin, site[k]);
                u[k][1] = gload(uin + pl, site[k]);
                if (row_in(k, 2)) {
#pragma unroll
                    for (int i = 0; i < 9; ++i) lf[k][i] = gload(fin + (size_t)i * pl, site[k]);
                    j[k][0] = TC(gload(jin, site[k]));
                    j[k][1] = TC(gload(jin + pl, site[k]));
                }
            }
        }
        if (GEN == WIN_GENERAL && p.mask) {
            bool any = false;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const bool m = row_in(k, 0) && lx < cols && (fl[k] & NODE) && !(gload(p.mask, site[k]) & 1);
                L.hole[(r0 + k * RS) * WW + lx] = m;
                any |= m;
            }
            if (__syncthreads_or(any)) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int i = (r0 + k * RS) * WW + lx;
                    if (!row_in(k, 1) || lx < 1 || lx > WW - 2) continue;
                    if (L.hole[i]) {
                        fl[k] = HOLE;
                        continue;
                    }
                    unsigned nb = 0;
#pragma unroll
                    for (int d = 1; d < 9; ++d) nb |= (unsigned)L.hole[i + kGy[d] * WW + kGx[d]] << d;
                    fl[k] |= nb << 8;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int i = 0; i < 9; ++i) f[k][i] = FS::cvt(lf[k][i], inv);
            const int ly = r0 + k * RS;
            if (row_in(k, 0)) put_u(ly * WW + lx, lx, ly, fl[k], u[k][0], u[k][1], g.uw[0]);
        }

        for (int s = 0; s < g.nsteps; ++s) {
            const int d = s * HS;
            const double(*uw)[2] = g.uw[s], (*uw1)[2] = g.uw[s + 1];
            TC H[K][4], S[K][2];
            __syncthreads();
            // K of u_n; with deviation storage the populations from the
            // stored deviations (a further step takes them as a store and
            // load would leave them)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (!row_in(k, d + 1)) continue;
                if (GEN && !(fl[k] & (NODE | GHOST))) continue;
                const int i = (r0 + k * RS) * WW + lx;
                TC Kv[4];
                grad(i, fl[k], uw, H[k]);
                const TC J = stress_sum(H[k], lam, mu, Kv);
                if (out[k] && (!GEN || (fl[k] & NODE)) && !(J > TC(0))) bad = true;
#pragma unroll
                for (int c = 0; c < 4; ++c) L.k[c][i] = Kv[c];
                if constexpr (DEV) {
                    TC fr[9];
                    ref_eq(H[k], j[k][0], j[k][1], fr);
                    if (s > 0) {
                        TC dv[9];
#pragma unroll
                        for (int q = 0; q < 9; ++q) dv[q] = f[k][q] - fr[q];
                        roundtrip_site<FS>(site[k], dv, scale, inv, sr, sr ? sr_key(p.seed, p.step + s) : 0u, f[k]);
                    }
#pragma unroll
                    for (int q = 0; q < 9; ++q) f[k][q] = fr[q] + f[k][q];
                }
            }
            __syncthreads();
            // source and collision
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (!row_in(k, d + 2)) continue;
                if (GEN && !(fl[k] & NODE)) continue;
                const int i = (r0 + k * RS) * WW + lx;
                TC fc[9], r, pxx;
                source(i, fl[k], H[k], S[k]);
                collide(f[k], j[k][0], j[k][1], S[k][0], S[k][1], omega, fc, r, pxx);
#pragma unroll
                for (int q = 1; q < 9; ++q) L.f[q - 1][i] = fc[q];
                if (GEN && (fl[k] & (EDGE | ~(NEAR * 2u - 1u)))) {
                    const TC *fk = f[k];
                    const TC m[4] = {r, pxx, (fk[2] + fk[4]) + ((fk[5] + fk[6]) + (fk[7] + fk[8])),
                                     (fk[5] - fk[6]) + (fk[7] - fk[8])};
                    walls(i, fl[k], H[k], m);
                }
                f[k][0] = fc[0];
            }
            __syncthreads();
            // pull streaming, moments, predictor (or the explicit update)
            TC jf[K][2];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (!row_in(k, d + 3)) continue;
                if (GEN && !(fl[k] & NODE)) continue;
                const int ly = r0 + k * RS, i = ly * WW + lx;
                TC *fn = f[k];
#pragma unroll
                for (int q = 1; q < 9; ++q) fn[q] = L.f[q - 1][slot(i, q)];
                const TC jfx = ((fn[1] - fn[3]) + (fn[5] - fn[6])) + (fn[8] - fn[7]);
                const TC jfy = ((fn[2] - fn[4]) + (fn[5] + fn[6])) - (fn[7] + fn[8]);
                if constexpr (MODE != 0) {
                    TC jpx = jfx + TC(0.5) * S[k][0], jpy = jfy + TC(0.5) * S[k][1];
                    if (p.pc == 2) {
                        const TJ *jold = static_cast<const TJ *>(p.j_prev);
                        jpx = TC(2) * j[k][0] - TC(jold[site[k]]);
                        jpy = TC(2) * j[k][1] - TC(jold[pl + site[k]]);
                    }
                    jf[k][0] = jfx;
                    jf[k][1] = jfy;
                    put_u(i, lx, ly, fl[k], u[k][0] + TU(TC(0.5) * (jpx + j[k][0])),
                          u[k][1] + TU(TC(0.5) * (jpy + j[k][1])), uw1);
                } else {
                    const TC jx = jfx + TC(0.5) * S[k][0], jy = jfy + TC(0.5) * S[k][1];
                    u[k][0] = u[k][0] + TU(TC(0.5) * (jx + j[k][0]));
                    u[k][1] = u[k][1] + TU(TC(0.5) * (jy + j[k][1]));
                    j[k][0] = TC(TJ(jx));
                    j[k][1] = TC(TJ(jy));
                    put_u(i, lx, ly, fl[k], u[k][0], u[k][1], uw1);
                }
            }
            if constexpr (MODE != 0) {
                __syncthreads();
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if (!row_in(k, d + 4)) continue;
                    if (GEN && !(fl[k] & (NODE | GHOST))) continue;
                    const int i = (r0 + k * RS) * WW + lx;
                    TC Kv[4];
                    grad(i, fl[k], uw1, H[k]);
                    stress_sum(H[k], lam, mu, Kv);
#pragma unroll
                    for (int c = 0; c < 4; ++c) L.k[c][i] = Kv[c];
                }
                __syncthreads();
                // corrector
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if (!row_in(k, d + 5)) continue;
                    if (GEN && !(fl[k] & NODE)) continue;
                    const int ly = r0 + k * RS, i = ly * WW + lx;
                    TC Sp[2];
                    source(i, fl[k], H[k], Sp);
                    const TC jx = jf[k][0] + TC(0.5) * Sp[0], jy = jf[k][1] + TC(0.5) * Sp[1];
                    u[k][0] = u[k][0] + TU(TC(0.5) * (jx + j[k][0]));
                    u[k][1] = u[k][1] + TU(TC(0.5) * (jy + j[k][1]));
                    j[k][0] = TC(TJ(jx));
                    j[k][1] = TC(TJ(jy));
                    if (DEV || s + 1 < g.nsteps) put_u(i, lx, ly, fl[k], u[k][0], u[k][1], uw1);
                }
            }
        }

        TF *__restrict__ fout = static_cast<TF *>(p.f_out);
        TU *__restrict__ uout = static_cast<TU *>(p.u_out);
        TJ *__restrict__ jout = static_cast<TJ *>(p.j_out);
        if constexpr (DEV) __syncthreads();
        const uint32_t key = sr ? sr_key(p.seed, p.step + g.nsteps) : 0u;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!out[k]) continue;
            if (GEN && !(fl[k] & NODE)) {  // a hole node: zero state
                gstore(uout, site[k], TU(0));
                gstore(uout + pl, site[k], TU(0));
                gstore(jout, site[k], TJ(0));
                gstore(jout + pl, site[k], TJ(0));
                continue;
            }
            gstore(uout, site[k], u[k][0]);
            gstore(uout + pl, site[k], u[k][1]);
            gstore(jout, site[k], TJ(j[k][0]));
            gstore(jout + pl, site[k], TJ(j[k][1]));
            if (!isfinite((double)u[k][0]) || !isfinite((double)u[k][1]) || !isfinite((double)j[k][0]) ||
                !isfinite((double)j[k][1]))
                bad = true;
            if constexpr (DEV) {
                // the deviation from the new state's reference equilibrium
                TC Hn[4], fr[9];
                grad((r0 + k * RS) * WW + lx, fl[k], g.uw[g.nsteps], Hn);
                ref_eq(Hn, j[k][0], j[k][1], fr);
#pragma unroll
                for (int q = 0; q < 9; ++q) f[k][q] = f[k][q] - fr[q];
            }
            store_site<FS>(fout, pl, site[k], f[k], scale, sr, key);
        }
        if (bad) p.flag[0] = 1u;
    }
};

template <class PR, int MODE, int WW, int WH, int K, int GEN>
__global__ void __launch_bounds__(WW *WH / K) window_step_kernel(const GenParams p, const WinGrid g)
{
    using W = Window<PR, MODE, WW, WH, K, GEN>;
    __shared__ typename W::Lds lds;
    const int bid = blockIdx.x;
    const int xq = g.nb >> 3, xr = g.nb & 7;
    const int xcd = bid & 7, loc = bid >> 3;
    const int tile = xcd * xq + min(xcd, xr) + loc;
    const int ty = tile / g.nbx, tx = tile - ty * g.nbx;
    W w(p, lds);
    w.run(g, tx * g.out_w, ty * g.out_h);
}

// Window shapes: columns, rows, rows per thread.
struct WinShape {
    int w, h, k;
};
constexpr WinShape kWinShapes[] = {{16, 16, 1}, {32, 16, 1}, {32, 32, 1}, {64, 16, 1}, {64, 32, 2}, {32, 32, 2}};
constexpr int kNumWinShapes = (int)(sizeof(kWinShapes) / sizeof(kWinShapes[0]));

// Cost of a launch of n blocks with a shape and a number of steps, in us:
// at least lat (up to one block per compute unit), base + thr per block on
// the fullest compute unit beyond. Measured with plates of 16 to 2048 full
// windows, per class (double; float; float with a double displacement; 16-bit
// storage) and for periodic plates and plates with walls or holes. A two-step
// launch pays where the plate is small enough that the launch itself and the
// load of the state count (64 x 64 FP64: 4.2 us per step with two 32 x 32
// steps, 4.3 with 16 x 16 and 7.0 with 32 x 32 windows of one step).
struct WinCost {
    int shape, steps;
    float lat, base, thr;
};
constexpr int kNumWinCosts = 8;
constexpr WinCost kWinCosts[4][2][kNumWinCosts] = {
    {{{0, 1, 4.4f, 3.3f, 0.9f}, {1, 1, 5.6f, 2.3f, 2.4f}, {2, 1, 9.0f, 3.3f, 7.2f}, {2, 2, 9.8f, 3.0f, 7.3f},
      {3, 1, 8.4f, 1.6f, 5.8f}, {5, 1, 9.4f, 3.2f, 7.5f}},
     {{0, 1, 7.2f, 4.9f, 1.4f}, {1, 1, 8.0f, 4.1f, 3.9f}, {2, 1, 12.3f, 5.8f, 8.3f}, {2, 2, 14.7f, 5.9f, 9.5f},
      {3, 1, 10.3f, 4.6f, 6.9f}, {5, 1, 12.1f, 4.9f, 8.6f}}},
    {{{0, 1, 3.9f, 3.2f, 0.5f}, {1, 1, 4.4f, 3.2f, 1.0f}, {2, 1, 6.1f, 2.2f, 3.2f}, {2, 2, 6.6f, 2.9f, 3.0f},
      {3, 1, 5.6f, 2.1f, 2.4f}, {4, 1, 10.0f, 5.2f, 7.1f}, {4, 2, 11.1f, 2.4f, 7.9f}, {5, 1, 6.8f, 2.4f, 3.3f}},
     {{0, 1, 6.4f, 5.5f, 0.6f}, {1, 1, 6.7f, 3.8f, 1.8f}, {2, 1, 8.1f, 4.1f, 4.4f}, {2, 2, 10.8f, 5.5f, 5.5f},
      {3, 1, 7.2f, 3.8f, 3.8f}, {4, 1, 11.8f, 6.7f, 7.9f}, {4, 2, 14.0f, 5.8f, 9.0f}, {5, 1, 9.3f, 4.2f, 3.7f}}},
    {{{0, 1, 3.9f, 3.3f, 0.5f}, {1, 1, 4.5f, 3.4f, 1.0f}, {2, 1, 6.6f, 2.6f, 3.4f}, {2, 2, 7.2f, 3.0f, 3.4f},
      {3, 1, 6.1f, 2.0f, 2.8f}, {4, 1, 11.4f, 0.0f, 11.1f}, {4, 2, 12.6f, 2.2f, 9.2f}, {5, 1, 7.2f, 2.7f, 3.7f}},
     {{0, 1, 6.4f, 5.4f, 0.7f}, {1, 1, 6.8f, 3.9f, 1.8f}, {2, 1, 8.3f, 4.0f, 4.8f}, {2, 2, 10.9f, 5.8f, 5.6f},
      {3, 1, 7.3f, 3.6f, 4.0f}, {4, 1, 13.7f, 0.0f, 12.6f}, {4, 2, 15.4f, 5.4f, 10.5f}, {5, 1, 9.5f, 4.7f, 5.6f}}},
    {{{0, 1, 4.3f, 3.5f, 0.6f}, {1, 1, 4.5f, 2.9f, 1.3f}, {2, 1, 6.3f, 2.3f, 4.2f}, {2, 2, 7.8f, 1.4f, 6.0f},
      {3, 1, 6.2f, 3.2f, 3.2f}, {4, 1, 10.3f, 2.9f, 8.0f}, {4, 2, 13.0f, 3.3f, 9.5f}, {5, 1, 7.3f, 3.1f, 3.5f}},
     {{0, 1, 7.7f, 6.2f, 0.9f}, {1, 1, 7.6f, 2.8f, 2.8f}, {2, 1, 9.1f, 4.6f, 5.0f}, {2, 2, 12.0f, 5.7f, 6.8f},
      {3, 1, 8.0f, 3.4f, 4.7f}, {4, 1, 14.1f, 5.2f, 9.8f}, {4, 2, 17.4f, 6.3f, 11.8f}, {5, 1, 10.9f, 5.2f, 6.3f}}},
};

// Class of a precision in kWinCosts.
inline int win_class(lbm_precision p)
{
    return p == LBM_FP64 ? 0 : p == LBM_FP32 ? 1 : p == LBM_FP32_U64 ? 2 : 3;
}

// LDS bytes of a site of a window
template <class PR>
constexpr int win_site_bytes()
{
    return 2 * (int)sizeof(typename PR::TU) + 12 * (int)sizeof(typename PR::TC) + 1;
}
template <class PR>
constexpr bool win_fits(int s)
{
    return kWinShapes[s].w * kWinShapes[s].h * win_site_bytes<PR>() <= 160 * 1024;
}

// Output rectangle of a window with rings h on a plate: the widest that fits,
// evened out over the plate. 0 columns where the rings fill the window.
inline WinGrid win_grid(const WinShape &s, int nx, int ny, int h, int nsteps)
{
    WinGrid g{};
    const int mw = s.w - 2 * h, mh = s.h - 2 * h;
    g.nsteps = nsteps;
    if (mw <= 0 || mh <= 0) return g;
    g.nbx = (nx + mw - 1) / mw;
    const int nby = (ny + mh - 1) / mh;
    g.out_w = (nx + g.nbx - 1) / g.nbx;
    g.out_h = (ny + nby - 1) / nby;
    g.nbx = (nx + g.out_w - 1) / g.out_w;
    g.nb = g.nbx * ((ny + g.out_h - 1) / g.out_h);
    return g;
}

// A window shape and the steps of its launches.
struct WinChoice {
    int shape, steps;
};

// The cheapest shape per step for a plate, launches of at most max_steps
// steps (win_reach rings each, one more with deviation storage).
inline WinChoice choose_window(int cls, bool gen, int nx, int ny, int reach, bool dev, int max_steps)
{
    WinChoice best{0, 1};
    double best_t = 1e300;
    for (const WinCost &c : kWinCosts[cls][gen ? 1 : 0]) {
        if (c.steps < 1 || c.steps > max_steps) continue;
        const WinGrid g = win_grid(kWinShapes[c.shape], nx, ny, c.steps * reach + (dev ? 1 : 0), c.steps);
        if (g.nb <= 0) continue;
        const double per_cu = (double)g.nb / 256.0, full = per_cu < 4.0 ? std::ceil(per_cu) : per_cu + 0.5;
        const double t = std::max((double)c.lat, c.base + c.thr * full) / c.steps;
        if (t < best_t) {
            best_t = t;
            best = WinChoice{c.shape, c.steps};
        }
    }
    return best;
}

template <class PR, int MODE, int GEN, int S = 0>
hipError_t launch_window(const GenParams &p, const WinGrid &g, int shape, hipStream_t st)
{
    if constexpr (S < kNumWinShapes) {
        constexpr WinShape w = kWinShapes[S];
        if (shape != S) return launch_window<PR, MODE, GEN, S + 1>(p, g, shape, st);
        if constexpr (win_fits<PR>(S)) {
            hipLaunchKernelGGL((window_step_kernel<PR, MODE, w.w, w.h, w.k, GEN>), dim3(g.nb),
                               dim3(w.w * w.h / w.k), 0, st, p, g);
            return hipGetLastError();
        }
    }
    return hipErrorInvalidConfiguration;
}

// Enqueue nsteps (1 or 2; 1 with j extrapolated) time steps with windows of
// shape `shape` built for `edges` (WIN_*); scratch as for general_step.
template <class PR>
hipError_t window_step(GenParams p, int edges, int shape, int nsteps, char *scratch, hipStream_t st)
{
    const int reach = p.pc ? win_reach<1>() : win_reach<0>();
    WinGrid g = win_grid(kWinShapes[shape], p.nx, p.ny, nsteps * reach + (FStore<typename PR::TF>::kDeviation ? 1 : 0),
                         nsteps);
    if (g.nb <= 0 || nsteps < 1 || nsteps > kWinMaxSteps) return hipErrorInvalidConfiguration;
    for (int s = 0; s <= nsteps; ++s)
        for (int e = 0; e < 4; ++e)
            for (int a = 0; a < 2; ++a)  // (rounded once, as the kernels' multiply-add)
                g.uw[s][e][a] = std::fma(p.val[e][a], (double)(p.step + s), p.uwb[e][a]);
    if (p.pc == 2) {
        const size_t bytes = (size_t)2 * p.nx * p.ny * sizeof(typename PR::TJ);
        const hipError_t e = hipMemcpyAsync(scratch, p.j_out, bytes, hipMemcpyDeviceToDevice, st);
        if (e != hipSuccess) return e;
        p.j_prev = scratch;
    }
    if (p.pc) return edges == WIN_GENERAL  ? launch_window<PR, 1, WIN_GENERAL>(p, g, shape, st)
                     : edges == WIN_YWALLS ? launch_window<PR, 1, WIN_YWALLS>(p, g, shape, st)
                                           : launch_window<PR, 1, WIN_PERIODIC>(p, g, shape, st);
    return edges == WIN_GENERAL  ? launch_window<PR, 0, WIN_GENERAL>(p, g, shape, st)
           : edges == WIN_YWALLS ? launch_window<PR, 0, WIN_YWALLS>(p, g, shape, st)
                                 : launch_window<PR, 0, WIN_PERIODIC>(p, g, shape, st);
}

extern template hipError_t window_step<PrecF64>(GenParams, int, int, int, char *, hipStream_t);
extern template hipError_t window_step<PrecF32>(GenParams, int, int, int, char *, hipStream_t);
extern template hipError_t window_step<PrecF32U64>(GenParams, int, int, int, char *, hipStream_t);
extern template hipError_t window_step<PrecF16>(GenParams, int, int, int, char *, hipStream_t);
extern template hipError_t window_step<PrecBF16>(GenParams, int, int, int, char *, hipStream_t);

}  // namespace lbm
