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
// or more dependent rows: 64^2 FP64 4.4 us (12.3), 256^2 FP32_U64 5.1 (16.4),
// 512^2 FP32_U64 9.5 (19.5), between y walls 10.9 (23.6); 100 x 150 with a hole
// FP64 8.3 (29.1 with the 2D tiles these replace, which spent 1500 of 2500
// vector instructions on index arithmetic, beside a fused share).
#pragma once

#include <algorithm>
#include <cmath>
#include <vector>

#include "../../include/lbm_solid.h"
#include "step_kernel.hpp"

namespace lbm {

enum : int { EDGE_XMIN = 0, EDGE_XMAX = 1, EDGE_YMIN = 2, EDGE_YMAX = 3 };

// Plate, state and edges of a window launch.
struct GenParams {
    const void *f_in, *u_in, *j_in;  // state n
    void *f_out, *u_out, *j_out;     // state n + 1
    const void *j_prev;              // j_{n-1} (j-extrapolation only)
    int nx, ny;
    long long plane;
    double omega, lam, mu, bx, by;  // lattice units
    int bc[4];                      // rule of each edge (BC_*), EDGE_* order
    double val[4][2];               // j* or T* of each edge, lattice units
    double uwb[4][2];               // momentum walls: displacement uwb + j* n at step n
    double f_scale, f_inv_scale;
    long long step;                 // index n of the input state
    int sr;
    unsigned long long seed;
    int pc;  // explicit (0), predictor-corrector (1), j extrapolated for the predictor (2)
    unsigned *flag;
    const unsigned char *mask;  // [ny][nx]: 1 material, 0 hole; nullptr: no holes
};

// D2Q9 of this implementation (see lattice.hpp)
__device__ constexpr int kGx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int kGy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
__device__ constexpr int kGopp[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};

// Ghost value k = 1 or 2 spacings beyond a wall from the node next to it
// (a): at a momentum wall the straight line through the wall displacement
// uw and a (2 uw - a, then 4 uw - 3 a), at a traction wall the value a.
template <class TU>
__device__ __forceinline__ TU gen_ghost(int kind, TU uw, TU a, int k)
{
    if (kind == BC_NEUMANN) return a;
    return k == 1 ? TU(2) * uw - a : TU(4) * uw - TU(3) * a;
}

constexpr int kWinMaxSteps = 2;  // steps per launch at most

// A rectangle of a plate tiled with windows: out_w x out_h nodes per block,
// nbx blocks per row of blocks, the first one block `first` of the launch.
struct WinRegion {
    int x, y, w, h, out_w, out_h, nbx, first;
};
constexpr int kWinRegions = 4;  // regions of a launch without a list: a frame's bands

// Geometry of a launch: blocks, steps, the output rectangles (a list in device
// memory, x, y, w, h per block, or regions); the momentum walls' displacement
// at steps n .. n + nsteps.
struct WinGrid {
    int nb, nsteps, n_regions;
    WinRegion reg[kWinRegions];
    const int4 *list;
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
    static constexpr int CAP = N / 4;  // wall nodes handled at once
    static_assert(N <= 2048, "LDS index in 11 bits");
    static_assert((WW & (WW - 1)) == 0 && BLOCK % WW == 0 && RS * K == WH, "window shape");
    struct Lds {
        TU u[2][N];
        TC k[4][N];
        TC f[8][N];  // directions 1..8
        unsigned char hole[GEN == WIN_GENERAL ? N : 1];
        // WIN_GENERAL: nodes beside a wall or hole (LDS index, flags << 11; 0:
        // none), the moments of their populations, and how many there are
        unsigned wn[GEN == WIN_GENERAL ? CAP : 1];
        TC wm[GEN == WIN_GENERAL ? 4 : 1][GEN == WIN_GENERAL ? CAP : 1];
        int nw;
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
        const TC Hn[4] = {n ? H[0] : TC(0), n ? TC(0) : H[1], n ? H[2] : TC(0), n ? TC(0) : H[3]};
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

    // y walls: the values the wall returns to its node i, into the slots the
    // pull reads, in the fused kernel's form. m: r, Pxx of the node's
    // populations, whose values after the collision are in the LDS.
    __device__ __forceinline__ void wall_row(int i, unsigned fl, TC r, TC pxx)
    {
        const bool top = opaque(fl) & YH;
        const int g = top ? i + WW : i - WW;
        const double val[2] = {top ? p.val[EDGE_YMAX][0] : p.val[EDGE_YMIN][0],
                               top ? p.val[EDGE_YMAX][1] : p.val[EDGE_YMIN][1]};
        const TC fco[3] = {L.f[top ? 1 : 3][i], L.f[top ? 4 : 6][i], L.f[top ? 5 : 7][i]};
        TC w[3];
        wall_populations(top, top ? p.bc[EDGE_YMAX] : p.bc[EDGE_YMIN], fco, val, r, pxx,
                         TC(0.5) * (L.k[1][i] + L.k[1][g]), TC(0.5) * (L.k[3][i] + L.k[3][g]), w);
        // returned as 4, 7, 8 (top) or 2, 5, 6
        L.f[top ? 3 : 1][g] = w[0];
        L.f[top ? 6 : 4][top ? g + 1 : g - 1] = w[1];
        L.f[top ? 7 : 5][top ? g - 1 : g + 1] = w[2];
    }

    // Value returned for the link o of node i if it leaves through a wall or
    // into a hole, into the slot the pull reads (m: r, Pxx, Pyy, Pxy of the
    // node's populations, whose values after the collision are in the LDS).
    // Bounce-back with the wall momentum (eq. (25)) if a crossed wall is a
    // momentum wall (the mean j* if both are); otherwise anti-bounce-back (eq.
    // (26)) with r_bd and Pbar* at the node: each traction wall's column of
    // Pbar* is -s T* + K n, K at the wall the mean of the node's and the one
    // beyond it (a ghost node, or at a hole, T* = 0, the hole K the node
    // sees); a tangential entry keeps the populations' second moment, and at a
    // corner the off-diagonal entry is the mean of both walls' values.
    __device__ __forceinline__ void link(int o, int i, unsigned fl, const TC m[4], const double uw[4][2])
    {
        const int ox = (int)((0x20919u >> (2 * o)) & 3u) - 1, oy = (int)((0x2865u >> (2 * o)) & 3u) - 1;
        const bool hole = near(fl, o);
        const bool bx = ox != 0 && (fl & (ox < 0 ? XL : XH)), by = oy != 0 && (fl & (oy < 0 ? YL : YH));
        if (!(hole || bx || by)) return;
        // holes beside the node across x and y; a link into a hole crosses the
        // wall its axis step enters, or both through a hole corner
        const bool nx = ox != 0 && near(fl, ox > 0 ? 1 : 3), ny = oy != 0 && near(fl, oy > 0 ? 2 : 4);
        const int sx = (hole ? nx || !ny : bx) ? ox : 0, sy = (hole ? ny || !nx : by) ? oy : 0;
        const bool lx = ox < 0, ly = oy < 0;
        const bool ddx = !hole && sx != 0 && (lx ? p.bc[EDGE_XMIN] : p.bc[EDGE_XMAX]) == BC_DIRICHLET;
        const bool ddy = !hole && sy != 0 && (ly ? p.bc[EDGE_YMIN] : p.bc[EDGE_YMAX]) == BC_DIRICHLET;
        // j* or T* of the edges (selected from scalars: an index would load)
        const double vx0 = lx ? p.val[EDGE_XMIN][0] : p.val[EDGE_XMAX][0];
        const double vx1 = lx ? p.val[EDGE_XMIN][1] : p.val[EDGE_XMAX][1];
        const double vy0 = ly ? p.val[EDGE_YMIN][0] : p.val[EDGE_YMAX][0];
        const double vy1 = ly ? p.val[EDGE_YMIN][1] : p.val[EDGE_YMAX][1];
        const TC w = o < 5 ? TC(1.0 / 9.0) : TC(1.0 / 36.0), cx = TC(ox), cy = TC(oy), fco = L.f[o - 1][i];
        TC val;
        if (ddx || ddy) {
            const double sc = ddx && ddy ? 0.5 : 1.0;
            const TC jx = TC(sc * ((ddx ? vx0 : 0.0) + (ddy ? vy0 : 0.0)));
            const TC jy = TC(sc * ((ddx ? vx1 : 0.0) + (ddy ? vy1 : 0.0)));
            val = fco - TC(6) * w * (cx * jx + cy * jy);
        } else {
            TC H[4] = {TC(0), TC(0), TC(0), TC(0)}, kh[4];
            if (fl >> 8) grad(i, fl, uw, H);
            TC Pxx = m[1], Pyy = m[2], Pxy = m[3], qx1 = TC(0);
            if (sx) {
                TC k0 = L.k[0][i + sx], k2 = L.k[2][i + sx];
                if (nx) {
                    k_hole(H, 0, kh);
                    k0 = kh[0];
                    k2 = kh[2];
                }
                Pxx = -cx * TC(hole ? 0.0 : vx0) + TC(0.5) * (L.k[0][i] + k0);
                Pxy = qx1 = -cx * TC(hole ? 0.0 : vx1) + TC(0.5) * (L.k[2][i] + k2);
            }
            if (sy) {
                TC k1 = L.k[1][i + sy * WW], k3 = L.k[3][i + sy * WW];
                if (ny) {
                    k_hole(H, 1, kh);
                    k1 = kh[1];
                    k3 = kh[3];
                }
                const TC qy0 = -cy * TC(hole ? 0.0 : vy0) + TC(0.5) * (L.k[1][i] + k1);
                Pyy = -cy * TC(hole ? 0.0 : vy1) + TC(0.5) * (L.k[3][i] + k3);
                Pxy = sx ? TC(0.5) * (qx1 + qy0) : qy0;
            }
            const TC r = m[0], third = TC(1) / TC(3);
            const TC axx = Pxx - r * third, ayy = Pyy - r * third;
            const TC q = axx * cx * cx + TC(2) * Pxy * cx * cy + ayy * cy * cy - (axx + ayy) * third;
            val = -fco + TC(2) * w * (r + TC(4.5) * q);
        }
        // the opposite link's plane (d - 1), at the site this one leads to
        L.f[(0x54761032u >> (4 * (o - 1))) & 7u][i + oy * WW + ox] = val;
    }

    // the output rectangle: ow x oh nodes from (x0, y0)
    __device__ __forceinline__ void run(const WinGrid &g, int x0, int y0, int ow, int oh)
    {
        const size_t pl = (size_t)p.plane;
        const TF *__restrict__ fin = static_cast<const TF *>(p.f_in);
        const TU *__restrict__ uin = static_cast<const TU *>(p.u_in);
        const TJ *__restrict__ jin = static_cast<const TJ *>(p.j_in);
        const int nx = p.nx, ny = p.ny;
        const int h = g.nsteps * HS + (DEV ? 1 : 0);
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
        int pos[K];  // WIN_GENERAL: place in the list of wall nodes
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
        int nw = 0;
        if constexpr (GEN == WIN_GENERAL) {
            if (threadIdx.x == 0) L.nw = 0;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < K; ++k) {
                pos[k] = -1;
                if ((fl[k] & NODE) && ((fl[k] & EDGE) || (fl[k] >> 8))) pos[k] = atomicAdd(&L.nw, 1);
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
            if (GEN == WIN_GENERAL && s == 0) nw = L.nw;
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
            TC m[K][4];
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
                if (GEN == WIN_GENERAL || (GEN == WIN_YWALLS && (fl[k] & EDGE))) {
                    const TC *fk = f[k];
                    m[k][0] = r;
                    m[k][1] = pxx;
                    m[k][2] = (fk[2] + fk[4]) + ((fk[5] + fk[6]) + (fk[7] + fk[8]));
                    m[k][3] = (fk[5] - fk[6]) + (fk[7] - fk[8]);
                    if constexpr (GEN == WIN_YWALLS) wall_row(i, fl[k], r, pxx);
                }
                f[k][0] = fc[0];
            }
            if constexpr (GEN == WIN_GENERAL) {
                // The links of the nodes beside walls and holes, one per
                // thread: an x wall puts one such node in every row of the
                // window, and run where it lies each wave would go through all
                // its links for one lane (the windows of the 4096^2 FP32_U64
                // plate with a hole: 113 against 147 us per two steps).
                for (int base = 0; base < nw; base += CAP) {
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const int q = pos[k] - base;
                        if (pos[k] < 0 || q < 0 || q >= CAP) continue;
                        L.wn[q] = row_in(k, d + 2) ? (unsigned)((r0 + k * RS) * WW + lx) | (fl[k] << 11) : 0u;
#pragma unroll
                        for (int c = 0; c < 4; ++c) L.wm[c][q] = m[k][c];
                    }
                    __syncthreads();
                    for (int q = threadIdx.x; q < 8 * min(CAP, nw - base); q += BLOCK) {
                        const int n = q >> 3;
                        const unsigned e = L.wn[n];
                        const TC mq[4] = {L.wm[0][n], L.wm[1][n], L.wm[2][n], L.wm[3][n]};
                        if (e) link((int)opaque((q & 7) + 1), (int)(e & 2047u), e >> 11, mq, uw);
                    }
                    if (base + CAP < nw) __syncthreads();
                }
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

// One block per output rectangle. Blocks are dealt round-robin to the 8 XCDs;
// the remap gives each XCD a run of consecutive rectangles, so the windows of
// horizontal neighbours overlap in one L2.
template <class PR, int MODE, int WW, int WH, int K, int GEN>
__global__ void __launch_bounds__(WW *WH / K) window_step_kernel(const GenParams p, const WinGrid g)
{
    using W = Window<PR, MODE, WW, WH, K, GEN>;
    __shared__ typename W::Lds lds;
    const int bid = blockIdx.x;
    const int xq = g.nb >> 3, xr = g.nb & 7;
    const int xcd = bid & 7, loc = bid >> 3;
    const int tile = xcd * xq + min(xcd, xr) + loc;
    int x0, y0, ow, oh;
    if (g.list) {
        const int4 e = g.list[tile];
        x0 = e.x, y0 = e.y, ow = e.z, oh = e.w;
    } else {
        WinRegion r = g.reg[0];
        if (g.n_regions > 1)
            for (int k = 1; k < g.n_regions; ++k)
                if (tile >= g.reg[k].first) r = g.reg[k];
        const int t = tile - r.first, ty = t / r.nbx, tx = t - ty * r.nbx;
        x0 = r.x + tx * r.out_w;
        y0 = r.y + ty * r.out_h;
        ow = min(r.out_w, r.x + r.w - x0);
        oh = min(r.out_h, r.y + r.h - y0);
    }
    W w(p, lds);
    w.run(g, x0, y0, ow, oh);
}

// Window shapes: columns, rows, rows per thread.
struct WinShape {
    int w, h, k;
};
constexpr WinShape kWinShapes[] = {{16, 16, 1}, {32, 16, 1}, {32, 32, 1}, {64, 16, 1}, {64, 32, 2}, {32, 32, 2}};
constexpr int kNumWinShapes = (int)(sizeof(kWinShapes) / sizeof(kWinShapes[0]));

// Cost of a launch of n blocks with a shape and a number of steps, in us:
// lat for a few blocks to lat1 for one per compute unit, base + thr per block
// on the fullest compute unit beyond (its number is rounded up, half way below
// two per compute unit, not at all from four). Measured with plates of 16 to 2048 full
// windows, per class (double; float; float with a double displacement; 16-bit
// storage) and kind of edges (WIN_*). A two-step
// launch pays where the plate is small enough that the launch itself and the
// load of the state count (64 x 64 FP64: 4.4 us per step with 32 x 32 windows of
// two steps, 4.7 with 16 x 16 and 7.7 with 32 x 32 windows of one).
struct WinCost {
    int shape, steps;
    float lat, lat1, base, thr;
};
constexpr int kNumWinCosts = 9;
constexpr WinCost kWinCosts[4][3][kNumWinCosts] = {
    {{{0, 1, 4.7f, 4.8f, 3.8f, 0.9f}, {1, 1, 5.4f, 6.1f, 2.9f, 2.4f}, {2, 1, 7.7f, 9.6f, 3.7f, 7.2f},
      {2, 2, 8.8f, 10.2f, 2.8f, 7.6f}, {3, 1, 6.5f, 8.8f, 2.2f, 5.8f}, {5, 1, 7.8f, 9.7f, 3.4f, 7.6f},
      {5, 2, 9.1f, 10.6f, 3.2f, 7.9f}},
     {{0, 1, 5.8f, 5.8f, 4.3f, 1.0f}, {1, 1, 6.3f, 6.3f, 3.0f, 2.5f}, {2, 1, 8.2f, 9.8f, 3.7f, 7.4f},
      {2, 2, 9.4f, 10.4f, 3.2f, 7.7f}, {3, 1, 7.0f, 8.8f, 2.0f, 6.0f}, {5, 1, 9.3f, 10.8f, 4.2f, 8.0f},
      {5, 2, 11.1f, 11.8f, 3.7f, 8.6f}},
     {{0, 1, 7.1f, 7.1f, 4.7f, 1.6f}, {1, 1, 7.8f, 8.2f, 4.9f, 4.2f}, {2, 1, 12.4f, 15.8f, 5.9f, 11.5f},
      {2, 2, 16.8f, 19.6f, 8.7f, 13.3f}, {3, 1, 11.1f, 14.2f, 7.0f, 9.3f}, {5, 1, 12.0f, 13.8f, 5.8f, 9.2f},
      {5, 2, 16.2f, 17.1f, 10.3f, 10.4f}}},
    {{{0, 1, 4.3f, 4.3f, 3.7f, 0.5f}, {1, 1, 4.5f, 4.8f, 3.6f, 1.0f}, {2, 1, 5.7f, 6.5f, 2.5f, 3.2f},
      {2, 2, 6.5f, 7.1f, 3.3f, 3.0f}, {3, 1, 5.1f, 5.9f, 2.3f, 2.5f}, {4, 1, 7.3f, 10.2f, 5.6f, 7.1f},
      {4, 2, 8.7f, 11.3f, 2.3f, 8.0f}, {5, 1, 6.2f, 7.0f, 2.5f, 3.4f}, {5, 2, 7.3f, 7.8f, 3.1f, 3.4f}},
     {{0, 1, 5.3f, 5.3f, 4.3f, 0.5f}, {1, 1, 5.5f, 5.5f, 3.4f, 1.3f}, {2, 1, 6.3f, 6.8f, 2.5f, 4.1f},
      {2, 2, 7.7f, 7.8f, 2.9f, 4.9f}, {3, 1, 5.7f, 6.1f, 2.1f, 2.8f}, {4, 1, 8.2f, 10.8f, 6.1f, 7.5f},
      {4, 2, 10.0f, 11.9f, 3.0f, 8.5f}, {5, 1, 7.5f, 7.8f, 3.2f, 3.5f}, {5, 2, 9.5f, 9.5f, 2.3f, 4.2f}},
     {{0, 1, 6.7f, 6.7f, 4.9f, 0.9f}, {1, 1, 6.9f, 6.9f, 3.5f, 2.1f}, {2, 1, 8.2f, 8.8f, 5.0f, 5.1f},
      {2, 2, 10.9f, 11.1f, 7.6f, 6.3f}, {3, 1, 7.5f, 8.2f, 4.9f, 4.4f}, {4, 1, 11.6f, 13.8f, 5.4f, 9.8f},
      {4, 2, 15.5f, 17.5f, 10.3f, 10.2f}, {5, 1, 10.2f, 10.6f, 6.4f, 6.2f}, {5, 2, 13.7f, 13.7f, 9.0f, 7.9f}}},
    {{{0, 1, 4.4f, 4.4f, 3.8f, 0.5f}, {1, 1, 4.6f, 5.0f, 3.9f, 1.0f}, {2, 1, 5.9f, 7.0f, 2.5f, 3.7f},
      {2, 2, 6.9f, 7.5f, 3.3f, 3.4f}, {3, 1, 5.2f, 6.5f, 2.2f, 2.9f}, {4, 1, 8.2f, 11.5f, 0.1f, 11.0f},
      {4, 2, 9.8f, 12.8f, 2.3f, 9.2f}, {5, 1, 6.4f, 7.5f, 2.7f, 3.8f}, {5, 2, 7.6f, 8.2f, 3.2f, 3.8f}},
     {{0, 1, 5.5f, 5.5f, 4.3f, 0.6f}, {1, 1, 5.6f, 5.6f, 3.5f, 1.4f}, {2, 1, 6.5f, 7.2f, 2.5f, 4.5f},
      {2, 2, 8.0f, 8.2f, 3.2f, 5.2f}, {3, 1, 5.8f, 6.5f, 2.4f, 3.7f}, {4, 1, 8.9f, 12.1f, 0.2f, 11.5f},
      {4, 2, 11.0f, 13.4f, 2.6f, 9.9f}, {5, 1, 7.7f, 8.2f, 3.7f, 3.7f}, {5, 2, 9.8f, 9.8f, 2.6f, 4.6f}},
     {{0, 1, 6.8f, 6.8f, 4.9f, 1.0f}, {1, 1, 7.0f, 7.0f, 3.7f, 2.3f}, {2, 1, 8.5f, 9.3f, 5.0f, 5.4f},
      {2, 2, 11.3f, 11.6f, 7.8f, 6.7f}, {3, 1, 7.7f, 8.6f, 5.3f, 4.6f}, {4, 1, 12.5f, 15.4f, 2.4f, 12.9f},
      {4, 2, 16.6f, 19.0f, 10.7f, 11.4f}, {5, 1, 10.5f, 11.0f, 6.7f, 6.5f}, {5, 2, 14.2f, 14.2f, 9.1f, 8.3f}}},
    {{{0, 1, 4.5f, 4.6f, 3.8f, 0.6f}, {1, 1, 4.5f, 4.8f, 3.0f, 1.3f}, {2, 1, 5.8f, 6.6f, 2.5f, 4.2f},
      {2, 2, 7.5f, 8.0f, 2.3f, 5.7f}, {3, 1, 5.3f, 6.3f, 3.4f, 3.3f}, {4, 1, 8.6f, 10.5f, 3.4f, 7.9f},
      {4, 2, 10.6f, 13.2f, 3.7f, 9.5f}, {5, 1, 6.9f, 7.5f, 3.3f, 3.6f}, {5, 2, 8.6f, 9.0f, 3.6f, 4.3f}},
     {{0, 1, 6.3f, 6.3f, 5.1f, 0.6f}, {1, 1, 6.1f, 6.1f, 3.4f, 1.6f}, {2, 1, 7.0f, 7.3f, 3.2f, 4.6f},
      {2, 2, 9.4f, 9.4f, 3.4f, 6.0f}, {3, 1, 6.3f, 6.5f, 3.4f, 3.5f}, {4, 1, 9.6f, 11.3f, 3.4f, 8.6f},
      {4, 2, 12.1f, 14.2f, 3.9f, 10.5f}, {5, 1, 8.9f, 8.9f, 3.8f, 3.9f}, {5, 2, 11.2f, 11.2f, 3.8f, 4.8f}},
     {{0, 1, 8.2f, 8.2f, 6.2f, 1.1f}, {1, 1, 8.1f, 8.1f, 3.9f, 2.6f}, {2, 1, 9.7f, 10.2f, 5.7f, 6.1f},
      {2, 2, 12.9f, 13.0f, 7.6f, 8.1f}, {3, 1, 9.0f, 9.6f, 5.7f, 5.5f}, {4, 1, 15.6f, 18.6f, 7.5f, 12.6f},
      {4, 2, 20.0f, 23.1f, 11.9f, 14.5f}, {5, 1, 12.4f, 12.4f, 7.3f, 7.2f}, {5, 2, 15.9f, 15.9f, 10.3f, 9.3f}}},
};

// Class of a precision in kWinCosts.
inline int win_class(lbm_precision p)
{
    return p == LBM_FP64 ? 0 : p == LBM_FP32 ? 1 : p == LBM_FP32_U64 ? 2 : 3;
}

template <class PR, int MODE, int GEN>
constexpr bool win_fits(int s)
{
    constexpr int tu = (int)sizeof(typename PR::TU), tc = (int)sizeof(typename PR::TC);
    const int n = kWinShapes[s].w * kWinShapes[s].h;
    return n * (2 * tu + 12 * tc) + (GEN == WIN_GENERAL ? n + n / 4 * (4 + 4 * tc) : 0) + 64 <= 160 * 1024;
}

// Output nodes of a window with rings h on each side (0: none).
inline int win_out(int n, int h) { return std::max(0, n - 2 * h); }

// A rectangle of nodes.
struct Rect {
    int x, y, w, h;
};

// Split of a rectangle into output rectangles of at most mw x mh nodes, evened
// out.
inline WinRegion win_region(const Rect &r, int mw, int mh, int first)
{
    const int nx = (r.w + mw - 1) / mw, ny = (r.h + mh - 1) / mh;
    WinRegion g{r.x, r.y, r.w, r.h, (r.w + nx - 1) / nx, (r.h + ny - 1) / ny, 0, first};
    g.nbx = (r.w + g.out_w - 1) / g.out_w;
    return g;
}
inline int win_blocks(const WinRegion &g) { return g.nbx * ((g.h + g.out_h - 1) / g.out_h); }

// A window shape and the steps of its launches.
struct WinChoice {
    int shape, steps;
};

// The cheapest shape per step for n_rects rectangles of a plate, launches of
// min_steps to max_steps steps (reach rings each, one more with deviation
// storage) on a device of `cus` compute units. Called for each lbm_step: no
// allocation.
inline WinChoice choose_window(int cus, int cls, int edges, const Rect *rects, int n_rects, int reach, bool dev,
                               int min_steps, int max_steps)
{
    WinChoice best{0, min_steps};
    double best_t = 1e300;
    for (const WinCost &c : kWinCosts[cls][edges]) {
        if (c.steps < min_steps || c.steps > max_steps) continue;
        const int h = c.steps * reach + (dev ? 1 : 0);
        const int mw = win_out(kWinShapes[c.shape].w, h), mh = win_out(kWinShapes[c.shape].h, h);
        if (!mw || !mh) continue;
        double nb = 0;
        for (int k = 0; k < n_rects; ++k) nb += win_blocks(win_region(rects[k], mw, mh, 0));
        const double per_cu = nb / cus, full = per_cu < 2.0   ? 0.5 * (per_cu + std::ceil(per_cu))
                                                       : per_cu < 4.0 ? std::ceil(per_cu)
                                                                      : per_cu;
        const double one = c.lat + (c.lat1 - c.lat) * std::min(1.0, per_cu);
        const double t = (per_cu <= 1.0 ? one : std::max(one, c.base + c.thr * full)) / c.steps;
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
        if constexpr (win_fits<PR, MODE, GEN>(S)) {
            hipLaunchKernelGGL((window_step_kernel<PR, MODE, w.w, w.h, w.k, GEN>), dim3(g.nb),
                               dim3(w.w * w.h / w.k), 0, st, p, g);
            return hipGetLastError();
        }
    }
    return hipErrorInvalidConfiguration;
}

// Enqueue g.nsteps (1 or 2; 1 with j extrapolated) time steps over the
// launch's rectangles (g.nb, g.nsteps and the list or the regions are set)
// with windows of shape `shape` built for `edges` (WIN_*).
template <class PR>
hipError_t window_step(const GenParams &p, WinGrid g, int edges, int shape, hipStream_t st)
{
    if (g.nb <= 0) return hipSuccess;
    if (g.nsteps < 1 || g.nsteps > kWinMaxSteps) return hipErrorInvalidConfiguration;
    for (int s = 0; s <= g.nsteps; ++s)
        for (int e = 0; e < 4; ++e)
            for (int a = 0; a < 2; ++a)  // (rounded once, as the kernels' multiply-add)
                g.uw[s][e][a] = std::fma(p.val[e][a], (double)(p.step + s), p.uwb[e][a]);
    if (p.pc) return edges == WIN_GENERAL  ? launch_window<PR, 1, WIN_GENERAL>(p, g, shape, st)
                     : edges == WIN_YWALLS ? launch_window<PR, 1, WIN_YWALLS>(p, g, shape, st)
                                           : launch_window<PR, 1, WIN_PERIODIC>(p, g, shape, st);
    return edges == WIN_GENERAL  ? launch_window<PR, 0, WIN_GENERAL>(p, g, shape, st)
           : edges == WIN_YWALLS ? launch_window<PR, 0, WIN_YWALLS>(p, g, shape, st)
                                 : launch_window<PR, 0, WIN_PERIODIC>(p, g, shape, st);
}

extern template hipError_t window_step<PrecF64>(const GenParams &, WinGrid, int, int, hipStream_t);
extern template hipError_t window_step<PrecF32>(const GenParams &, WinGrid, int, int, hipStream_t);
extern template hipError_t window_step<PrecF32U64>(const GenParams &, WinGrid, int, int, hipStream_t);
extern template hipError_t window_step<PrecF16>(const GenParams &, WinGrid, int, int, hipStream_t);
extern template hipError_t window_step<PrecBF16>(const GenParams &, WinGrid, int, int, hipStream_t);

}  // namespace lbm
