// split_plan.hpp -- how a large plate with walls or holes is shared between the
// fused step kernel and windows.
//
// Where a tile's outputs lie farther than the stencil's reach from every wall
// and hole, the fused kernel's periodic arithmetic is the general rules'
// arithmetic, and it runs those sites at its own rate; windows
// (window_kernel.hpp) run the rest. Both read the state of step n and write
// disjoint sites of the new state, whatever the steps of the launch.
#pragma once

#include <algorithm>
#include <cstring>
#include <queue>
#include <utility>
#include <vector>

#include "host_common.hpp"
#include "window_kernel.hpp"

namespace lbm {

// Smallest fused share worth its launch beside the windows'.
constexpr int kSplitMinCols = 96, kSplitMinRows = 32;

struct SplitPlan {
    bool built = false, use = false;
    bool beside = false;  // the windows run on the handle's second stream
    Shape shape{};  // of the fused share
    Rect box{};     // its part of the plate (no list)
    const int4 *fused_list = nullptr;  // or its tiles, x, columns, y0, y1
    int n_fused = 0;
    WinGrid win{};
    int win_shape = 0;
    // with j extrapolated, which has no fused form: windows of the periodic
    // form in its place (they mind no flags: a third less than the general
    // form's), inner.list = fused_list with a mask
    WinGrid inner{};
    int inner_shape = 0;
};

struct SplitEdges {
    int nx, ny;
    bool perx, pery;
    int reach;  // of a launch's steps
    int align;  // columns: a strip starts on a multiple (whole 128-byte lines)
};

// The part of the plate clear of its walls.
inline Rect split_box(const SplitEdges &e)
{
    Rect b{0, 0, e.nx, e.ny};
    if (!e.perx) {
        b.x = (e.reach + e.align - 1) / e.align * e.align;
        b.w = (e.nx - e.reach) / e.align * e.align - b.x;
    }
    if (!e.pery) {
        b.y = e.reach;
        b.h = e.ny - 2 * e.reach;
    }
    return b;
}

// The rest of the plate, at most four bands.
inline std::vector<Rect> split_frame(const SplitEdges &e, const Rect &b)
{
    std::vector<Rect> r;
    auto add = [&](int x, int y, int w, int h) {
        if (w > 0 && h > 0) r.push_back(Rect{x, y, w, h});
    };
    add(0, 0, e.nx, b.y);
    add(0, b.y + b.h, e.nx, e.ny - b.y - b.h);
    add(0, b.y, b.x, b.h);
    add(b.x + b.w, b.y, e.nx - b.x - b.w, b.h);
    return r;
}

// A plate with holes (mask [ny][nx], 0: hole). Bands of rows are grouped into
// runs whose columns (in blocks of e.align) clear of walls and holes are the same;
// a run's clear columns become strips of fused tiles (x, columns, y0, y1 in
// `tiles`), the rest of the plate rectangles for windows. Neighbouring runs
// are merged, at the cost of the columns clear in only one of them, where the
// rows a fused tile marches before its first output cost more. Tiles are cut
// to at most `slots`, one wave of blocks, where strips allow. A last strip of
// fewer than min_strip columns is left to the windows.
inline void split_mask(const SplitEdges &e, const unsigned char *mask, int strip_w, int min_strip, int slots,
                       std::vector<int4> &tiles, std::vector<Rect> &rects)
{
    constexpr int RH = 4;
    const int CW = e.align;
    const int nc = (e.nx + CW - 1) / CW, nb = (e.ny + RH - 1) / RH;
    std::vector<unsigned char> row((size_t)nb * nc, 0);  // a hole within reach in x of the block, in the band's rows
    auto mark = [&](int band, int x0, int x1) {  // columns [x0, x1), wrapped across periodic edges
        for (int x = x0; x < x1;) {
            int c = x;
            if (c < 0 || c >= e.nx) {
                if (!e.perx) {
                    ++x;
                    continue;
                }
                c = ((c % e.nx) + e.nx) % e.nx;
            }
            row[(size_t)band * nc + c / CW] = 1;
            x += std::min(CW - c % CW, e.nx - c);
        }
    };
    for (int y = 0; y < e.ny; ++y) {
        const unsigned char *m = mask + (size_t)y * e.nx;
        for (int x = 0; x < e.nx;) {
            const void *q = std::memchr(m + x, 0, e.nx - x);
            if (!q) break;
            const int a = (int)(static_cast<const unsigned char *>(q) - m);
            int b = a + 1;
            while (b < e.nx && m[b] == 0) ++b;
            mark(y / RH, a - e.reach, b + e.reach);
            x = b;
        }
    }
    // bands within reach in y, and walls
    const int db = (e.reach + RH - 1) / RH;
    const Rect box = split_box(e);
    struct Run {
        int y0, y1;
        std::vector<unsigned char> dirty;
    };
    std::vector<Run> runs;
    for (int b = 0; b < nb; ++b) {
        Run r{b * RH, std::min(e.ny, b * RH + RH), std::vector<unsigned char>(nc, 0)};
        for (int d = -db; d <= db; ++d) {
            int k = b + d;
            if (k < 0 || k >= nb) {
                if (!e.pery) continue;
                k = ((k % nb) + nb) % nb;
                // (the last band may be short: one more beyond the seam)
                for (int c = 0; c < nc; ++c) r.dirty[c] |= row[(size_t)((k + (d < 0 ? nb - 1 : 1)) % nb) * nc + c];
            }
            for (int c = 0; c < nc; ++c) r.dirty[c] |= row[(size_t)k * nc + c];
        }
        for (int c = 0; c < nc; ++c)
            if (r.y0 < box.y || r.y1 > box.y + box.h || c * CW < box.x || std::min(e.nx, c * CW + CW) > box.x + box.w)
                r.dirty[c] = 1;
        if (!runs.empty() && runs.back().dirty == r.dirty)
            runs.back().y1 = r.y1;
        else
            runs.push_back(std::move(r));
    }
    auto gain = [&](const Run &a, const Run &b) {  // block-rows saved by merging
        long long lost = 0, kept = 0;
        for (int c = 0; c < nc; ++c) {
            if (!a.dirty[c] && b.dirty[c]) lost += a.y1 - a.y0;
            if (a.dirty[c] && !b.dirty[c]) lost += b.y1 - b.y0;
            if (!a.dirty[c] && !b.dirty[c]) kept += 2 * e.reach;
        }
        return kept - lost;
    };
    // The pair with the largest gain first, the first of equal ones. A merge
    // changes the gains of the two pairs beside it only, so a heap of the pairs'
    // gains (stale entries are passed over) plans 8192^2 nodes with 4096 small
    // holes in 25 ms, where a scan of every pair per merge took 0.86 s; 16384^2
    // with 8192 take 0.1 s.
    const int n_runs = (int)runs.size();
    std::vector<int> next(n_runs), prev(n_runs);
    std::vector<long long> g(n_runs, 0);  // gain of a run with the next one; 0: none, or merged away
    std::priority_queue<std::pair<long long, int>> heap;  // (gain, -run)
    auto price = [&](int i) {
        if (i < 0) return;
        g[i] = next[i] < n_runs ? gain(runs[i], runs[next[i]]) : 0;
        if (g[i] > 0) heap.push({g[i], -i});
    };
    for (int i = 0; i < n_runs; ++i) next[i] = i + 1, prev[i] = i - 1;
    for (int i = 0; i + 1 < n_runs; ++i) price(i);
    while (!heap.empty()) {
        const long long top = heap.top().first;
        const int i = -heap.top().second;
        heap.pop();
        if (top != g[i]) continue;
        const int j = next[i];
        runs[i].y1 = runs[j].y1;
        for (int c = 0; c < nc; ++c) runs[i].dirty[c] |= runs[j].dirty[c];
        runs[j].y0 = runs[j].y1;  // (empty: merged away)
        g[j] = 0;
        next[i] = next[j];
        if (next[i] < n_runs) prev[next[i]] = i;
        price(i);
        price(prev[i]);
    }
    runs.erase(std::remove_if(runs.begin(), runs.end(), [](const Run &r) { return r.y0 == r.y1; }), runs.end());
    // clear columns of each run: strips
    struct Strip {
        int x, w, y0, y1;
    };
    std::vector<Strip> strips;
    for (Run &r : runs) {
        for (int c = 0; c < nc;) {
            if (r.dirty[c]) {
                ++c;
                continue;
            }
            int d = c;
            while (d < nc && !r.dirty[d]) ++d;
            const int x0 = c * CW, x1 = std::min(e.nx, d * CW);
            if (x1 - x0 < kSplitMinCols || r.y1 - r.y0 < kSplitMinRows) {
                for (int k = c; k < d; ++k) r.dirty[k] = 1;
            } else {
                for (int x = x0; x < x1; x += strip_w) {
                    if (x > x0 && x1 - x < min_strip) {
                        for (int k = x / CW; k < d; ++k) r.dirty[k] = 1;
                        break;
                    }
                    strips.push_back(Strip{x, std::min(strip_w, x1 - x), r.y0, r.y1});
                }
            }
            c = d;
        }
        for (int c = 0; c < nc;) {
            if (!r.dirty[c]) {
                ++c;
                continue;
            }
            int d = c;
            while (d < nc && r.dirty[d]) ++d;
            rects.push_back(Rect{c * CW, r.y0, std::min(e.nx, d * CW) - c * CW, r.y1 - r.y0});
            c = d;
        }
    }
    // the shortest segments that fit the wave
    auto count = [&](int rows) {
        long long n = 0;
        for (const Strip &s : strips) n += (s.y1 - s.y0 + rows - 1) / rows;
        return n;
    };
    int lo = 8, hi = std::max(8, e.ny);
    while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (count(mid) <= slots)
            hi = mid;
        else
            lo = mid + 1;
    }
    for (const Strip &s : strips) {
        const int n = (s.y1 - s.y0 + lo - 1) / lo;
        for (int q = 0; q < n; ++q)
            tiles.push_back(int4{s.x, s.w, s.y0 + (int)((long long)q * (s.y1 - s.y0) / n),
                                 s.y0 + (int)((long long)(q + 1) * (s.y1 - s.y0) / n)});
    }
    // row by row, so that horizontal neighbours share an XCD's L2
    std::stable_sort(tiles.begin(), tiles.end(), [](const int4 &a, const int4 &b) { return a.z < b.z; });
}

// The rectangles' windows of at most mw x mh outputs that hold material.
inline void split_windows(int nx, const unsigned char *mask, const std::vector<Rect> &rects, int mw, int mh,
                          std::vector<int4> &list)
{
    for (const Rect &r : rects) {
        const WinRegion g = win_region(r, mw, mh, 0);
        for (int y = r.y; y < r.y + r.h; y += g.out_h)
            for (int x = r.x; x < r.x + r.w; x += g.out_w) {
                const int w = std::min(g.out_w, r.x + r.w - x), h = std::min(g.out_h, r.y + r.h - y);
                bool any = false;
                for (int k = y; k < y + h && !any; ++k) any = std::memchr(mask + (size_t)k * nx + x, 1, w) != nullptr;
                if (any) list.push_back(int4{x, y, w, h});
            }
    }
}

}  // namespace lbm
