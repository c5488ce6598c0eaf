"""Host planning of plates with holes (no GPU; csrc/split_plan.hpp compiled for
the host alone): the fused tiles and the windows' rectangles cover every node
once, no fused tile lies within the stencil's reach of a wall or hole, and a
plan's time grows with the plate, not with the square of its rows."""
import ctypes
import os
import subprocess
import time

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdlib>
#include "split_plan.hpp"
static long news = 0;
void *operator new(size_t n) { ++news; return std::malloc(n); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
// shape and steps chosen for n rectangles of w x h nodes, and the host allocations made for it
extern "C" long choose(int cus, int cls, int edges, int w, int h, int n, int *shape, int *steps)
{
    std::vector<lbm::Rect> r(n, lbm::Rect{0, 0, w, h});
    const long before = news;
    const lbm::WinChoice c = lbm::choose_window(cus, cls, edges, r.data(), n, 5, cls == 3, 1, lbm::kWinMaxSteps);
    *shape = c.shape;
    *steps = c.steps;
    return news - before;
}
// tiles (x, columns, y0, y1) and rectangles (x, y, w, h), at most cap each
extern "C" void plan_mask(int nx, int ny, int perx, int pery, int reach, int align, const unsigned char *mask,
                          int strip_w, int min_strip, int slots, int cap, int *tiles, int *n_tiles, int *rects, int *n_rects)
{
    const lbm::SplitEdges e{nx, ny, perx != 0, pery != 0, reach, align};
    std::vector<int4> t;
    std::vector<lbm::Rect> r;
    lbm::split_mask(e, mask, strip_w, min_strip, slots, t, r);
    *n_tiles = (int)t.size();
    *n_rects = (int)r.size();
    for (int k = 0; k < std::min(cap, *n_tiles); ++k) {
        const int v[4] = {t[k].x, t[k].y, t[k].z, t[k].w};
        std::copy(v, v + 4, tiles + 4 * k);
    }
    for (int k = 0; k < std::min(cap, *n_rects); ++k) {
        const int v[4] = {r[k].x, r[k].y, r[k].w, r[k].h};
        std::copy(v, v + 4, rects + 4 * k);
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text(SOURCE)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "paper_2208_13769_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def _plan(lib, mask, perx, pery, reach, align, strip_w, slots, min_strip=0):
    ny, nx = mask.shape
    cap = mask.size // 8 + 4096
    tiles, rects = np.zeros((cap, 4), np.int32), np.zeros((cap, 4), np.int32)
    nt, nr = ctypes.c_int(), ctypes.c_int()
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    t0 = time.perf_counter()
    lib.plan_mask(nx, ny, int(perx), int(pery), reach, align, ptr(mask), strip_w, min_strip, slots, cap, ptr(tiles),
                  ctypes.byref(nt), ptr(rects), ctypes.byref(nr))
    dt = time.perf_counter() - t0
    assert nt.value <= cap and nr.value <= cap
    return tiles[:nt.value], rects[:nr.value], dt


def _scattered(nx, ny, rng, holes, size):
    m = np.ones((ny, nx), np.uint8)
    for x, y in zip(rng.integers(0, nx, holes), rng.integers(0, ny, holes)):
        w, h = rng.integers(2, size + 1, 2)
        m[y:y + h, x:x + w] = 0
    return m


def _near(mask, perx, pery, reach):
    """Nodes within `reach` of a hole in both coordinates."""
    out = np.zeros(mask.shape, bool)
    ny, nx = mask.shape
    for y, x in np.argwhere(mask == 0):
        ys, xs = np.arange(y - reach, y + reach + 1), np.arange(x - reach, x + reach + 1)
        ys = ys % ny if pery else ys[(ys >= 0) & (ys < ny)]
        xs = xs % nx if perx else xs[(xs >= 0) & (xs < nx)]
        out[np.ix_(ys, xs)] = True
    return out


@pytest.mark.parametrize("seed", range(24))
def test_plans_cover_the_plate_clear_of_walls_and_holes(lib, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    nx, ny = int(rng.integers(150, 700)), int(rng.integers(60, 500))
    perx, pery = bool(rng.integers(2)), bool(rng.integers(2))
    reach, align = int(rng.choice([3, 5, 6, 10])), int(rng.choice([16, 32]))
    strip_w, slots = int(rng.choice([64, 96, 224])), int(rng.choice([1, 16, 512]))
    mask = _scattered(nx, ny, rng, int(rng.integers(1, 12)), 40)
    min_strip = 32 if seed % 3 == 0 else 0
    tiles, rects, _ = _plan(lib, mask, perx, pery, reach, align, strip_w, slots, min_strip)
    seen = np.zeros((ny, nx), np.int32)
    fused = np.zeros((ny, nx), bool)
    for x, w, y0, y1 in tiles:
        assert 0 < w <= strip_w and x % align == 0 and y1 > y0
        seen[y0:y1, x:x + w] += 1
        fused[y0:y1, x:x + w] = True
    for x, y, w, h in rects:
        seen[y:y + h, x:x + w] += 1
    assert (seen == 1).all()
    assert not (fused & _near(mask, perx, pery, reach)).any()
    if not perx:
        assert not fused[:, :reach].any() and not fused[:, nx - reach:].any()
    if not pery:
        assert not fused[:reach].any() and not fused[ny - reach:].any()


def test_a_plan_takes_time_in_proportion_to_the_plate(lib):
    """Scattered holes (most row bands with clear columns of their own): eight
    times the rows, about eight times the time. Rescanning every pair of
    neighbouring runs after each merge took sixty times."""
    t = []
    for ny in (16384, 131072):
        mask = _scattered(256, ny, np.random.Generator(np.random.PCG64(1)), ny // 16, 8)
        t.append(min(_plan(lib, mask, True, True, 10, 16, 224, 512)[2] for _ in range(3)))
    print(f"plans of 256 x 16384 and 256 x 131072: {t[0] * 1e3:.1f} and {t[1] * 1e3:.1f} ms")
    assert t[1] < 24 * t[0]


@pytest.mark.parametrize("cls", range(4))
@pytest.mark.parametrize("edges", range(3))
def test_choosing_a_window_allocates_nothing(lib, cls, edges):
    """It is part of every lbm_step of a small plate."""
    for w, h in ((5, 5), (64, 64), (300, 97), (1021, 777)):
        shape, steps = ctypes.c_int(-1), ctypes.c_int(-1)
        assert lib.choose(256, cls, edges, w, h, 1, ctypes.byref(shape), ctypes.byref(steps)) == 0
        assert 0 <= shape.value < 6 and steps.value in (1, 2)


@pytest.mark.parametrize("edges", range(3))
def test_windows_are_priced_by_the_device_s_compute_units(lib, edges):
    """An eighth of the windows on an eighth of the compute units: the same
    choice."""
    def choice(cus, w, h, n):
        shape, steps = ctypes.c_int(), ctypes.c_int()
        lib.choose(cus, 1, edges, w, h, n, ctypes.byref(shape), ctypes.byref(steps))
        return shape.value, steps.value

    seen = set()
    for side in (20, 64, 100, 150, 220, 300, 500):
        want = choice(256, side, side, 8)
        seen.add(want)
        assert choice(32, side, side, 1) == want
    assert len(seen) > 1  # (the size matters)
