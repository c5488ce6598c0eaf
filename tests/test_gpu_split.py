"""Large plates with walls or holes: the fused kernel's periodic form over the
part clear of them, windows over the rest, against the oracle. Sizes beyond
the ones windows run whole; holes across periodic seams, next to strips, one
node wide and round; heights that leave a short last band; pairs of steps and
an odd last one."""
import numpy as np
import pytest

from tests.helpers import rel_l2
from tests.test_gpu_hole import D_, N_, P_, _gpu, _oracle

pytestmark = pytest.mark.gpu


def _mask(nx, ny, kinds, holes):
    m = np.ones((ny, nx), np.uint8)
    if holes == "round":
        y, x = np.mgrid[:ny, :nx]
        m[(y - 0.45 * ny) ** 2 + (x - 0.6 * nx) ** 2 < (0.2 * min(nx, ny)) ** 2] = 0
        m[5, 7] = 0
        m[ny // 2:ny // 2 + 40, 40] = 0
    if holes == "seam":  # across the periodic edges there are
        m[ny // 3:ny // 3 + 60, nx // 2:nx // 2 + 33] = 0
        if kinds[0] == P_:
            m[100:140, :20] = m[100:140, -25:] = 0
        if kinds[2] == P_:
            m[:9, 300:420] = m[-7:, 300:420] = 0
    return m


@pytest.mark.parametrize("precision,scheme,tol", [("fp64", "pc", 1e-12), ("fp64", "explicit", 1e-12),
                                                  ("fp64", "extrap", 1e-12), ("fp32", "pc", 1e-5),
                                                  ("fp16", "pc", 1e-3)])
@pytest.mark.parametrize("kinds,holes", [((N_, D_, D_, N_), None), ((N_, N_, N_, N_), "round"), ((P_, P_, D_, N_), "seam"),
                                         ((D_, N_, P_, P_), "seam"), ((P_, P_, P_, P_), "seam"),
                                         ((P_, P_, D_, N_), None)])
def test_split_plate_matches_oracle(gpu, precision, scheme, tol, kinds, holes):
    nx, ny, n = 1187, 949, 5
    m = _mask(nx, ny, kinds, holes)
    rng = np.random.Generator(np.random.PCG64(77))
    u0 = 0.002 * rng.standard_normal((2, ny, nx)) * m[None]
    v0 = 0.002 * rng.standard_normal((2, ny, nx)) * m[None]
    vals = [(0.0, 0.0) if k == P_ else ((0.0001, 0.0) if e == 0 else (0.0, 2e-4) if k == N_ else (0.0, 0.0))
            for e, k in enumerate(kinds)]
    mask = m if holes else None
    uo, vo, Po, so, do = _oracle(nx, ny, u0, v0, n, kinds, vals, mask, scheme=scheme, lam=0.05)
    ug, vg, Pg, sg, dg, st, _ = _gpu(nx, ny, u0, v0, n, kinds, vals, mask, precision=precision, scheme=scheme, lam=0.05)
    assert st == 0
    e = [rel_l2(ug, uo), rel_l2(vg, vo), rel_l2(Pg, Po)]
    print(f"split {precision} {scheme} {kinds} {holes}: rel-L2 u {e[0]:.3e} v {e[1]:.3e} P {e[2]:.3e}", flush=True)
    assert max(e[0], e[2]) < tol
    assert np.abs(ug[:, m == 0]).sum() == 0.0
