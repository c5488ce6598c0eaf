"""Split plates against the oracle in v as well as u and P, over the whole plate
and at its worst node: a wrong momentum store at a seam between the fused
kernel and windows in the last step shows in v alone. The velocity of 16-bit
populations takes their rounding (2^-11 of a population) once per step; the
other forms hold the bounds of u and P."""
import numpy as np
import pytest

from tests.helpers import MAX_NORM_FACTOR, max_rel, rel_l2
from tests.test_gpu_hole import D_, N_, P_, _gpu, _oracle
from tests.test_gpu_split import _mask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,precision,scheme,kinds,holes,n", [
    (1187, 949, "fp64", "pc", (N_, D_, D_, N_), None, 4),        # pairs: the last launch is one
    (1187, 949, "fp64", "pc", (N_, N_, N_, N_), "round", 4),
    (1187, 949, "fp64", "pc", (P_, P_, D_, N_), "seam", 5),      # a single last step
    (1187, 949, "fp64", "pc", (P_, P_, D_, N_), None, 4),
    (1187, 949, "fp64", "explicit", (D_, N_, P_, P_), "seam", 3),
    (1187, 949, "fp64", "extrap", (N_, N_, N_, N_), "round", 3),
    (1187, 949, "fp32", "pc", (N_, D_, D_, N_), "round", 4),
    (1187, 949, "fp32", "explicit", (N_, D_, D_, N_), None, 3),
    (1187, 949, "fp16", "pc", (N_, N_, N_, N_), "round", 5),
    (3301, 3067, "fp32", "pc", (N_, N_, D_, N_), "round", 4),    # windows on the second stream
    (2111, 2099, "fp64", "explicit", (N_, N_, D_, N_), "round", 3),  # windows beside the share, a thin strip theirs
])
def test_split_plate_velocity(gpu, nx, ny, precision, scheme, kinds, holes, n):
    m = _mask(nx, ny, kinds, holes)
    rng = np.random.Generator(np.random.PCG64(78))
    u0, v0 = (0.002 * rng.standard_normal((2, ny, nx)) * m[None] for _ in range(2))
    vals = [(0.0, 0.0) if k == P_ else ((0.0001, 0.0) if e == 0 else (0.0, 2e-4) if k == N_ else (0.0, 0.0))
            for e, k in enumerate(kinds)]
    mask = m if holes else None
    uo, vo, Po, so, do = _oracle(nx, ny, u0, v0, n, kinds, vals, mask, scheme=scheme, lam=0.05)
    ug, vg, Pg, sg, dg, st, _ = _gpu(nx, ny, u0, v0, n, kinds, vals, mask, precision=precision, scheme=scheme, lam=0.05)
    assert st == 0
    tol = {"fp64": 1e-12, "fp32": 1e-5, "fp16": 1e-3}[precision]
    tol_v = n * 2.0 ** -11 if precision == "fp16" else tol
    e = [rel_l2(ug, uo), rel_l2(vg, vo), rel_l2(Pg, Po)]
    print(f"{precision} {scheme} {kinds} {holes}: rel-L2 u {e[0]:.3e} v {e[1]:.3e} P {e[2]:.3e}, "
          f"max v {max_rel(vg, vo):.3e}", flush=True)
    assert e[0] < tol and e[1] < tol_v and e[2] < tol
    assert max_rel(vg, vo) < MAX_NORM_FACTOR * tol_v
    assert np.abs(ug[:, m == 0]).sum() == 0.0 and np.abs(vg[:, m == 0]).sum() == 0.0
