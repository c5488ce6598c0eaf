"""The windows that run small plates' steps (one or two steps per launch, each
block a 2D window held in registers and LDS) against the fused step kernel:
bitwise equal on periodic and y-walled plates, at the smallest plate, plates
narrower than a window, tiles with remainders, odd step counts, both schemes
and every storage form."""
import numpy as np
import pytest

from paper_2208_13769_amd import inputs

pytestmark = pytest.mark.gpu


def _run(nx, ny, precision, scheme, walled, fused, steps, rounding="nearest"):
    from paper_2208_13769_amd import lbm

    s = lbm.Solver(nx, ny, 1.0, precision, scheme)
    s.set_material(1.0, 0.07, 0.04, 0.75)
    s.set_body_force((1e-5, -2e-5))
    if walled:
        s.set_boundary(lbm.LBM_EDGE_YMIN, lbm.LBM_BC_DIRICHLET_J, (0.0004, 0.0002))
        s.set_boundary(lbm.LBM_EDGE_YMAX, lbm.LBM_BC_NEUMANN_T, (0.0003, 0.001))
    if rounding == "stochastic":
        s.set_rounding("stochastic", 77)
    if fused:
        s.set_general_path(False)
    rng = np.random.Generator(np.random.PCG64(5))
    u0, v0 = 1e-3 * rng.standard_normal((2, ny, nx)), np.zeros((2, ny, nx))
    if min(nx, ny) >= 16:
        u0, v0 = inputs.filtered_random_velocity(nx, ny, 3.0, 9, 0.01)
    s.set_fields(u0, v0)
    for n in steps:
        s.step(n)
    u, v, P, d, st = s.read()
    s.close()
    assert d.steps == sum(steps)
    return u, v, P, st


@pytest.mark.parametrize("nx,ny", [(5, 5), (7, 40), (23, 13), (67, 45), (129, 257)])
@pytest.mark.parametrize("walled", [False, True])
@pytest.mark.parametrize("precision,scheme", [("fp64", "pc"), ("fp64", "explicit"), ("fp32", "pc"),
                                              ("fp32u64", "pc"), ("fp16", "pc"), ("bf16", "explicit")])
def test_windows_equal_the_fused_kernel(gpu, precision, scheme, walled, nx, ny):
    """One step, a pair, and a longer odd run: single- and two-step launches."""
    a = _run(nx, ny, precision, scheme, walled, False, (1, 2, 6, 5))
    b = _run(nx, ny, precision, scheme, walled, True, (14,))
    assert a[3] == b[3]
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
def test_windows_round_stochastically_as_the_fused_kernel(gpu, precision):
    """The values a two-step launch hands on are rounded with the bits a
    store would use."""
    a = _run(90, 64, precision, "pc", False, False, (9,), "stochastic")
    b = _run(90, 64, precision, "pc", False, True, (9,), "stochastic")
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("precision,walled,nx,ny", [("fp64", False, 1021, 777), ("fp64", True, 1021, 777),
                                                    ("fp32", False, 1603, 900), ("fp32", True, 1603, 900),
                                                    ("fp32u64", False, 1603, 900), ("fp32u64", True, 1603, 900),
                                                    ("fp16", False, 1603, 900), ("fp16", True, 1603, 900)])
def test_default_plan_of_larger_plates_equals_single_steps(gpu, precision, walled, nx, ny):
    """Plates just beyond the windows' sizes: the library's own plan (two steps
    per launch where it can, an odd remainder) against one step per launch."""
    a = _run(nx, ny, precision, "pc", walled, False, (1, 4, 3))
    b = _run(nx, ny, precision, "pc", walled, True, (8,))
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)
