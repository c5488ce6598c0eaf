"""The tuner offers the library's own plan where none of the other choices is
it (no GPU), and a handle can go back to that plan (GPU)."""
import numpy as np
import pytest

from paper_2208_13769_amd.autotune import DEFAULT, GENERAL, apply_tiling, candidates
from tests.test_autotune_host import FakeSolver

P_, D_, N_ = 0, 1, 2


class Plate(FakeSolver):
    def __init__(self, kinds, mask=False):
        super().__init__()
        self.kinds, self.mask, self.calls = kinds, mask, []

    def edges(self):
        return self.kinds, self.mask

    def __getattr__(self, name):
        return lambda *a: self.calls.append((name, *a))


@pytest.mark.parametrize("kinds,mask,own", [((P_, P_, P_, P_), False, False), ((P_, P_, D_, N_), False, True),
                                            ((P_, P_, N_, N_), False, True), ((P_, P_, D_, N_), True, False),
                                            ((N_, N_, D_, N_), False, False), ((P_, P_, P_, P_), True, False)])
def test_own_plan_is_a_candidate_between_y_walls(kinds, mask, own):
    c = candidates(Plate(kinds, mask), 1024, 900, "fp64", "pc")
    assert (DEFAULT in c) == own and c[-1] == GENERAL and len(set(c)) == len(c)


def test_applying_the_own_plan():
    s = Plate((P_, P_, D_, N_))
    apply_tiling(s, list(DEFAULT))
    assert s.calls == [("set_default_plan",)]


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,precision", [(96, 70, "fp64"), (1187, 949, "fp64"), (1187, 949, "fp16")])
def test_going_back_to_the_own_plan(gpu, nx, ny, precision):
    """After every other choice the handle reports the shape it was made with
    and gives the bits of one that never chose."""
    from paper_2208_13769_amd import inputs, lbm

    def plate():
        s = lbm.Solver(nx, ny, 1.0, precision, "pc")
        s.set_material(1.0, 0.1, 0.05, 0.8)
        s.set_boundary(lbm.LBM_EDGE_YMIN, lbm.LBM_BC_DIRICHLET_J, (0.0, 0.0))
        s.set_boundary(lbm.LBM_EDGE_YMAX, lbm.LBM_BC_NEUMANN_T, (0.0, 0.001))
        s.set_fields(*inputs.filtered_random_velocity(nx, ny, 4.0, 3, 0.01))
        return s

    a, b = plate(), plate()
    assert a.edges() == ((0, 0, 1, 2), False)
    made = a.tiling(), a.steps_per_launch()
    for choice in ((64, 3, 1), GENERAL) + (((128, 2, 2),) if precision == "fp64" else ()):
        apply_tiling(a, choice)
    apply_tiling(a, DEFAULT)
    assert (a.tiling(), a.steps_per_launch()) == made
    for s in (a, b):
        s.step(5)
    for x, y in zip(a.read()[:3], b.read()[:3]):
        assert np.array_equal(x, y)
    a.close()
    b.close()
