"""sample_series for every `every` that min(every, steps left) made sense of:
beyond the run, up to the largest 64-bit integer and past it."""
import numpy as np
import pytest

from paper_2208_13769_amd import inputs

pytestmark = pytest.mark.gpu


def _solver():
    from paper_2208_13769_amd import lbm

    s = lbm.Solver(40, 33, 1.0, "fp64", "pc")
    s.set_material(1.0, 0.1, 0.05, 0.8)
    s.set_fields(*inputs.filtered_random_velocity(40, 33, 3.0, 3, 0.01))
    return s


@pytest.mark.parametrize("every", [7, 8, 2 ** 62, 2 ** 63 - 3, 2 ** 63 - 1, 2 ** 70, float("inf")])
def test_one_interval_longer_than_the_run(gpu, every):
    xs, ys = [1, 30, 7], [2, 5, 32]
    a, b = _solver(), _solver()
    steps, vals = a.sample_series(xs, ys, 7, every)
    want = [b.sample(xs, ys)]
    b.step(7)
    want.append(b.sample(xs, ys))
    assert list(steps) == [0, 7] and np.array_equal(vals, np.array(want))
    steps, vals = a.sample_series(xs, ys, 0, every)
    assert list(steps) == [0] and np.array_equal(vals, np.array(want[1:]))
    a.close()
    b.close()


def test_the_library_itself_takes_the_largest_interval(gpu):
    from paper_2208_13769_amd import lbm

    a, b = _solver(), _solver()
    vals = lbm.lbm_sample_series(a.h, [3], [4], 5, 2 ** 63 - 1)
    b.step(5)
    assert vals.shape == (2, 1, 17) and np.array_equal(vals[1], b.sample([3], [4]))
    a.close()
    b.close()
