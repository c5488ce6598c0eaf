"""The library's own plan on either side of a size limit gives the bits of the
fused kernel's single steps (the explicit scheme between y walls)."""
import numpy as np
import pytest

from tests.test_gpu_windows import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,precision", [(1021, 777, "fp64"), (1703, 1702, "fp64"), (1704, 1703, "fp64"),
                                             (1021, 777, "fp32")])
def test_explicit_plans_between_y_walls(gpu, nx, ny, precision):
    a = _run(nx, ny, precision, "explicit", True, False, (1, 2))
    b = _run(nx, ny, precision, "explicit", True, True, (3,))
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)
