"""Read-outs into page-locked memory whose doubles lie off their alignment go
through copies, as into any other array."""
import numpy as np
import pytest

from paper_2208_13769_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [1, 4])
def test_misaligned_page_locked_arrays(gpu, offset):
    import torch

    from paper_2208_13769_amd import lbm

    nx, ny = 61, 47
    s = lbm.Solver(nx, ny, 1.0, "fp64", "pc")
    s.set_material(1.0, 0.1, 0.05, 0.8)
    s.set_fields(*inputs.filtered_random_velocity(nx, ny, 3.0, 3, 0.01))
    s.step(3)
    want = [np.empty((2, ny, nx)), np.empty((2, 2, ny, nx))]
    lbm.lbm_read_fields(s.h, want[0], None, want[1])
    got = []
    for a in want:
        raw = torch.zeros(a.nbytes + 16, dtype=torch.uint8, pin_memory=True).numpy()
        got.append(np.ndarray(a.shape, np.float64, raw, offset))
    assert not got[0].flags["ALIGNED"]
    lbm.lbm_read_fields(s.h, got[0], None, got[1])
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
    s.close()
