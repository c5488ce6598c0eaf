"""Read-outs into page-locked arrays (written by the kernel over the link),
pageable ones (through the staging area) and mixtures give the same values;
a probe series enqueued together equals one sampled step by step."""
import numpy as np
import pytest

from paper_2208_13769_amd import inputs

pytestmark = pytest.mark.gpu


def _solver(nx, ny, precision="fp64"):
    from paper_2208_13769_amd import lbm

    s = lbm.Solver(nx, ny, 0.5, precision, "pc", walled=True)
    s.set_material(1.0, 0.1, 0.05, 0.8)
    s.set_boundary(lbm.LBM_EDGE_YMAX, lbm.LBM_BC_NEUMANN_T, (0.0, 0.001))
    m = np.ones((ny, nx), np.uint8)
    m[ny // 3:ny // 2, nx // 3:nx // 2] = 0
    s.set_mask(m)
    s.set_fields(*inputs.filtered_random_velocity(nx, ny, 3.0, 3, 0.01))
    return s


def _pinned(*shape):
    import torch

    return torch.empty(shape, dtype=torch.float64, pin_memory=True).numpy()


# (1500 x 1400: more than one chunk of the staging area)
@pytest.mark.parametrize("nx,ny", [(13, 11), (300, 97), (1500, 1400)])
def test_page_locked_and_pageable_read_outs_are_equal(gpu, nx, ny):
    from paper_2208_13769_amd import lbm

    s = _solver(nx, ny, "fp32u64")
    s.step(3)
    want = [np.empty((2, ny, nx)), np.empty((2, ny, nx)), np.empty((2, 2, ny, nx))]
    assert lbm.lbm_read_fields(s.h, *want) == lbm.LBM_OK
    for pins in ((1, 1, 1), (1, 0, 1), (0, 1, 0)):
        got = [(_pinned if p else np.empty)(*a.shape) if p else np.empty(a.shape) for p, a in zip(pins, want)]
        assert lbm.lbm_read_fields(s.h, *got) == lbm.LBM_OK
        for a, b in zip(got, want):
            assert np.array_equal(a, b)
    part = _pinned(2, 2, ny, nx)
    lbm.lbm_read_fields(s.h, None, None, part)
    assert np.array_equal(part, want[2])
    # not 128-byte aligned
    odd = _pinned(2 * nx * ny + 1)[1:].reshape(2, ny, nx)
    lbm.lbm_read_fields(s.h, odd)
    assert np.array_equal(odd, want[0])
    sig, E, W = s.read_derived()
    psig, pW = _pinned(2, 2, ny, nx), _pinned(ny, nx)
    lbm.lbm_read_derived(s.h, psig, None, pW)
    assert np.array_equal(psig, sig) and np.array_equal(pW, W)
    s.close()


def test_unstable_flag_through_a_page_locked_read(gpu):
    """The flag reported with a read the kernel writes itself (the second read on)."""
    from paper_2208_13769_amd import lbm

    n = 32
    s = lbm.Solver(n, n, 1.0, "fp64", "pc")
    s.set_material(1.0, 0.1, 0.05, 0.8)
    out = [_pinned(2, n, n), _pinned(2, n, n), _pinned(2, 2, n, n)]
    s.set_fields(np.zeros((2, n, n)), np.zeros((2, n, n)))
    s.step(1)
    assert lbm.lbm_read_fields(s.h, *out) == lbm.LBM_OK and lbm.lbm_read_fields(s.h, *out) == lbm.LBM_OK
    rng = np.random.Generator(np.random.PCG64(1))
    s.set_fields(np.zeros((2, n, n)), 2.0 * rng.standard_normal((2, n, n)))
    s.step(20)
    assert lbm.lbm_read_fields(s.h, *out) == lbm.LBM_ERR_UNSTABLE
    s.close()


@pytest.mark.parametrize("nodes,nsteps,every", [(1, 0, 3), (5, 1, 4), (8, 13, 4), (40, 30, 2), (700, 6, 1)])
def test_sample_series_equals_stepwise_samples(gpu, nodes, nsteps, every):
    """40 x 16 samples pass the 64 KiB buffer; 700 nodes do not fit it."""
    nx, ny = 96, 64
    rng = np.random.Generator(np.random.PCG64(2))
    xs, ys = rng.integers(0, nx, nodes), rng.integers(0, ny, nodes)
    a, b = _solver(nx, ny), _solver(nx, ny)
    steps, vals = a.sample_series(xs, ys, nsteps, every)
    want, at = [b.sample(xs, ys)], [0]
    while at[-1] < nsteps:
        k = min(every, nsteps - at[-1])
        b.step(k)
        at.append(at[-1] + k)
        want.append(b.sample(xs, ys))
    assert list(steps) == at and np.array_equal(vals, np.array(want))
    a.close()
    b.close()
