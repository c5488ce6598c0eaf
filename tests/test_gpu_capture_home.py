"""A captured lbm_step reads the same buffers however many even eager calls
and restarts lie between its replays: a call of an even number of steps ends in
the copy it began with, and set_fields starts in the copy that the graph
reads. Replays, eager steps and restarts together give the bits of a handle
that never captured. (A restart of a plate with 16-bit populations chooses
their scale anew, and the graph holds the old one: no restart there.)"""
import numpy as np
import pytest

from tests.test_gpu_hole import D_, N_, P_
from tests.test_gpu_split import _mask

pytestmark = pytest.mark.gpu

WALLS, FREE = (N_, D_, D_, N_), (P_, P_, P_, P_)


def _plate(nx, ny, precision, scheme, kinds, holes, stream):
    from paper_2208_13769_amd import lbm

    s = lbm.Solver(nx, ny, 1.0, precision, scheme, stream=stream, walled=True)
    s.set_material(1.0, 0.05, 0.05, 0.8)
    for e, k in enumerate(kinds):
        if k != P_:
            s.set_boundary(e, k, (0.0, 2e-4) if k == N_ else (0.0, 0.0))
    if holes:
        s.set_mask(_mask(nx, ny, kinds, holes))
    return s


def _fields(nx, ny, kinds, holes, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    m = _mask(nx, ny, kinds, holes) if holes else np.ones((ny, nx), np.uint8)
    return tuple(0.002 * rng.standard_normal((2, ny, nx)) * m[None] for _ in range(2))


def _read(s):
    u, v, P, d, st = s.read()
    assert st == 0
    return u, v, P


def _equal(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def _run(nx, ny, precision, scheme, kinds, holes, warm, n, choose=lambda s: None):
    """warm steps, capture of n, replay, two and four eager steps, replay; a
    restart with other fields, replay, six eager steps, replay."""
    import torch

    first, second = (_fields(nx, ny, kinds, holes, seed) for seed in (5, 6))
    stream = torch.cuda.Stream()

    def replay(g):
        with torch.cuda.stream(stream):
            g.replay()
        torch.cuda.synchronize()

    s = _plate(nx, ny, precision, scheme, kinds, holes, stream)
    choose(s)
    s.set_fields(*first)
    s.step(warm)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        s.step(n)
    replay(g)
    got = [_read(s)]
    s.step(2)
    s.step(4)
    replay(g)
    got.append(_read(s))
    restart = precision not in ("fp16", "bf16")
    if restart:
        s.set_fields(*second)
        replay(g)
        got.append(_read(s))
        s.step(6)
        replay(g)
        got.append(_read(s))
    s.close()

    s = _plate(nx, ny, precision, scheme, kinds, holes, stream)
    choose(s)
    s.set_fields(*first)
    s.step(warm + n)
    _equal(got[0], _read(s))
    s.step(6 + n)
    _equal(got[1], _read(s))
    if restart:
        s.set_fields(*second)
        s.step(n)
        _equal(got[2], _read(s))
        s.step(6 + n)
        _equal(got[3], _read(s))
    s.close()


@pytest.mark.parametrize("nx,ny,precision,scheme,kinds,holes,n", [
    (64, 64, "fp64", "pc", FREE, None, 4),                  # windows
    (64, 60, "fp16", "pc", (P_, P_, D_, N_), None, 2),      # windows, two steps, y walls
    (120, 90, "fp32", "pc", WALLS, "round", 4),             # windows with walls and holes
    (1409, 1303, "fp64", "pc", FREE, None, 4),              # the fused kernel's pairs
    (1187, 949, "fp32", "pc", (P_, P_, D_, N_), None, 2),   # the split plan
    (1187, 949, "fp64", "pc", WALLS, "seam", 4),
    (120, 90, "fp64", "extrap", WALLS, None, 2),            # j of three states
    (1187, 949, "fp32", "extrap", FREE, "seam", 4),
    (3301, 3067, "fp32", "pc", WALLS, "round", 4),          # windows on the second stream
])
def test_replays_between_even_eager_calls_and_restarts(gpu, nx, ny, precision, scheme, kinds, holes, n):
    _run(nx, ny, precision, scheme, kinds, holes, 2, n)


@pytest.mark.parametrize("n", [2, 6])
@pytest.mark.parametrize("nx,ny,kinds", [(96, 70, FREE), (300, 129, (P_, P_, D_, N_))])
def test_chosen_two_step_launches_replay_too(gpu, nx, ny, kinds, n):
    """Two steps per launch set by the caller: a captured call still makes an
    even number of launches."""
    _run(nx, ny, "fp64", "pc", kinds, None, 2, n, lambda s: s.set_steps_per_launch(2))
