"""A captured lbm_step of an even number of steps can be replayed: it leaves
the state in the buffers it read it from, whichever kernels and steps per
launch run it. Replays, with eager work between them, give the bits of eager
steps."""
import numpy as np
import pytest

from tests.test_gpu_hole import D_, N_, P_
from tests.test_gpu_split import _mask

pytestmark = pytest.mark.gpu

WALLS, FREE = (N_, D_, D_, N_), (P_, P_, P_, P_)


@pytest.mark.parametrize("nx,ny,precision,scheme,kinds,holes,n", [
    (64, 64, "fp64", "pc", FREE, None, 2),            # windows, an odd pair as two single steps
    (64, 60, "fp16", "pc", FREE, None, 6),
    (120, 90, "fp32", "pc", WALLS, "round", 2),       # windows with walls and holes
    (1409, 1303, "fp64", "pc", FREE, None, 6),        # the fused kernel's pairs
    (1187, 949, "fp32", "pc", (P_, P_, D_, N_), None, 2),  # the split plan
    (1187, 949, "fp64", "pc", WALLS, "seam", 6),
    (120, 90, "fp64", "extrap", WALLS, None, 2),      # j of two steps in two buffers
    (1187, 949, "fp32", "extrap", FREE, "seam", 4),
])
def test_replays_of_captured_steps_equal_eager_steps(gpu, nx, ny, precision, scheme, kinds, holes, n):
    import torch

    from paper_2208_13769_amd import lbm

    rng = np.random.Generator(np.random.PCG64(5))
    m = _mask(nx, ny, kinds, holes) if holes else np.ones((ny, nx), np.uint8)
    u0 = 0.002 * rng.standard_normal((2, ny, nx)) * m[None]
    v0 = 0.002 * rng.standard_normal((2, ny, nx)) * m[None]
    stream = torch.cuda.Stream()
    out = []
    for captured in (True, False):
        s = lbm.Solver(nx, ny, 1.0, precision, scheme, stream=stream, walled=True)
        s.set_material(1.0, 0.05, 0.05, 0.8)
        for e, k in enumerate(kinds):
            if k != P_:
                s.set_boundary(e, k, (0.0, 2e-4) if k == N_ else (0.0, 0.0))
        if holes:
            s.set_mask(m)
        s.set_fields(u0, v0)
        s.step(4)
        if captured:
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                s.step(n)
            for _ in range(3):
                with torch.cuda.stream(stream):
                    g.replay()
                torch.ones(1 << 16, device="cuda").mul_(2.0)
                torch.cuda.synchronize()
        else:
            for _ in range(3):
                s.step(n)
        u, v, P, d, st = s.read()
        s.close()
        assert st == 0
        out.append((u, v, P))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
