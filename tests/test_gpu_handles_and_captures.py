"""A handle that has sampled (and so holds page-locked memory) may be closed
while another stream is being captured: the capture goes on."""
import numpy as np
import pytest

from paper_2208_13769_amd import inputs

pytestmark = pytest.mark.gpu


def test_closing_a_handle_leaves_a_capture_alone(gpu):
    import torch

    from paper_2208_13769_amd import lbm

    n = 64

    def plate():
        s = lbm.Solver(n, n, 1.0, "fp64", "pc", stream=torch.cuda.Stream())
        s.set_material(1.0, 0.1, 0.05, 0.8)
        s.set_fields(*inputs.shear_wave(n, n, 1e-4, n))
        return s

    a, b, ref = plate(), plate(), plate()
    b.sample([1, 2], [3, 4])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=a.stream):
        a.step(4)
        b.close()
        a.step(4)
    with torch.cuda.stream(a.stream):
        g.replay()
    torch.cuda.synchronize()
    ref.step(8)
    for x, y in zip(a.read()[:3], ref.read()[:3]):
        assert np.array_equal(x, y)
    a.close()
    ref.close()
