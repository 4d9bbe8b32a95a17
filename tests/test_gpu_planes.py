"""Units of several planes in the row kernels of the network (many small grids).

Where an output plane has few tiles a unit takes several, the last one of a grid
what is left: forward layers and gradients of such batches against the FP64
references of the layer tests, and the time of many grids against their number."""
import pytest

from tests import test_gpu_network as network
from tests.parity import say
from tests.test_gpu_surrogate import lbfd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,h,w", [(8, 60, 9, 11), (1, 401, 10, 9), (8, 45, 12, 12)])
def test_forward_of_small_planes(lbfd, B, d, h, w):  # noqa: F811
    network.test_forward_sizes(lbfd, B, d, h, w)


@pytest.mark.parametrize("T,B", [(3, 160), (5, 70)])
def test_gradient_of_small_tiles(lbfd, T, B):  # noqa: F811
    network.test_gradient_sizes(lbfd, T, B)


def test_many_small_grids_share_their_start(lbfd):  # noqa: F811
    """1,024 crops of 12^3 input nodes take 156 us, 6 times as long as 8 of them; 355 us and 13
    times with a unit for every plane."""
    import torch

    us = []
    for B in (8, 1024):
        sg = lbfd.Surrogate(tile=4, max_batch=B)
        x = torch.zeros((B, 12, 12, 12, 16), dtype=torch.bfloat16, device="cuda")
        out = torch.empty((B, 4, 4, 4, lbfd.SG_NOUT), device="cuda")
        sg.forward(x, out)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        runs = []
        for _ in range(5):
            a.record()
            for _ in range(10):
                sg.forward(x, out)
            b.record()
            torch.cuda.synchronize()
            runs.append(100.0 * a.elapsed_time(b))
        us.append(min(runs))
        say(f"{B} crops: {us[-1]:.1f} us")
        sg.close()
    assert us[1] < 9.0 * us[0]
