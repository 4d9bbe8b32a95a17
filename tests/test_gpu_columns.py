"""Columns of the marching forward kernel, cut along z where a grid has few of them.

Depths at and beside the cuts (one plane a column, an odd last column, one column
of 32) against the FP64 reference, as in the layer tests; and a grid that is
wide enough for this kernel must not take a multiple of the time of one just
narrower, which another kernel takes."""
import pytest

from tests import test_gpu_network as network
from tests.parity import say
from tests.test_gpu_surrogate import lbfd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,h,w", [(1, 10, 12, 70), (1, 75, 11, 68), (1, 41, 40, 100), (2, 20, 17, 75),
                                     (1, 43, 70, 131)])
def test_forward_of_few_columns(lbfd, B, d, h, w):  # noqa: F811
    network.test_forward_sizes(lbfd, B, d, h, w)


@pytest.mark.parametrize("d,h,w", [(12, 12, 68), (30, 30, 100), (72, 72, 72)])
def test_few_columns_fill_the_chip(lbfd, d, h, w):  # noqa: F811
    """Microseconds of a forward call: 31, 43 and 100 with columns of a few planes, against 32, 40
    and 113 for the narrower grids; 86, 254 and 321 with columns of 32."""
    import torch

    us = []
    for width in (w, 57):
        sg = lbfd.Surrogate(tile=4, max_batch=1, field=(width - 8, h - 8, d - 8))
        x = torch.zeros((1, d, h, width, 16), dtype=torch.bfloat16, device="cuda")
        out = torch.empty((1, d - 8, h - 8, width - 8, lbfd.SG_NOUT), device="cuda")
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
        say(f"forward {d} x {h} x {width}: {us[-1]:.1f} us")
        sg.close()
    assert us[0] < 2.2 * us[1]
