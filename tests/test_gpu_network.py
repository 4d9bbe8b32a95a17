"""The network's layer kernels at the sizes where their tiles end: rows of output
nodes from one to several tiles of 30 and 32, planes past one column of 32, rows
past one group of 8, the width at which a layer changes kernel, several grids a
call, and the smallest ones. References and tolerances are those of the
surrogate tests: BF16 roundings of the kernels, sums in FP64, and the error that
roundings of a sum on the edge of two BF16 values leave (5e-3 of the largest
output, 2e-2 of the largest gradient)."""
import numpy as np
import pytest

from oracle import surrogate as OS
from tests.parity import say
from tests.test_gpu_surrogate import (bf16, bf16_tensor, gpu_params, lbfd, padded_input,  # noqa: F401
                                      ref_forward, ref_gradient)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,h,w", [(1, 9, 9, 9), (3, 9, 17, 10), (1, 11, 75, 21), (2, 10, 12, 40), (1, 10, 12, 67),
                                     (1, 44, 19, 70), (2, 12, 9, 100), (1, 9, 26, 131)])
def test_forward_sizes(lbfd, B, d, h, w):  # noqa: F811
    import torch

    rng = np.random.default_rng(100 * d + w)
    ps = gpu_params(OS.init_params(3, out_scale=1.0))
    x6 = bf16(rng.uniform(-1.0, 1.0, (B, d, h, w, 6)))
    if B == 1:
        sg = lbfd.Surrogate(tile=4, max_batch=1, field=(w - 8, h - 8, d - 8))
    else:
        t = 4   # a tile batch that holds these grids
        while 8 * (t + 6) ** 3 < B * d * h * w or 8 * t ** 3 < B * (d - 8) * (h - 8) * (w - 8):
            t += 1
        sg = lbfd.Surrogate(tile=t, max_batch=8)
    sg.set_params(OS.flatten(ps))
    n = (B, d - 8, h - 8, w - 8, OS.NOUT)
    out = torch.full((int(np.prod(n)) + 64,), 7.0, dtype=torch.float32, device="cuda")   # a guard behind
    got = out[:int(np.prod(n))].view(n)
    sg.forward(bf16_tensor(padded_input(x6)), got)
    ref, _ = ref_forward(ps, x6)
    err = float(np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max())
    say(f"forward {B} x {d} x {h} x {w}: max rel err {err:.2e}")
    assert err < 5e-3
    assert bool((out[int(np.prod(n)):] == 7.0).all())


@pytest.mark.parametrize("T,B", [(3, 1), (7, 3), (23, 2)])
def test_gradient_sizes(lbfd, T, B):  # noqa: F811
    import torch

    rng = np.random.default_rng(T)
    ps = gpu_params(OS.init_params(4, out_scale=1.0))
    x6 = bf16(rng.uniform(-1.0, 1.0, (B, T + 8, T + 8, T + 8, 6)))
    t = rng.standard_normal((B, T, T, T, 4)).astype(np.float32)
    t[..., 2:] = rng.uniform(0.05, 2.0, (B, T, T, T, 2))
    sg = lbfd.Surrogate(tile=T, max_batch=B, dpsi_s=0.02, dphi_s=0.005)
    sg.set_params(OS.flatten(ps))
    loss, g = sg.gradient(bf16_tensor(padded_input(x6)), torch.from_numpy(t).cuda())
    Lr, gr = ref_gradient(ps, x6, t.astype(np.float64), 0.02 / 0.005)
    assert abs(loss - Lr) <= 1e-3 * Lr
    o = 0
    for li, (w, b) in enumerate(gr):
        for name, ref in (("w", w), ("b", b)):
            got = g[o:o + ref.size].reshape(ref.shape)
            o += ref.size
            err = float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-30))
            say(f"tile {T}: layer {li} {name}: max rel err {err:.2e}")
            assert err < 2e-2, (li, name, err)
