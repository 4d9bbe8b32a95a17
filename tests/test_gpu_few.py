"""Batches of a few large instances: the groups of the persistent solve over several XCDs.

One to seven instances of more than 32 tiles (512 nodes of a colour) have groups of
other sizes than more of them have; an instance has the bits of a run of its own
either way, and a batch of one or two must not take a multiple of its time."""
import pytest

import workloads as W
from tests.parity import say
from tests.test_gpu_batch import assert_identical, lbfd  # noqa: F401  (the fixture)
from tests.test_gpu_solve import case

pytestmark = pytest.mark.gpu

P, WALL = W.PERIODIC, W.WALL
# 75 tiles; 33 (a remainder on every span); 257 (groups that share an XCD); a 3-D grid with seams
SHAPES = {
    "2d": ((300, 256, 1), (P, WALL, P)),
    "2d_seams": ((131, 255, 1), (P, P, P)),
    "2d_shared": ((512, 513, 1), (WALL, P, P)),
    "3d_seams": ((41, 39, 43), (P, P, P)),
}


@pytest.mark.parametrize("n", [1, 2, 3, 5, 7, 9])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_few_instances(lbfd, name, n):  # noqa: F811
    shape, bc = SHAPES[name]
    prec = "fp64" if n % 2 else "fp32"
    inst = [case(shape, bc, 1.0, prec) for _ in range(n)]
    say(f"[few] {n} of {name} {shape} {prec}")
    b = lbfd.Batch([p for p, _ in inst])
    for i, (m, (_, q)) in enumerate(zip(b.members, inst)):
        m.init_fields(dict(q, psi0=0.2 + 0.01 * i))
    b.step(3)
    for i in {0, n // 2, n - 1}:
        p, q = inst[i]
        s = lbfd.Solver(p).init_fields(dict(q, psi0=0.2 + 0.01 * i)).step(3)
        sweeps = s.observables()["sor_sweeps"]
        assert max(sweeps) > 3   # past the sweeps that are launches
        assert_identical(b[i], s, f"{name} {i} of {n}")
        s.close()
    b.close()


@pytest.mark.parametrize("n", [1, 2])
def test_few_large_instances_use_the_chip(lbfd, n):  # noqa: F811
    """1024^2 FP32, ten sweeps: a batch of one takes 1.2 times a run of its own, of two 2.1 times
    (4.4 and 4.8 times with a group on one XCD)."""
    import torch

    p, q = case((1024, 1024, 1), (P, P, P), 1.0, "fp32")
    p.update(sor_max_sweeps=10, sor_tol=0.0, Ds=2.0, Db=2.0)   # every sweep of the budget
    s = lbfd.Solver(p).init_fields(q)
    b = lbfd.Batch([p] * n)
    for m in b.members:
        m.init_fields(q)
    ms = []
    for run in (s, b):
        run.step(4)
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        t = []
        for _ in range(3):
            e0.record()
            run.step(6)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1) / 6)
        ms.append(min(t))
    say(f"[few] {n} of 1024^2: {ms[1]:.3f} ms a step, one run {ms[0]:.3f}")
    b.close()
    s.close()
    assert ms[1] < (1.3 + n) * ms[0]
