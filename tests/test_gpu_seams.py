"""Seam classes by one workgroup and by all of them.

Grids with long rows, columns or edges on their seams spread these over the
workgroups, the others give them to one; a batch does what its longest instance
needs. The rows and their order are the same, so an instance has the same bits
either way, and a long seam must not cost a multiple of the sweep it belongs to."""
import pytest

import workloads as W
from tests.parity import say
from tests.test_gpu_batch import assert_identical, lbfd  # noqa: F401  (the fixture)
from tests.test_gpu_solve import case

pytestmark = pytest.mark.gpu

P, WALL = W.PERIODIC, W.WALL
ALL = (P, P, P)
# an instance with short seams, and one with more than 768 nodes on them beside it. Up to 32 x 512
# nodes of a colour a batch is solved by the persistent launch alone.
PAIRS = {
    "2d_persistent": ((33, 31, 1), ALL, (15, 1001, 1), ALL),
    "2d_one_axis": ((40, 37, 1), ALL, (801, 16, 1), (P, WALL, P)),
    "2d_launched": ((257, 255, 1), ALL, (63, 1201, 1), ALL),
    "3d_persistent": ((17, 15, 13), ALL, (7, 9, 401), ALL),
    "3d_two_axes": ((17, 15, 14), ALL, (5, 5, 803), (P, P, WALL)),
    "3d_launched": ((33, 31, 29), ALL, (9, 9, 801), ALL),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(PAIRS))
def test_short_seams_spread_with_long_ones(lbfd, name, prec):  # noqa: F811
    shape, bc, long_shape, long_bc = PAIRS[name]
    inst = [case(shape, bc, 1.0, prec), case(long_shape, long_bc, 1.0, prec)]
    say(f"[seams] {name} {shape} beside {long_shape} {prec}")
    b = lbfd.Batch([p for p, _ in inst])
    for m, (_, q) in zip(b.members, inst):
        m.init_fields(q)
    b.step(3)
    for m, (p, q) in zip(b.members, inst):
        s = lbfd.Solver(p).init_fields(q).step(3)
        sweeps = s.observables()["sor_sweeps"]
        say("sweeps", sweeps)
        assert max(sweeps) > 3   # past the sweeps that are launches everywhere
        assert_identical(m, s, f"{name} {prec}")
        s.close()
    b.close()


@pytest.mark.parametrize("odd,even", [((63, 4001, 1), (64, 4002, 1)), ((9, 9, 8001), (10, 10, 8002))])
def test_long_seams_cost_less_than_the_sweep(lbfd, odd, even):  # noqa: F811
    """Time of a step with 40 sweeps, odd periodic extents against even ones: some 2 times with the
    seams spread (a half-sweep of a few launches or meetings more), 4 to 9 with one workgroup."""
    import torch

    ms = []
    for shape in (odd, even):
        p, q = case(shape, ALL, 1.0, "fp64")
        p.update(sor_max_sweeps=40, sor_tol=0.0, Ds=2.0, Db=2.0)   # every sweep of the budget
        s = lbfd.Solver(p).init_fields(q).step(4)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        runs = []
        for _ in range(3):
            a.record()
            s.step(4)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b) / 4)
        ms.append(min(runs))
        say(f"[seams] {shape}: {1e3 * ms[-1]:.0f} us a step")
        s.close()
    assert ms[0] < 3.0 * ms[1]
