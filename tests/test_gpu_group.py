"""The persistent solve by fewer workgroups than its grid has work for.

On a busy device the group of an implicit solve is made of the workgroups that are
running: it is closed before all have come, each member takes several tiles, and
rows are no longer kept in registers. Here the launch has fewer workgroups than
tiles, or waits for more than there are and closes by itself. The result has the
bits of the full group's."""
import pytest

import workloads as W
from paper_2311_15242_amd import lbfd as L
from tests.parity import say
from tests.test_gpu_batch import assert_identical, lbfd  # noqa: F401  (the fixture)
from tests.test_gpu_solve import GRIDS, case

pytestmark = pytest.mark.gpu

P = W.PERIODIC
# (most workgroups, expected): one, a few, closed early with some and with all of them
GROUPS = [(1, 0), (3, 0), (5, 9), (0, 300)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16dev"])
@pytest.mark.parametrize("name", sorted(GRIDS))
def test_short_groups(lbfd, name, prec):  # noqa: F811
    nx, ny, nz, bc, omega = GRIDS[name]
    p, q = case((nx, ny, nz), bc, omega, prec)
    full = lbfd.Solver(p).init_fields(q).step(3)
    assert max(full.observables()["sor_sweeps"]) > 3
    for most, expected in GROUPS:
        say(f"[group] {name} {prec} {most} {expected}")
        s = lbfd.Solver(p).init_fields(q)
        L._check(L.load().lbfd_set_solve_group(s.h, most, expected), "lbfd_set_solve_group")
        s.step(3)
        assert_identical(s, full, f"{name} {most} {expected}")
        s.close()
    full.close()


@pytest.mark.parametrize("most,expected", GROUPS)
@pytest.mark.parametrize("shape", [(96, 40, 1), (33, 31, 1), (17, 15, 13), (150, 140, 1)])
def test_short_groups_of_a_batch(lbfd, shape, most, expected):  # noqa: F811
    inst = [case(shape, (P, P, P), 1.0, "fp64") for _ in range(3)]
    say(f"[group] batch {shape} {most} {expected}")
    b = lbfd.Batch([p for p, _ in inst])
    for m, (_, q) in zip(b.members, inst):
        m.init_fields(q)
    L._check(L.load().lbfd_batch_set_solve_group(b.b, most, expected), "lbfd_batch_set_solve_group")
    b.step(3)
    s = lbfd.Solver(inst[0][0]).init_fields(inst[0][1]).step(3)
    assert_identical(b[2], s, f"{shape} {most} {expected}")
    s.close()
    b.close()


def test_two_runs_on_two_streams(lbfd):  # noqa: F811
    """Solves that compete for the chip: whatever their groups are, the bits are those of a run alone."""
    import torch

    p, q = case((512, 512, 1), (P, P, P), 1.0, "fp64")
    alone = lbfd.Solver(p).init_fields(q).step(12)
    runs = [lbfd.Solver(p, stream=torch.cuda.Stream()).init_fields(q) for _ in range(3)]
    torch.cuda.synchronize()
    for _ in range(3):
        for s in runs:
            s.step(4)
    for i, s in enumerate(runs):
        assert_identical(s, alone, f"stream {i}")
        s.close()
    alone.close()


def test_group_arguments():
    assert L.load(build_if_missing=True).lbfd_set_solve_group(None, 1, 0) == L.LBFD_EINVAL
    assert L.load().lbfd_batch_set_solve_group(None, 1, 0) == L.LBFD_EINVAL
