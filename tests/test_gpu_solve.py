"""The implicit solve by launches and by the persistent launch.

Which of the two takes a sweep depends on the grid (and, in a batch, on the
largest instance). The rows, their red-black order (with the seam classes of odd
periodic extents) and the stopping test are the same, so a grid must give the
same bits either way (the launches follow the FP64 oracle in the parity tests)."""
import pytest

import workloads as W
from tests.parity import say
from tests.test_gpu_batch import assert_identical, lbfd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

P, WALL = W.PERIODIC, W.WALL
# a workgroup of the persistent solve takes 512 nodes of a colour; 32 of them share an XCD, 256 the chip
GRIDS = {
    "one_tile": (32, 32, 1, (P, P, P), 1.0),
    "remainder_seams": (33, 31, 1, (P, P, P), 1.2),
    "last_near": (128, 256, 1, (P, WALL, P), 1.0),
    "first_far_seam": (128, 257, 1, (P, P, P), 1.0),
    "last_far": (512, 512, 1, (P, P, P), 1.2),
    "first_launched_seam": (512, 513, 1, (WALL, P, P), 1.0),
    "near_3d_seams": (33, 31, 29, (P, P, P), 1.0),
    "far_3d": (64, 34, 36, (WALL, P, WALL), 1.0),
    "far_3d_seams": (65, 33, 35, (P, P, P), 1.2),
    "launched_3d_seams": (81, 81, 81, (P, P, P), 1.0),
    "launched_3d_edge": (80, 81, 83, (P, P, P), 1.0),
}


def case(shape, bc, omega, prec):
    nx, ny, nz = shape
    three = nz > 1
    p = dict(lattice=W.D3Q19 if three else W.D2Q9, nx=nx, ny=ny, nz=nz, bc=list(bc), rhoR0=0.5, muR0=0.1,
             sigma0=0.01, E0=0.4, Ds=0.3, Db=0.2, ra=0.05, rd=0.01, sor_omega=omega, precision=prec)
    r = min(nx, ny, nz if three else nx) / 4.0
    # the drop crosses the last planes, where the seam classes are
    return W.make(p, dict(drops=[(nx - 1 - 0.6 * r, ny - 1 - 0.6 * r, nz - 1 - 0.6 * r if three else 0.0, r)], width=3.0,
                          psi0=0.2, phi0_out=0.06, phi0_in=0.01))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(GRIDS))
def test_launched_and_persistent_solves_agree(lbfd, name, prec):  # noqa: F811
    nx, ny, nz, bc, omega = GRIDS[name]
    p, q = case((nx, ny, nz), bc, omega, prec)
    # a second instance of more than 32 x 512 nodes of a colour: the batch starts by launches
    other = case((96, 90, 8) if nz > 1 else (256, 140, 1), (P, P, P), omega, prec)
    steps = 3
    say(f"[solve] {name} {nx}x{ny}x{nz} omega {omega} {prec}")
    s = lbfd.Solver(p).init_fields(q).step(steps)
    b = lbfd.Batch([p, other[0]])
    b[0].init_fields(q)
    b[1].init_fields(other[1])
    b.step(steps)
    sweeps = s.observables()["sor_sweeps"]
    say("sweeps", sweeps)
    assert_identical(b[0], s, name)
    assert max(sweeps) > 3   # past the sweeps that are launches everywhere
    b.close()
    s.close()


def test_small_batches_solve_persistently(lbfd):  # noqa: F811
    """More instances than groups of the persistent solve (256): a group takes several."""
    inst = [case((16 + i % 7, 12 + i % 5, 1), (P, P, P), 1.0, "fp64") for i in range(300)]
    b = lbfd.Batch([p for p, _ in inst])
    for m, (_, q) in zip(b.members, inst):
        m.init_fields(q)
    b.step(4)
    for i in (0, 37, 255, 256, 299):
        s = lbfd.Solver(inst[i][0]).init_fields(inst[i][1]).step(4)
        assert_identical(b[i], s, f"instance {i}")
        s.close()
    b.close()
