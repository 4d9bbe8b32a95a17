"""The explicit transport terms on the grids where their tiles end.

The convection of a node reads two nodes along each axis, x and y from the
workgroup's staged cross and z from memory, and takes one upwind difference
away from the band of zero velocity and both inside it. Sprev and Bprev are
those terms alone: against the FP64 oracle's after two steps (the first one
starts at rest, so part of the grid is in the band)."""
import pytest

import oracle
import workloads as W
from tests.parity import rel, say
from tests.test_gpu_batch import lbfd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

P, WALL = W.PERIODIC, W.WALL
# workgroups of 64 x by 1, 2 or 4 rows; 4 nodes is the smallest extent
GRIDS = {
    "smallest": (4, 4, 1, (P, P, P)),
    "smallest_walls": (4, 5, 1, (WALL, WALL, P)),
    "below_a_tile": (63, 7, 1, (P, WALL, P)),
    "a_tile": (64, 8, 1, (WALL, P, P)),
    "above_a_tile": (65, 9, 1, (P, P, P)),
    "overhang": (130, 6, 1, (WALL, WALL, P)),
    "smallest_3d": (4, 4, 4, (P, P, P)),
    "walls_3d": (5, 6, 7, (WALL, WALL, WALL)),
    "overhang_3d": (67, 5, 4, (P, P, WALL)),
}


# FP64: relative changes of 1e-14 of the parameters change the oracle's terms by up to 2e-13; the
# two sides differ by rounding (some 1e-15) and by what the solve's tolerance of 1e-13 leaves
TOL = 1e-10


@pytest.mark.parametrize("rows", [1, 2, 4])
@pytest.mark.parametrize("name", sorted(GRIDS))
def test_transport_terms_follow_the_oracle(lbfd, name, rows):  # noqa: F811
    nx, ny, nz, bc = GRIDS[name]
    three = nz > 1
    p = dict(lattice=W.D3Q19 if three else W.D2Q9, nx=nx, ny=ny, nz=nz, bc=list(bc), rhoR0=0.5, muR0=0.1,
             sigma0=0.01, E0=0.4, Ds=0.3, Db=0.2, ra=0.05, rd=0.01, gravity=[2e-4, -3e-4, 1e-4 if three else 0.0],
             precision="fp64")
    r = min(nx, ny, nz if three else ny) / 3.0
    p, q = W.make(p, dict(drops=[((nx - 1) / 2.0, (ny - 1) / 2.0, (nz - 1) / 2.0, r)], width=1.5, psi0=0.2,
                          phi0_out=0.06, phi0_in=0.01))
    say(f"[transport] {name} {nx}x{ny}x{nz} rows {rows}")
    s = lbfd.Solver(p).init_fields(q)
    s.set_tuning(dict(rows=rows))
    s.step(2)
    o = oracle.Oracle(p).init(q).step(2)
    for f in ("Sprev", "Bprev"):
        e = rel(s.field(f), o.field(f))
        say(f, e)
        assert e < TOL
