"""Results to the last bit.

In the 32-bit modes a rounding that changes in one kernel reaches every field
within a few steps, and 16-bit populations (stored with stochastic rounding)
carry it to 1e-4 of the colour function in some hundred. So the digests below
hold the bits of whole runs: SHA-1 of the fields as FP64 arrays, recorded on
gfx950 (ROCm 7.2) with kernels that gathered every operand from memory and formed
both one-sided differences of a line at every node. Fields that hold FP64 sums
(the surfactant total scales psi and phi as they are read) are not among them,
nor are FP64 runs, where that scale enters the step."""
import hashlib

import pytest

import workloads as W
from tests.parity import say
from tests.test_gpu_batch import lbfd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

P, WALL = W.PERIODIC, W.WALL
FIELDS = ("f", "rhoN", "u", "G", "force", "Sprev", "Bprev")


def box(nx, ny, nz, bc, prec):
    """A drop off the centre of a box, in a body force along every axis."""
    three = nz > 1
    p = dict(lattice=W.D3Q19 if three else W.D2Q9, nx=nx, ny=ny, nz=nz, bc=list(bc), rhoR0=0.5, muR0=0.1,
             sigma0=0.01, E0=0.4, Ds=0.3, Db=0.2, ra=0.05, rd=0.01, gravity=[2e-4, -3e-4, 1e-4 if three else 0.0],
             precision=prec)
    r = min(nx, ny, nz if three else ny) / 4.0
    return W.make(p, dict(drops=[((nx - 1) / 2.0 + 1.3, (ny - 1) / 2.0 - 0.7, (nz - 1) / 2.0 if three else 0.0, r)],
                          width=3.0, psi0=0.2, phi0_out=0.06, phi0_in=0.01))


RUNS = {
    "shear_fp32": (lambda: W.shear_droplet(nx=200, ny=101, radius=16.0, precision="fp32"), 40),
    "box2d_fp32": (lambda: box(133, 131, 1, (P, P, P), "fp32"), 10),
    "box3d_fp32": (lambda: box(67, 35, 30, (P, P, WALL), "fp32"), 12),
    "column_bf16dev": (lambda: W.bubble_rise(nx=40, ny=37, nz=80, radius=5.0, precision="bf16dev"), 30),
    "box3d_fp16dev": (lambda: box(33, 31, 29, (P, P, P), "fp16dev"), 12),
    "bubble2d_bf16dev": (lambda: W.bubble_rise(nx=70, ny=131, nz=1, radius=9.0, lattice=W.D2Q9,
                                               precision="bf16dev"), 40),
}
DIGEST = {
    "shear_fp32": "b3c702b2e4a0613a",
    "box2d_fp32": "c5f93f4a9a9c492d",
    "box3d_fp32": "947d672bd6d29f10",
    "column_bf16dev": "266eadf272e95fd4",
    "box3d_fp16dev": "f584751d23c7186f",
    "bubble2d_bf16dev": "d8d8ce0b294ca75a",
}


def digest(fields):
    h = hashlib.sha1()
    for a in fields:
        h.update(a.tobytes())
    return h.hexdigest()[:16]


@pytest.mark.parametrize("name", sorted(RUNS))
def test_runs_keep_their_bits(lbfd, name):  # noqa: F811
    make, steps = RUNS[name]
    p, q = make()
    s = lbfd.Solver(p).init_fields(q).step(steps)
    got = digest(s.field(f) for f in FIELDS)
    say(f"[rounding] {name}: {got}")
    s.close()
    assert got == DIGEST[name]
