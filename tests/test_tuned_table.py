"""The stored table of launch shapes serves every run of its keys."""
import json

import pytest

import workloads as W
from paper_2311_15242_amd import lbfd as L
from tests.parity import say
from tests.test_gpu_batch import lbfd  # noqa: F401  (the fixture)


def entries():
    with open(L.TUNING_FILE) as fh:
        return json.load(fh)["entries"]


def test_batches_are_tuned_over_what_they_use():
    """A batch uses the rows alone: candidates that differ in nothing else would store noise."""
    for key, e in entries().items():
        if key.startswith("batch"):
            rows = [c["rows"] for c in e["candidates"]]
            assert sorted(rows) == sorted(set(rows)), key
            assert dict(e["tuning"], rows=0) == dict(L.DEFAULT_TUNING, rows=0), key


def runs(key):
    """A run of a solver's key with enough diffusion that its solve goes past the launched sweeps."""
    lat, prec, n = key.split("/")
    nodes = 2 ** int(n.split("^")[1])
    if lat == "D3Q19":
        nx = 32
        while nx ** 3 * 3 < nodes * 0.75:
            nx += 16
        p, q = W.bubble_rise(nx=nx, ny=nx, nz=3 * nx, radius=nx / 8.0, precision=prec)
    else:
        nx = int(nodes ** 0.5) // 16 * 16
        p, q = W.droplet_adsorption(n=nx, radius=nx / 5.0, precision=prec)
    assert L.tuning_key(p) == key
    return dict(p, Ds=0.5, Db=0.5), q


@pytest.mark.gpu
@pytest.mark.parametrize("key", sorted(k for k in entries() if not k.startswith("batch")))
def test_tuned_shape_serves_a_solve_of_many_sweeps(lbfd, key):  # noqa: F811
    """Time of a step under the stored shape against the default one (1.02 and less for a shape that is
    the faster; 1.9 with 64 workgroups in the persistent launch of the bubble column)."""
    import torch

    p, q = runs(key)
    ms = []
    for tuning in ("auto", None):
        s = lbfd.Solver(p, tuning=tuning).init_fields(q).step(4)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        t = []
        for _ in range(3):
            a.record()
            s.step(6)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b) / 6)
        ms.append(min(t))
        sweeps = s.observables()["sor_sweeps"]
        say(f"[tuned] {key} {tuning}: {ms[-1]:.3f} ms a step, sweeps {sweeps}")
        assert max(sweeps) > 3
        s.close()
    assert ms[0] < 1.1 * ms[1]
