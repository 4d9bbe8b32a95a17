"""Launch-shape autotuner of the solver.

The shapes it sweeps never change the results (each node's arithmetic and the
red-black order of the implicit solve are the same for every shape; the FP64
reductions keep a fixed shape):

* ``rows``: the step's node kernels (collision, macroscopic fields, geometry,
  FD right-hand sides, forces) run workgroups of 64 x rows nodes, a wavefront
  per row of 64 consecutive x; rows = 1, 2 or 4 trades LDS halo overhead of
  the staged kernels (66 x (rows + 2) cells per 64 x rows nodes) against
  workgroup count and occupancy;
* ``sor_wg_per_cu``: the persistent grid of the SOR half-sweeps, in workgroups
  of 256 per compute unit;
* ``sor_narrow``: the most workgroups of the one launch that runs the sweeps
  past the third (grids of more than one tile of 512 same-colour nodes per
  compute unit). A run that converges sooner does not use it, but its first
  steps and other runs of the same key do, so it is timed on the same workload
  with diffusivities that need more sweeps.

A batch uses ``rows`` alone.

Each candidate is timed over whole steps with HIP events on the solver's
stream (median of several timed regions); the fastest is stored per workload
key (lattice, storage, size class, batch size) in ``tuning.json`` next to this
module, which ``Solver`` and ``Batch`` read at creation.
"""
from __future__ import annotations

import itertools
import json
import os

import numpy as np

from . import lbfd

ROWS = (1, 2, 4)
SOR_WG_PER_CU = (2, 4, 8, 16)
SOR_NARROW = (64, 128, 256)
LEAD = 3            # sweeps by launches before the persistent launch
DIFFUSIVITY = 0.5   # of both surfactants: some five sweeps a step on the bubble column


def _time(obj, steps: int, regions: int) -> float:
    """Median milliseconds per step over `regions` timed regions of `steps` steps."""
    import torch

    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    runs = []
    for _ in range(regions):
        torch.cuda.synchronize()
        a.record()
        obj.step(steps)
        b.record()
        torch.cuda.synchronize()
        runs.append(a.elapsed_time(b) / steps)
    return float(np.median(runs))


def _sweep(obj, shapes, steps: int, regions: int) -> list:
    """(milliseconds per step, shape) of each shape."""
    table = []
    for t in shapes:
        obj.set_tuning(t).step(4)          # captures the graphs of this shape
        table.append((_time(obj, steps, regions), t))
    return table


def _entry(key, table, default_ms) -> dict:
    best_ms, best = min(table, key=lambda r: r[0])
    return dict(key=key, tuning=best, ms_per_step=round(best_ms, 4), default_ms_per_step=round(default_ms, 4),
                candidates=[dict(t, ms_per_step=round(ms, 4)) for ms, t in table])


def tune_narrow(params: dict, init: dict, steps: int, warmup: int, regions: int) -> list:
    """The grids of the persistent launch, timed on the workload with more diffusion: empty where
    its solve still needs no more than the launched sweeps (the default serves there)."""
    p = dict(params, Ds=DIFFUSIVITY, Db=DIFFUSIVITY)
    p["sor_max_sweeps"] = max(p["sor_max_sweeps"], 60)
    s = lbfd.Solver(p, tuning=None).init_fields(init).step(warmup)
    table = _sweep(s, [dict(lbfd.DEFAULT_TUNING, sor_narrow=n) for n in SOR_NARROW], steps, regions)
    used = max(s.observables()["sor_sweeps"])
    s.close()
    return table if used > LEAD else []


def tune_solver(params: dict, init: dict, steps: int = 20, warmup: int = 6, regions: int = 3) -> dict:
    """Sweep rows x SOR grid on one solver of the workload, and the persistent launch's grid on
    one that uses it."""
    narrow = tune_narrow(params, init, steps, warmup, regions)
    nar = min(narrow, key=lambda r: r[0])[1]["sor_narrow"] if narrow else lbfd.DEFAULT_TUNING["sor_narrow"]
    s = lbfd.Solver(params, tuning=None).init_fields(init).step(warmup)
    table = _sweep(s, [dict(rows=r, sor_wg_per_cu=wg, sor_narrow=nar) for r, wg in
                       itertools.product(ROWS, SOR_WG_PER_CU)], steps, regions)
    s.set_tuning(lbfd.DEFAULT_TUNING).step(4)
    default_ms = _time(s, steps, regions)
    if s.observables()["status"] != 0:
        raise RuntimeError("solver error while tuning")
    s.close()
    e = _entry(lbfd.tuning_key(params), table, default_ms)
    if narrow:
        e["narrow"] = [dict(sor_narrow=t["sor_narrow"], ms_per_step=round(ms, 4)) for ms, t in narrow]
    return e


def tune_batch(params_list, inits, steps: int = 10, warmup: int = 4, regions: int = 3) -> dict:
    """Sweep the rows of a batch's node kernels (its solve follows from the instances alone)."""
    b = lbfd.Batch(params_list, tuning=None)
    for m, q in zip(b.members, inits):
        m.init_fields(q)
    b.step(warmup)
    table = _sweep(b, [dict(lbfd.DEFAULT_TUNING, rows=r) for r in ROWS], steps, regions)
    b.set_tuning(lbfd.DEFAULT_TUNING).step(4)
    default_ms = _time(b, steps, regions)
    key = b.key
    b.close()
    return _entry(key, table, default_ms)


def write(results, path: str = lbfd.TUNING_FILE, device: str = "") -> dict:
    """Merge tuned entries into the table at `path`."""
    table = dict(entries={})
    if os.path.exists(path):
        with open(path) as fh:
            table = json.load(fh)
    for r in results:
        table["entries"][r["key"]] = dict({k: v for k, v in r.items() if k != "key"}, device=device)
    with open(path, "w") as fh:
        json.dump(table, fh, indent=1, sort_keys=True)
        fh.write("\n")
    return table
