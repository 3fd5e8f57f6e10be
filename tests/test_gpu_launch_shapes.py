"""The launch shapes that the runtime chooses by itself, and slots of which only
a part of the lanes take rows: bit-identical to the oracle."""
from __future__ import annotations

import math
import sys

import numpy as np
import pytest

from oracle import oracle as eo
from paper_2304_03311_amd import ee

BC2 = 0.5 * math.log(1.0 + math.sqrt(2.0))
BC3 = 0.2216546

pytestmark = pytest.mark.gpu


def check(s: ee.JobSpec, cfg, n_therm: int = 2):
    print(f"[gpu] {s} {cfg}", file=sys.stderr, flush=True)
    I, sp = eo.run(eo.Job(s.dim, s.lt, s.lx, s.ly, s.n, s.beta, s.l, s.n_step, s.n_traj, s.seed, s.reverse,
                          s.subsets, s.whole), n_therm, want_spins=True)
    j = ee.Job(s)
    j.set_launch(cfg)
    j.thermalize(n_therm)
    j.run_protocol()
    assert np.array_equal(j.work(), I) and np.array_equal(j.spins(), sp)
    j.close()
    j = ee.Job(s)
    ee.batch_run([j], n_therm, cfg=cfg)
    assert np.array_equal(j.work(), I) and np.array_equal(j.spins(), sp)
    j.close()


@pytest.mark.parametrize("kw", [
    dict(dim=2, lt=8, lx=8, ly=1, n=2, beta=BC2, l=3, n_step=3, n_traj=9001),  # several per wave, one row per lane
    dict(dim=2, lt=64, lx=32, ly=1, n=2, beta=BC2, l=11, n_step=2, n_traj=8193),  # two per wave
    dict(dim=2, lt=48, lx=48, ly=1, n=3, beta=BC2, l=30, n_step=2, n_traj=520),  # three lanes per row
    dict(dim=2, lt=16, lx=16, ly=1, n=2, beta=BC2, l=4, n_step=4, n_traj=1),
    dict(dim=3, lt=32, lx=32, ly=32, n=2, beta=BC3, l=9, n_step=2, n_traj=3),  # a wide workgroup per trajectory
    dict(dim=3, lt=6, lx=22, ly=10, n=2, beta=BC3, l=5, n_step=10, n_traj=300, subsets=True),
], ids=["8x8", "64x32", "48x48_n3", "16x16_one", "32cube", "ragged"])
def test_runtime_shapes_match_oracle(kw):
    check(ee.JobSpec(seed=91, **kw), None)


@pytest.mark.parametrize("block", [512, 576, 1024])
def test_slots_with_idle_lanes_match_oracle(block):
    # 24 wide in y: 512 lanes hold 256 row slots per replica, of which 240 take
    # rows in parity-major order; 1024 lanes 504 of 512
    check(ee.JobSpec(dim=3, lt=24, lx=24, ly=24, n=2, beta=BC3, l=7, n_step=3, n_traj=3, seed=92, reverse=True),
          dict(block_threads=block, lds_bytes=28672))


# Rows whose words do not fill their lanes: pad sites, the edge neighbours of
# the first and last lane, glued and ramped columns in the last word.  64 and
# 192 lanes per trajectory hold fewer row slots than rows, so the rows go in
# parity-major order.
@pytest.mark.parametrize("block", [64, 192])
@pytest.mark.parametrize("lx", [2, 6, 10, 14, 18, 20, 22, 26, 30, 34, 40, 44, 50, 56, 58, 62, 100])
@pytest.mark.parametrize("dim", [2, 3])
def test_rows_with_pad_sites_match_oracle(dim, lx, block):
    kw = dict(dim=2, lt=200, ly=1, beta=BC2, n_step=4) if dim == 2 else dict(dim=3, lt=14, ly=10, beta=BC3, n_step=10)
    for k, opts in enumerate((dict(l=lx - 1), dict(l=lx // 2, reverse=True, spin_format=1), dict(l=lx, whole=True),
                              dict(l=max(1, lx - 3), n=3, subsets=dim == 3))):
        s = ee.JobSpec(lx=lx, n_traj=2, seed=200 + 4 * lx + k, **{"n": 2, **kw, **opts, "l": min(
            opts["l"], lx if opts.get("whole") else lx - 1)})
        if 2 * s.n * s.lt * s.ly * -(-lx // 8) * 4 <= 160 * 1024 - 256:
            check(s, dict(block_threads=block, lds_bytes=1024), n_therm=1)


def test_noalloc_batch_of_more_units_than_its_scratch_holds():
    # accepted (ten of these trajectories in 80 KB), and run one to a workgroup:
    # 136,070 units of 16 bytes, in two pieces
    specs = [ee.JobSpec(dim=2, lt=64, lx=64, ly=1, n=2, beta=BC2, l=9, n_step=1, n_traj=n, seed=88 + i)
             for i, n in enumerate((65535, 65535, 5000))]
    out = []
    for run in (ee.batch_run_noalloc, ee.batch_run):
        jobs = [ee.Job(s) for s in specs]
        run(jobs, 0, cfg=None)
        out.append([(j.work(), j.estimate().dF) for j in jobs])
        for j in jobs:
            j.close()
    for (wa, fa), (wb, fb) in zip(*out):
        assert np.array_equal(wa, wb) and fa == fb
