"""Routes that depend on the size of a set, each on both sides of where it
changes (tests/test_runtime_host.py asserts that these sizes take them): a batch
without allocation in one and in two pieces, streamed jobs of one and of two
rows per lane."""
from __future__ import annotations

import math
import sys

import numpy as np
import pytest

from paper_2304_03311_amd import ee

BC2 = 0.5 * math.log(1.0 + math.sqrt(2.0))
BC3 = 0.2216546

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(65535, 5000), (65535, 65535, 5000)], ids=["one_piece", "two_pieces"])
def test_noalloc_pieces_match_batch(counts):
    print(f"[gpu] noalloc batch {counts}", file=sys.stderr, flush=True)
    specs = [ee.JobSpec(dim=2, lt=128, lx=64, ly=1, n=2, beta=BC2, l=9, n_step=1, n_traj=n, seed=88 + i)
             for i, n in enumerate(counts)]
    out = []
    for run in (ee.batch_run_noalloc, ee.batch_run):
        jobs = [ee.Job(s) for s in specs]
        run(jobs, 0, cfg=None)
        out.append([(j.work(), j.estimate().dF, j.estimate().dF_err, j.spins(3)) for j in jobs])
        for j in jobs:
            j.close()
    for a, b in zip(*out):
        assert np.array_equal(a[0], b[0]) and a[1:3] == b[1:3] and np.array_equal(a[3], b[3])


@pytest.mark.parametrize("more", [0, 1], ids=["one_row", "two_rows"])
@pytest.mark.parametrize("kw,per_traj", [
    (dict(dim=2, lt=32, lx=32, ly=1, n=2), 64), (dict(dim=2, lt=34, lx=24, ly=1, n=3), 102),
    (dict(dim=2, lt=32, lx=8, ly=1, n=2), 64), (dict(dim=3, lt=12, lx=32, ly=10, n=2), 240),
    (dict(dim=3, lt=6, lx=14, ly=10, n=3), 360)], ids=lambda v: "x".join(map(str, v.values())) if isinstance(v, dict) else "")
def test_rows_per_lane_match_on_chip(kw, per_traj, more):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    s = ee.JobSpec(beta=BC2 if kw["dim"] == 2 else BC3, l=3, n_step=6, n_traj=4 * cus * 1024 // per_traj + more, seed=310, **kw)
    print(f"[gpu] {s}", file=sys.stderr, flush=True)
    out = []
    for flags in (ee.EE_LAUNCH_STREAMING | ee.EE_LAUNCH_TWO_PASS, 0):
        j = ee.Job(s)
        j.set_launch({"flags": flags})
        j.thermalize(1)
        j.run_protocol()
        out.append((j.work(), j.spins()))
        j.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
