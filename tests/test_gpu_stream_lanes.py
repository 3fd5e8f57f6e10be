"""Rows and lanes of the streaming sweep kernel: one row per lane on small jobs, two
on large ones (against the on-chip kernels on the same job: the chains are
bit-identical), every width of a lane, rows with pad sites, partly idle workgroups."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from paper_2304_03311_amd import ee

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(dim=2, lt=32, lx=32, ly=1, n=2, n_traj=16500),  # four words per lane, two rows
    dict(dim=2, lt=34, lx=24, ly=1, n=3, n_traj=10400),  # three
    dict(dim=2, lt=16, lx=16, ly=1, n=2, n_traj=33000),  # two
    dict(dim=2, lt=32, lx=8, ly=1, n=2, n_traj=16500),   # one
    dict(dim=2, lt=10, lx=22, ly=1, n=2, n_traj=17600),  # three lanes per row, pad sites
    dict(dim=3, lt=12, lx=32, ly=10, n=2, n_traj=4400),
    dict(dim=3, lt=6, lx=8, ly=10, n=2, n_traj=9000),
    dict(dim=3, lt=6, lx=14, ly=10, n=3, n_traj=3000),
    dict(dim=3, lt=6, lx=24, ly=6, n=2, n_traj=3, reverse=True),  # one row per lane from here
    dict(dim=3, lt=10, lx=18, ly=6, n=2, n_traj=5, subsets=True),
    dict(dim=2, lt=126, lx=80, ly=1, n=2, n_traj=3, whole=True),
], ids=lambda kw: f"{kw['lt']}x{kw['lx']}x{kw['ly']}_n{kw['n']}")
@pytest.mark.parametrize("l", [0, 5])
def test_streamed_rows_match_on_chip(kw, l):
    if kw.get("whole"):
        l = max(1, l)
    s = ee.JobSpec(beta=0.4406867935097715 if kw["dim"] == 2 else 0.2216546, l=l, n_step=12, seed=300 + l, **kw)
    print(f"[gpu] {s}", file=sys.stderr, flush=True)
    out = []
    for cfg in ({"flags": ee.EE_LAUNCH_STREAMING | ee.EE_LAUNCH_TWO_PASS}, None):
        j = ee.Job(s)
        if cfg:
            j.set_launch({"block_threads": 0, "lds_bytes": 0, "grid_blocks": 0, "use_graph": 0, **cfg})
        j.thermalize(2)
        j.run_protocol()
        out.append((j.work(), j.spins()))
        j.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
