"""The estimator at the trajectory counts where its launches change: one
workgroup up to 895 trajectories, several launches above, waves of 64
leave-one-out sums, groups of 16 terms; alone and in a batch of mixed
counts.  Against the definition evaluated on the job's works: the operations
and their order are the same, so mean and variance of W are equal, and the
others differ only where the host's exp or log rounds the other way (one ulp
each, 1e-12 in the results)."""
from __future__ import annotations

import math
import sys

import pytest

from oracle import oracle as eo
from paper_2304_03311_amd import ee

pytestmark = pytest.mark.gpu
BC2 = 0.5 * math.log(1.0 + math.sqrt(2.0))


def spec(n: int, seed: int) -> ee.JobSpec:
    return ee.JobSpec(dim=2, lt=4, lx=8, ly=1, n=3, beta=BC2, l=3, n_step=5, n_traj=n, seed=seed)


def check(j: ee.Job):
    s, r, I = j.spec, j.estimate(), j.work()
    e = eo.estimate(I, s.beta, s.S, s.n)
    assert abs(r.dF - e.dF) <= 1e-12 * max(abs(e.dF), 1e-3)
    assert abs(r.dS - e.dS) <= 1e-12 * max(abs(e.dS), 1e-3)
    assert (r.w_mean, r.w_var, r.i_min, r.i_max, r.n_traj) == (e.w_mean, e.w_var, e.i_min, e.i_max, s.n_traj)
    assert r.ess == pytest.approx(e.ess, rel=1e-12)
    if s.n_traj == 1:
        assert math.isnan(r.dF_err)
    else:
        assert r.dF_err == pytest.approx(e.dF_err, rel=1e-12, abs=1e-300)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 894, 895, 896, 897, 960, 1023, 1024, 1025, 4097])
def test_estimate_at_every_launch_edge(n):
    print(f"[gpu] estimator n = {n}", file=sys.stderr, flush=True)
    j = ee.Job(spec(n, n))
    j.thermalize(2)
    j.run_protocol()
    check(j)
    j.close()


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("counts", [(3, 1, 64, 895), (896, 2, 1, 2050, 257)], ids=["small", "mixed"])
def test_estimates_of_a_batch(counts, graph):
    print(f"[gpu] estimators of a batch {counts} graph {graph}", file=sys.stderr, flush=True)
    jobs = [ee.Job(spec(n, 100 + n)) for n in counts]
    for _ in range(3):  # the recorded launches are replayed
        for j in jobs:
            j.reset()
        ee.batch_run(jobs, 2, cfg=dict(use_graph=graph))
        for j in jobs:
            check(j)
    for j in jobs:
        j.close()
