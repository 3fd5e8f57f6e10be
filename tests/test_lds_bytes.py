"""LDS bytes of a trajectory: rows with pad sites are kept at a pitch of whole
lanes, and the launch shapes that the tuner offers are sized by it."""
from __future__ import annotations

import pytest

from paper_2304_03311_amd import autotune, ee


def spec(dim, lx, **kw):
    return ee.JobSpec(**{**dict(dim=dim, lt=12, lx=lx, ly=1 if dim == 2 else 4, n=2, beta=0.3, l=1, n_step=4, n_traj=9,
                                seed=1), **kw})


# sites in x: words of a row on chip (stored: lx / 8 rounded up)
PITCH = {2: 1, 6: 1, 8: 1, 10: 2, 16: 2, 18: 3, 22: 3, 24: 3, 26: 4, 32: 4, 34: 6, 36: 6, 40: 6, 48: 6, 50: 8, 56: 8,
         58: 8, 64: 8, 100: 14, 128: 16}


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("lx", PITCH)
def test_bytes_of_a_trajectory(dim, lx):
    s = spec(dim, lx)
    want = 2 * 2 * 12 * s.ly * PITCH[lx] * 4
    assert ee.ee_job_lds_bytes(s.desc()) == want
    assert autotune.traj_bytes(s) == want


@pytest.mark.parametrize("lx", [34, 40, 50, 56, 64])
def test_offered_shapes_hold_one_to_four_trajectories(lx):
    s = spec(2, lx, lt=40)
    one = ee.ee_job_lds_bytes(s.desc())
    for block in (64, 128):
        held = {c["lds_bytes"] // one for c in autotune.candidates_for([s]) if c["block_threads"] == block}
        assert {1, 2, 3, 4} <= held


def test_padded_only_where_it_fits():
    # 160 KB - 256 B hold this lattice as stored (5 words a row), not at 6
    s = spec(2, 40, lt=2000)
    assert ee.ee_job_on_chip(s.desc()) and ee.ee_job_lds_bytes(s.desc()) == 2 * 2 * 2000 * 5 * 4
    with pytest.raises(ee.EEError):
        ee.ee_job_lds_bytes(spec(2, 7).desc())
