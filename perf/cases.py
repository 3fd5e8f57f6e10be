"""The workloads on which this framework's speed is measured.

Each case is one estimate, or one set of estimates, of entropy increments as
a program makes it: jobs are described and created once (`prepare`), then a
pass (`run`) redraws every spin and uniform on the device, thermalises,
drives the protocol and reads the results and the integer works.

Kinds of case:
  job     one job through the per-job calls (thermalise, protocol, estimate)
  batch   the increments l = 0, 1, ... of one lattice in one persistent launch
  uneven  a seeded set of lattices of several sizes and protocol lengths in
          one persistent launch
  serve   requests of the serving mix through the serving loop, all at once
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np

from paper_2304_03311_amd import autotune, ee, serve, workloads

B2, B3 = workloads.BETA_C_2D, workloads.BETA_3D


def listed():
    return [
        # the smallest call: a first look at one increment, a handful of
        # trajectories; launches and latency only.  The final spins are read too
        {"name": "job_2d16_8traj", "kind": "job", "dim": 2, "lt": 16, "ly": 1, "lx": 16, "n": 2, "l": 4,
         "n_step": 32, "n_traj": 8, "n_therm": 10, "spins": True},
        # the small latency-bound configuration: 64 trajectories of 16 x 16
        {"name": "batch_2d16_64traj", "kind": "batch", "dim": 2, "lt": 16, "ly": 1, "lx": 16, "n": 2, "l": 4,
         "jobs": 1, "n_step": 256, "n_traj": 64, "n_therm": 100},
        # ragged: 22 sites in x (rows that end inside a word), three replicas,
        # the reverse ramp row by row, bit-packed storage
        {"name": "job_3d_ragged_n3", "kind": "job", "dim": 3, "lt": 10, "ly": 6, "lx": 22, "n": 3, "l": 9,
         "n_step": 60, "n_traj": 64, "n_therm": 20, "packed": True, "reverse": True, "subsets": True},
        # the headline set: S_2(1..64) of the 64 x 64 lattice, 64 jobs
        {"name": "batch_2d64_64jobs", "kind": "batch", "dim": 2, "lt": 64, "ly": 1, "lx": 64, "n": 2, "l": 0,
         "jobs": 64, "n_step": 1000, "n_traj": 1024, "n_therm": 100},
        # one 3D increment, bit-packed: a whole workgroup's LDS per trajectory
        {"name": "batch_3d32_packed", "kind": "batch", "dim": 3, "lt": 32, "ly": 32, "lx": 32, "n": 2, "l": 8,
         "jobs": 1, "n_step": 2000, "n_traj": 512, "n_therm": 100, "packed": True},
        # 24 jobs of eight lattices and three protocol lengths in one launch
        {"name": "uneven_24jobs", "kind": "uneven", "n_traj": 256, "n_therm": 100, "scale": 1.0},
        # a zero-temperature cylinder of the physics campaign (L_tau = 8 L),
        # every increment, the library's own launch shape
        {"name": "batch_2d32_cylinder", "kind": "batch", "dim": 2, "lt": 256, "ly": 1, "lx": 32, "n": 2, "l": 0,
         "jobs": 32, "n_step": 200, "n_traj": 256, "n_therm": 400},
        # the thermalisation scan: one increment at very many trajectories,
        # where the estimator's leave-one-out sums count
        {"name": "job_2d32_16384traj", "kind": "job", "dim": 2, "lt": 64, "ly": 1, "lx": 32, "n": 2, "l": 3,
         "n_step": 200, "n_traj": 16384, "n_therm": 100},
        # lattices larger than a workgroup's LDS, streamed: the largest of the
        # serving mix in the benchmark's trajectory count, ...
        {"name": "stream_3d96_32traj", "kind": "job", "dim": 3, "lt": 96, "ly": 96, "lx": 96, "n": 2, "l": 40,
         "n_step": 100, "n_traj": 32, "n_therm": 10},
        # ... a small streamed job as the serving mix sends them, ...
        {"name": "stream_3d48_16traj", "kind": "job", "dim": 3, "lt": 48, "ly": 48, "lx": 48, "n": 2, "l": 17,
         "n_step": 500, "n_traj": 16, "n_therm": 100},
        # ... and one increment of the L = 128 cylinder of the campaign
        {"name": "stream_2d128_cylinder", "kind": "job", "dim": 2, "lt": 1024, "ly": 1, "lx": 128, "n": 2, "l": 31,
         "n_step": 100, "n_traj": 256, "n_therm": 100},
        # 48 requests of the serving mix, all there at once
        {"name": "serve_48_requests", "kind": "serve", "requests": 48, "mix": 1, "n_therm": 100},
    ]


# attempts of a drawn case at most; the headline set has 5.9e11
DRAW_MOST = 3e11
# a trajectory of at most so many bytes (rows padded to whole words) stays in
# a workgroup's LDS
ON_CHIP = 160 * 1024 - 256


def _padded(n, lt, ly, lx):
    return 2 * n * lt * ly * -(-lx // 8) * 4


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def even(lo, hi):
        return max(2, 2 * int(round(log_int(lo, hi) / 2)))

    while True:
        kind = rng.choice(["job", "job", "job", "batch", "batch", "stream", "uneven", "serve"])
        if kind == "serve":
            return {"kind": "serve", "requests": rng.randint(4, 40), "mix": rng.randint(2, 10 ** 6),
                    "n_therm": rng.choice([50, 100])}
        if kind == "uneven":
            return {"kind": "uneven", "n_traj": log_int(16, 256), "n_therm": rng.choice([20, 50, 100]),
                    "scale": round(rng.uniform(0.1, 1.0), 3)}
        dim = rng.choice([2, 3])
        c = {"kind": kind, "dim": dim, "n": rng.choice([2, 2, 2, 3])}
        if kind == "stream":
            lx = even(40, 96) if dim == 3 else even(128, 256)
            ly = lx if dim == 3 else 1
            lt = even(40, 96) if dim == 3 else 8 * lx
            c["kind"], c["n"] = "job", 2
            if _padded(c["n"], lt, ly, lx) <= ON_CHIP:
                continue
            n_traj, n_step, n_therm = log_int(4, 64), log_int(20, 300), rng.randint(0, 50)
        else:
            lx = even(6, 128) if dim == 2 else even(4, 40)
            ly = even(4, 32) if dim == 3 else 1
            lt = (8 * lx if rng.random() < 0.3 and lx <= 32 else even(6, 128)) if dim == 2 else even(4, 40)
            if _padded(c["n"], lt, ly, lx) > ON_CHIP:
                continue
            n_traj, n_step, n_therm = log_int(4, 4096), log_int(16, 1000), rng.randint(0, 200)
        c |= {"lt": lt, "ly": ly, "lx": lx, "n_step": n_step, "n_traj": n_traj, "n_therm": n_therm}
        jobs = 1
        if kind == "batch":
            jobs = c["jobs"] = rng.randint(1, min(lx, 32))
            c["l"] = rng.randint(0, lx - jobs)
        else:
            c["l"] = rng.randint(0, lx - 1)
            if kind == "job":
                c["reverse"] = rng.random() < 0.3
                if dim == 3 and rng.random() < 0.3:
                    c["subsets"] = True
                    c["n_step"] = max(1, round(n_step / ly)) * ly
                elif c["l"] > 0 and rng.random() < 0.15:
                    c["whole"] = True
        if kind != "stream" and dim == 3 and rng.random() < 0.5:
            c["packed"] = True
        if _attempts(c) > DRAW_MOST or 2.0 * c["n"] * ly * lx * c["n_step"] >= 2 ** 31:
            continue
        return c


def _specs(case, seed):
    """Job descriptions of a case; the seed sets every random number."""
    key = 1000003 * (int(seed) + 1)
    if case["kind"] == "serve":
        stream = workloads.serving_stream(case["requests"], 200.0, seed=case["mix"], **workloads.SERVE_MIX)
        return [dataclasses.replace(s, seed=key + i) for i, (_, s) in enumerate(stream)]
    if case["kind"] == "uneven":
        return [dataclasses.replace(s, seed=key + i, n_step=max(1, round(s.n_step * case["scale"])))
                for i, s in enumerate(workloads.config4_jobs(case["n_traj"]))]
    fmt = ee.EE_SPINS_BITPACKED if case.get("packed") else ee.EE_SPINS_INT8
    return [ee.JobSpec(dim=case["dim"], lt=case["lt"], lx=case["lx"], ly=case["ly"], n=case["n"],
                       beta=B2 if case["dim"] == 2 else B3, l=case["l"] + i, n_step=case["n_step"],
                       n_traj=case["n_traj"], seed=key + i, spin_format=fmt, reverse=case.get("reverse", False),
                       subsets=case.get("subsets", False), whole=case.get("whole", False))
            for i in range(case.get("jobs", 1))]


def _attempts(case):
    return sum(s.n_traj * s.sites * (case["n_therm"] + s.n_step) for s in _specs(case, 0))


def prepare(case, seed):
    specs = _specs(case, seed)
    st = {"case": case, "n_therm": case["n_therm"]}
    if case["kind"] == "serve":
        st["specs"] = specs
        st["server"] = serve.Server(hbm_budget_bytes=workloads.SERVE_HBM_BUDGET, n_therm=case["n_therm"],
                                    launch=workloads.SERVE_LAUNCH, keep_work=True)
        return st
    st["jobs"] = [ee.Job(s) for s in specs]
    # the shape tuned for the set where the tuner's shipped cache has one,
    # else the library's own
    st["launch"] = autotune.cached(specs, case["n_therm"]) if case["kind"] != "job" else None
    return st


def run(state):
    n_therm = state["n_therm"]
    if "server" in state:
        reqs = [serve.Request(i, s, 0.0) for i, s in enumerate(state["specs"])]
        done = sorted(state["server"].run(reqs, realtime=False), key=lambda r: r.rid)
        return _outputs([r.result for r in done], [r.work for r in done])
    jobs = state["jobs"]
    for j in jobs:
        j.reset()
    if state["case"]["kind"] == "job":
        for j in jobs:
            j.thermalize(n_therm)
            j.run_protocol()
    else:
        ee.batch_run(jobs, n_therm, cfg=state["launch"])
    out = _outputs([j.estimate() for j in jobs], [j.work() for j in jobs])
    if state["case"].get("spins"):
        out["spins"] = jobs[0].spins()
    return out


FLOATS = ("dF", "dS", "dF_err", "w_mean", "w_var", "ess")


def _outputs(results, works):
    out = {k: np.array([getattr(r, k) for r in results]) for k in FLOATS}
    out["i_range"] = np.array([[r.i_min, r.i_max] for r in results])
    out["work"] = np.concatenate(works)
    return out


def work(case):
    """Bytes: the ramp tables read, the final spins and the works written;
    where a lattice does not fit a workgroup's LDS, every spin read and
    written once per sweep.  Operations: per attempt an eighth of a
    Philox4x32-10 call (80 integer operations), 2 dim neighbour terms, the
    threshold and the decision."""
    nbytes = flops = 0.0
    for s in _specs(case, 0):
        sweeps = case["n_therm"] + s.n_step
        sites = float(s.n_traj) * s.sites
        flops += sites * sweeps * (10 + 2 * s.dim + 2)
        spin_bytes = sites / (8 if s.spin_format == ee.EE_SPINS_BITPACKED else 1)
        nbytes += 32.0 * s.dim * (s.S + 1) + 8.0 * s.n_traj
        nbytes += spin_bytes if _padded(s.n, s.lt, s.ly, s.lx) <= ON_CHIP else 2.0 * sites * sweeps
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# The same estimate in plain numpy: checkerboard Metropolis on explicit
# neighbours, the Philox streams by their definition.
# ---------------------------------------------------------------------------
EXACT_MOST = 3e7  # attempts


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on uint64 arrays of 32-bit counter words."""
    m = np.uint64(0xFFFFFFFF)
    c = [np.asarray(v, dtype=np.uint64) for v in (c0, c1, c2, c3)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(np.broadcast_arrays(*c), axis=-1)


def _simulate(s, n_therm):
    """Spins (trajectory, replica, t, y, x) after the protocol, and the works."""
    J, n, lt, ly, lx, l, S, N = s.n_traj, s.n, s.lt, s.ly, s.lx, s.l, s.S, s.n_step
    H = lx // 2
    j, r, t, y, h = np.ogrid[0:J, 0:n, 0:lt, 0:ly, 0:H]
    rho = t * ly + y
    shape = (J, n, lt, ly, H)
    sites = [np.broadcast_to(2 * h + ((c + t + y) & 1), shape) for c in (0, 1)]

    def fields(phase, g, c):
        u = _philox(rho * -(-H // 8) + (h >> 3)[..., ::8], g, j, (phase << 28) | (r << 1) | c, s.seed)
        u = np.stack([u & np.uint64(0xFFFF), u >> np.uint64(16)], axis=-1)  # (..., group, word, half)
        return u.reshape(shape[:4] + (-1,))[..., :H].astype(np.int64)

    sp = np.zeros((J, n, lt, ly, lx), dtype=np.int64)
    for c in (0, 1):
        u = _philox(rho * -(-H // 4) + (h >> 2)[..., ::4], 0, j, (r << 1) | c, s.seed)
        u = u.reshape(shape[:4] + (-1,))[..., :H]
        np.put_along_axis(sp, sites[c], np.where(u < 2 ** 31, 1, -1), axis=4)

    yy, xx = np.ogrid[0:ly, 0:lx]
    ramped = np.broadcast_to((xx < l) if s.whole else (xx == l), (ly, lx))
    glued = np.zeros((ly, lx), bool) if s.whole else np.broadcast_to(xx < l, (ly, lx))

    def m_of(pos):
        return np.broadcast_to(np.clip(pos - yy * S, 0, S) if s.subsets else pos, (ly, lx))

    def threshold(K):
        K, inv = np.unique(K, return_inverse=True)
        U = np.empty(len(K), dtype=np.int64)
        for i, k in enumerate(K):
            U[i] = 2 ** 32 - 1 if s.beta * float(k) <= 0 else \
                max(math.floor(math.ldexp(math.exp(-(2.0 * s.beta * float(k)) / float(S)), 32)), 1) - 1
        return U, inv

    works = np.zeros(J, dtype=np.int64)
    pos0, d = (N, -1) if s.reverse else (0, 1)
    for g in range(n_therm + N):
        k = g - n_therm
        pos = pos0 + d * (k + 1) if k >= 0 else pos0
        mm = m_of(pos)
        if k >= 0:
            dm = (mm - m_of(pos - d)) * ramped
            bond = sp[:, :, 0] * (np.roll(sp, -1, axis=1)[:, :, 1] - sp[:, :, 1])
            works += (bond * dm).sum(axis=(1, 2, 3))
        inter = np.where(ramped, mm, np.where(glued, S, 0))
        for c in (0, 1):
            f = np.roll(sp, 1, 4) + np.roll(sp, -1, 4)
            if s.dim == 3:
                f = f + np.roll(sp, 1, 3) + np.roll(sp, -1, 3)
            up, down = np.roll(sp, -1, 2), np.roll(sp, 1, 2)
            up[:, :, 0] = 0
            down[:, :, 1] = 0
            f = S * (f + up + down)
            f[:, :, 0] += (S - inter) * sp[:, :, 1] + inter * np.roll(sp, -1, 1)[:, :, 1]
            f[:, :, 1] += (S - inter) * sp[:, :, 0] + inter * np.roll(sp, 1, 1)[:, :, 0]
            own = np.take_along_axis(sp, sites[c], 4)
            U, inv = threshold(own * np.take_along_axis(f, sites[c], 4))
            u = (fields(1, g, c) << 16) + fields(2, g, c)
            np.put_along_axis(sp, sites[c], np.where(u <= U[inv].reshape(shape), -own, own), axis=4)
    return sp, works


def exact(case, seed):
    if case["kind"] == "serve" or _attempts(case) > EXACT_MOST:
        return None
    out = {k: [] for k in FLOATS + ("i_range", "work")}
    for s in _specs(case, seed):
        sp, I = _simulate(s, case["n_therm"])
        e = np.exp(np.longdouble(s.beta) * (I - I.max()) / s.S)
        shift = np.longdouble(s.beta) * int(I.max()) / s.S
        dF = -(shift + np.log(e.sum() / len(I)))
        W = -np.longdouble(s.beta) * I / s.S
        err = np.nan
        if len(I) > 1:
            loo = -(shift + np.log((e.sum() - e) / (len(I) - 1)))
            err = np.sqrt((len(I) - 1) * ((loo - loo.mean()) ** 2).mean())
        for k, v in zip(FLOATS, (dF, dF / (s.n - 1), err, W.mean(), W.var(), e.sum() ** 2 / (e * e).sum())):
            out[k].append(float(v))
        out["i_range"].append([int(I.min()), int(I.max())])
        out["work"].append(I)
    res = {k: np.array(out[k]) for k in FLOATS + ("i_range",)}
    res["work"] = np.concatenate(out["work"])
    if case.get("spins"):
        res["spins"] = sp.reshape(len(I), -1).astype(np.int8)
    return res
