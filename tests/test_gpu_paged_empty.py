"""Calls of several steps on plasmas that leave buckets empty: a slab in a
vacuum, slabs that leave their tiles and fill others, a slab that a wall takes,
in every dimension, precision and model. Nine steps in one call (particles in
pages) against nine calls of one step, as in test_gpu_paged_step.py. Each case
checks that it ends with empty buckets whose place in the arrays lies inside a
line, where the copy back once read beyond the bucket's pages."""
import numpy as np
import pytest

import test_gpu_paged_step as paged
from test_gpu_paged_step import STEPS, torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

# slabs: (first cell, last cell, drift along x in cells per unit time); a step is 0.1, a call 0.9, and the gaps are wider than
# what drift, spread and the slabs' own fields (the excess over the ions' density times half the width) close in a call
CASES = {
    "1d_vacuum": dict(dim=1, vdim=1, cells=(256,), tile=(16, 0), n=10007, slabs=[(36, 60, 0.0)]),
    "1d_drift": dict(dim=1, vdim=1, cells=(256,), tile=(16, 0), n=10007, slabs=[(32, 48, 120.0), (200, 204, 0.0)]),
    "2d_vacuum": dict(dim=2, vdim=2, cells=(256, 32), tile=(16, 16), n=20011, slabs=[(80, 144, 0.0)]),
    "2d_drift": dict(dim=2, vdim=3, cells=(256, 32), tile=(16, 16), n=20011, bz=0.1, slabs=[(16, 48, 120.0), (176, 192, -90.0)]),
    "2d_walls": dict(dim=2, vdim=2, cells=(128, 32), tile=(16, 16), n=20011, walls=True, slabs=[(4, 12, -60.0), (70, 74, 0.0)]),
    "2d_all_taken": dict(dim=2, vdim=2, cells=(64, 32), tile=(16, 16), n=20011, walls=True, slabs=[(4, 12, -60.0)], none=True),
    "3d_vacuum": dict(dim=3, vdim=3, cells=(128, 8, 16), tile=(8, 4, 8), n=40009, slabs=[(60, 76, 0.0)]),
    # (a particle of the electromagnetic step moves less than a cell: narrow gaps, small fields)
    "em_vacuum": dict(dim=2, vdim=3, cells=(32, 32), tile=(4, 8), n=20011, em=True, c=5.0, bz=0.1, thermal=0.1,
                      slabs=[(8, 26, 0.0)]),
    "many_buckets": dict(dim=2, vdim=2, cells=(256, 136), tile=(2, 4), n=2300017, slabs=[(3, 120, 5.0)]),
}


def state(rng, cfg):
    n, dim = cfg["n"], cfg["dim"]
    pos = [rng.uniform(0.0, m, n) for m in cfg["cells"]]
    vel = [cfg.get("thermal", 0.5) * rng.normal(size=n) for _ in range(cfg["vdim"])]
    part = np.array_split(np.arange(n), len(cfg["slabs"]))
    for ids, (lo, hi, drift) in zip(part, cfg["slabs"]):
        pos[0][ids] = rng.uniform(lo, hi, len(ids))
        vel[0][ids] += drift
    return pos, vel


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("name", list(CASES))
def test_empty_buckets(torch, name, precision):  # noqa: F811
    cfg = CASES[name]
    pos, vel = state(np.random.default_rng(17), cfg)
    one, done, pone = paged._run(torch, cfg, pos, vel, precision, 1)
    many, dmany, pmany = paged._run(torch, cfg, pos, vel, precision, STEPS)
    start = pmany["bucket_start"].astype(np.int64)
    assert np.array_equal(pone["bucket_start"], pmany["bucket_start"])
    empty = start[:-1][np.diff(start) == 0]
    assert len(empty) > 0
    if cfg.get("none"):
        assert start[-1] == 0
    else:
        assert np.any(empty % (32 if precision == "mixed" else 16) != 0)
    a, b = paged._ordered(pone), paged._ordered(pmany)
    em = cfg.get("em")
    # tolerances as in test_gpu_paged_step.py: the mixed electrostatic path bit for bit, sums of
    # binary64 to their rounding amplified over nine steps
    if precision == "mixed" and not em:
        for k in one:
            assert np.array_equal(one[k], many[k]), k
        for k in a:
            assert np.array_equal(a[k], b[k]), k
        assert np.array_equal(done[:, :2], dmany[:, :2])
    else:
        tol = 1e-5 if precision == "mixed" else 1e-11
        for k in one:
            assert np.max(np.abs(one[k] - many[k])) <= tol * np.max(np.abs(one[k])), k
        for k in a:
            if precision == "mixed":
                assert np.array_equal(np.sort(a["cell"]), np.sort(b["cell"]))
            elif len(a[k]):
                assert np.max(np.abs(a[k] - b[k])) <= tol * max(1.0, np.max(np.abs(a[k]))), k
    assert np.allclose(done[:, 2], dmany[:, 2], rtol=1e-6 if em and precision == "mixed" else 1e-12, atol=0.0)
