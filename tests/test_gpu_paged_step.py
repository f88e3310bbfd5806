"""Calls of several steps keep the particles in pages between the steps; calls
of one step reorder them. Both advance the same plasma: a call of nine steps
against nine calls of one. Mixed path bit for bit (fields, charge and field
energy, bucket table, the particles of every bucket as a set; the kinetic sums
to rounding), FP64 path to rounding amplified over the steps. The sizes are
those where the exchange can go wrong: partial tiles, tiles that are their own
neighbours, jumps beyond the neighbour tiles, buckets that empty and fill
(pages taken and given back, compaction beyond one bitmap), absorbing walls,
more buckets than one launch scans. (Buckets without a particle:
test_gpu_paged_empty.py.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

STEPS = 9


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2608_15249_amd import apic
    apic.load_library()
    return t


def _state(rng, dim, vdim, cells, n, speed, cluster):
    pos = []
    for a in range(dim):
        x = rng.uniform(0.0, cells[a], n)
        if cluster:   # most particles in one small blob that flies apart
            x[: n * 9 // 10] = np.mod(cells[a] * 0.4 + 1.5 * rng.normal(size=n * 9 // 10), cells[a])
        pos.append(x)
    return pos, [speed * rng.normal(size=n) for _ in range(vdim)]


def _context(cfg, n, precision):
    from paper_2608_15249_amd.apic import Context
    cells = cfg["cells"] + (1,) * (3 - cfg["dim"])
    return Context(dim=cfg["dim"], vdim=cfg["vdim"], nx=cells[0], ny=cells[1], nz=cells[2], lx=float(cells[0]),
                   ly=float(cells[1]), lz=float(cells[2]), dt=0.1, n=n, precision=precision, tile=cfg["tile"],
                   bz=cfg.get("bz", 0.0), pusher=cfg.get("pusher", "boris"), c_light=cfg.get("c", 0.0),
                   walls=cfg.get("walls", False), model="em" if cfg.get("em") else "es")


def _load(torch, ctx, cfg, pos, vel):
    from paper_2608_15249_amd.apic import Particles
    p = Particles(ctx)
    if ctx.mixed:
        from paper_2608_15249_amd import workloads as W
        both = [W.to_cell_offset(x, 1.0, m) for x, m in zip(pos, cfg["cells"])]
        cell = W.pack_cell(*([b[0] for b in both] + [None] * (2 - len(both)))[:2], both[2][0] if len(both) == 3 else None)
        p.upload(cell=cell, ox=both[0][1], oy=both[1][1] if len(both) > 1 else None,
                 oz=both[2][1] if len(both) > 2 else None, **dict(zip(("vx", "vy", "vz"), vel)))
    else:
        p.upload(**dict(zip(("x", "y", "z"), pos)), **dict(zip(("vx", "vy", "vz"), vel)))
    ctx.sort_by_cell(p)
    return p


def _run(torch, cfg, pos, vel, precision, per_call):
    n = len(pos[0])
    ctx = _context(cfg, n, precision)
    p = _load(torch, ctx, cfg, pos, vel)
    z = lambda m, t=torch.float64: torch.zeros(m, dtype=t, device="cuda")
    diag = z(4 * STEPS)
    if cfg.get("em"):
        F, J = z(6 * ctx.G), z(3 * ctx.G)
        ctx.em_init_fields(p, F)
        for k in range(0, STEPS, per_call):
            ctx.em_step(p, F, per_call, diag[4 * k:], J=J)
        fields = dict(F=F, J=J)
    else:
        rho = z(ctx.G, torch.int64 if ctx.mixed else torch.float64)
        E, E32 = z(ctx.dim * ctx.G), z(ctx.dim * ctx.G, torch.float32) if ctx.mixed else None
        ctx.deposit(p, rho)
        ctx.field_solve(rho, E, E32)
        for k in range(0, STEPS, per_call):
            ctx.step(p, E, E32, per_call, diag[4 * k:], rho=rho)
        fields = dict(E=E, rho=rho, **(dict(E32=E32) if ctx.mixed else {}))
    ctx.sync()
    out = {k: v.cpu().numpy() for k, v in fields.items()}
    return out, diag.cpu().numpy().reshape(STEPS, 4), p.download()


def _ordered(state):
    """Particle arrays with every bucket's particles in an order of their own."""
    b = state["bucket_start"].astype(np.int64)
    live = int(b[-1])
    keys = [k for k in ("cell", "x", "ox", "y", "oy", "z", "oz", "vx", "vy", "vz") if state[k] is not None]
    bucket = np.repeat(np.arange(len(b) - 1), np.diff(b))
    order = np.lexsort([state[k][:live] for k in reversed(keys)] + [bucket])
    return {k: state[k][:live][order] for k in keys}


CASES = {
    "1d": dict(dim=1, vdim=1, cells=(61,), tile=(8, 0), n=20011),
    "2d_ragged": dict(dim=2, vdim=2, cells=(75, 52), tile=(16, 8), n=60013),
    "2d_one_tile_wide": dict(dim=2, vdim=3, cells=(16, 40), tile=(16, 16), n=20001, bz=1.5),
    "2d_two_tiles": dict(dim=2, vdim=2, cells=(32, 32), tile=(16, 16), n=16385),
    "2d_far": dict(dim=2, vdim=2, cells=(64, 64), tile=(4, 4), n=200003, speed=60.0),
    "2d_cluster": dict(dim=2, vdim=2, cells=(64, 64), tile=(16, 16), n=90001, speed=30.0, cluster=True),
    "2d_hc": dict(dim=2, vdim=3, cells=(64, 32), tile=(8, 8), n=40007, pusher="hc", c=4.0, bz=1.0),
    "2d_walls": dict(dim=2, vdim=2, cells=(48, 40), tile=(16, 8), n=40009, walls=True, speed=3.0),
    "3d": dict(dim=3, vdim=3, cells=(20, 12, 18), tile=(8, 4, 8), n=50021),
    "3d_far_hc": dict(dim=3, vdim=3, cells=(16, 16, 16), tile=(4, 4, 4), n=60017, speed=60.0, pusher="hc", c=200.0),
    "many_buckets": dict(dim=2, vdim=2, cells=(256, 136), tile=(2, 4), n=2300017, speed=2.0),
    "em": dict(dim=2, vdim=3, cells=(75, 52), tile=(16, 8), n=60013, em=True, c=5.0, bz=1.0),
    "em_hc": dict(dim=2, vdim=3, cells=(64, 64), tile=(16, 16), n=50001, em=True, c=5.0, pusher="hc", bz=1.0),
}


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("name", list(CASES))
def test_call_of_steps_matches_single_steps(torch, name, precision):
    cfg = CASES[name]
    rng = np.random.default_rng(31)
    pos, vel = _state(rng, cfg["dim"], cfg["vdim"], cfg["cells"], cfg["n"], cfg.get("speed", 1.0),
                      cfg.get("cluster", False))
    one, done, pone = _run(torch, cfg, pos, vel, precision, 1)
    many, dmany, pmany = _run(torch, cfg, pos, vel, precision, STEPS)
    assert np.array_equal(pone["bucket_start"], pmany["bucket_start"])
    a, b = _ordered(pone), _ordered(pmany)
    em = cfg.get("em")
    if precision == "mixed" and not em:
        for k in one:
            assert np.array_equal(one[k], many[k]), k
        for k in a:
            assert np.array_equal(a[k], b[k]), k
        assert np.array_equal(done[:, :2], dmany[:, :2])
    else:
        # FP64 sums (the charge, or the current of the electromagnetic step) round by their order:
        # 1e-16 of the sums, amplified over nine steps of a noisy plasma by less than 1e4; a
        # binary32 state may also round the other way
        tol = 1e-5 if precision == "mixed" else 1e-11
        for k in one:
            assert np.max(np.abs(one[k] - many[k])) <= tol * np.max(np.abs(one[k])), k
        for k in a:
            if precision == "mixed":
                assert np.array_equal(np.sort(a["cell"]), np.sort(b["cell"]))
            else:
                assert np.max(np.abs(a[k] - b[k])) <= tol * max(1.0, np.max(np.abs(a[k]))), k
    assert np.allclose(done[:, 2], dmany[:, 2], rtol=1e-6 if em and precision == "mixed" else 1e-12, atol=0.0)


def test_same_call_twice_same_bits(torch):
    cfg = CASES["2d_cluster"]
    rng = np.random.default_rng(5)
    pos, vel = _state(rng, 2, 2, cfg["cells"], cfg["n"], 3.0, True)
    a, da, pa = _run(torch, cfg, pos, vel, "mixed", STEPS)
    b, db, pb = _run(torch, cfg, pos, vel, "mixed", STEPS)
    assert np.array_equal(da, db)
    for k in ("cell", "ox", "oy", "vx", "vy", "bucket_start"):
        assert np.array_equal(pa[k], pb[k]), k
