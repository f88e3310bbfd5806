"""Tiled deposit and gather + push at the particle counts where their loads ahead change, with buckets of 0, 1, 255 to 257,
1023 to 1025 particles and the rest: the direct kernels' results, exactly where the arithmetic is the same (the push, the
fixed-point deposit)."""
import numpy as np
import pytest

import test_gpu_paged_step as paged
from test_gpu_paged_step import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 255, 256, 257, 0, 1023, 1024, 1025]
CASES = {
    "1d": dict(dim=1, vdim=1, cells=(256,), tile=(16, 0)),
    "2d": dict(dim=2, vdim=2, cells=(64, 64), tile=(16, 16)),
    "2d_hc": dict(dim=2, vdim=3, cells=(64, 64), tile=(16, 16), pusher="hc", c=4.0, bz=1.0),
    "3d": dict(dim=3, vdim=3, cells=(16, 16, 16), tile=(8, 8, 4)),
    "many": dict(dim=2, vdim=3, cells=(128, 128), tile=(4, 4), bz=1.0),
}


def state(rng, cfg, per_bucket):
    """Buckets of SIZES first, the others share what is left to an average of per_bucket."""
    cells, tile = np.array(cfg["cells"]), np.array([t or 1 for t in cfg["tile"]][:cfg["dim"]])
    nb = np.prod(cells // tile)
    rest = nb - len(SIZES)
    counts = np.concatenate([SIZES, np.full(rest, max(1, (per_bucket * nb - sum(SIZES)) // rest))]).astype(np.int64)
    bucket = rng.permutation(np.repeat(np.arange(nb), counts))
    pos = []
    for a in range(cfg["dim"]):
        ntile = cells[a] // tile[a]
        pos.append((bucket % ntile + rng.uniform(0.01, 0.99, len(bucket))) * tile[a])
        bucket = bucket // ntile
    # slow enough to stay in their cells' tiles or the next, as tiled calls meet them after a sort
    return pos, [0.3 * rng.normal(size=len(pos[0])) for _ in range(cfg["vdim"])]


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("per_bucket", [300, 513, 1030])
@pytest.mark.parametrize("name", list(CASES))
def test_tiled_calls_equal_direct_ones(torch, name, per_bucket, precision):  # noqa: F811
    cfg = CASES[name]
    pos, vel = state(np.random.default_rng(per_bucket), cfg, per_bucket)
    ctx = paged._context(cfg, len(pos[0]), precision)
    p, q = (paged._load(torch, ctx, cfg, pos, vel) for _ in range(2))
    start = p.download()["bucket_start"].astype(np.int64)
    assert list(np.diff(start)[:len(SIZES)]) == SIZES
    rho, ref = (torch.zeros(ctx.G, dtype=torch.int64 if ctx.mixed else torch.float64, device="cuda") for _ in range(2))
    ctx.deposit(p, rho)
    ctx.deposit(p, ref, tiled=False)
    ctx.sync()
    if ctx.mixed:
        assert torch.equal(rho, ref)
    else:
        # sums of up to 1e5 weights in another order: 1e5 roundings of 1e-16 at most
        assert float((rho - ref).abs().max()) <= 1e-11 * float(ref.abs().max())
    E = torch.randn(ctx.dim * ctx.G, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda",
                    dtype=torch.float64).to(torch.float32 if ctx.mixed else torch.float64)
    for scale, move in ((-0.5, False), (1.0, True)):
        ctx.gather_push(p, E, scale, move)
        ctx.gather_push(q, E, scale, move, tiled=False)
        ctx.sync()
        a, b = p.download(), q.download()
        for k in ("cell", "ox", "oy", "oz", "x", "y", "z", "vx", "vy", "vz"):
            if a[k] is not None:
                assert np.array_equal(a[k], b[k]), (k, move)


def test_a_tiled_move_costs_less_than_a_direct_one(torch):  # noqa: F811
    """16.8M mixed particles, gathered, pushed and moved bucket by bucket: less than 0.9 of the time of the direct kernel, which
    gathers from the whole field (0.99 with four particles loaded ahead in every build, 0.73 now)."""
    import time
    from paper_2608_15249_amd.apic import Context, Particles
    n = 1 << 24
    ctx = Context(dim=2, vdim=3, nx=512, ny=512, lx=512.0, ly=512.0, dt=0.05, n=n, precision="mixed")
    g = torch.Generator(device="cuda").manual_seed(1)
    x, y = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 512 for _ in range(2))
    v = torch.zeros(n, device="cuda", dtype=torch.float64)
    p = Particles(ctx)
    ctx.import_state(p, x, y, v, v, v)
    ctx.sort_by_cell(p)
    E = torch.zeros(2 * ctx.G, dtype=torch.float32, device="cuda")

    def best(tiled):
        out = []
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(10):
                ctx.gather_push(p, E, 0.0, True, tiled=tiled)
            torch.cuda.synchronize()
            out.append(time.perf_counter() - t)
        return min(out)

    tiled, direct = best(True), best(False)
    ctx.sync()
    assert tiled < 0.9 * direct, (tiled, direct)
