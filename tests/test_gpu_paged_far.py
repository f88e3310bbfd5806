"""Particles that cross more than a tile per step, in calls of several steps: their cost is their own number, as in calls of
one step (which reorder the particles), not their number times the buckets'."""
import time

import pytest

from test_gpu_paged_step import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_far_leavers_cost_no_more_than_in_single_steps(torch, precision):  # noqa: F811
    """One particle in ten jumps two and a half tiles per step: a call of 16 steps takes no longer than 16 calls of one
    (with one list of all far leavers, searched by every bucket, it took 1.8 times as long; with the buckets' own chains
    0.3 times)."""
    from paper_2608_15249_amd.apic import Context, Particles
    n, nx, steps = 4000037, 256, 16
    ctx = Context(dim=2, vdim=2, nx=nx, ny=nx, lx=float(nx), ly=float(nx), dt=0.1, n=n, precision=precision, tile=(8, 8))
    p = Particles(ctx)
    g = torch.Generator(device="cuda").manual_seed(1)
    u = lambda: torch.rand(n, generator=g, device="cuda", dtype=torch.float64)  # noqa: E731
    x, y, far = u() * nx, u() * nx, u() < 0.1
    v = torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    ctx.import_state(p, x, y, v + torch.where(far, 200.0, 0.0), v)
    ctx.sort_by_cell(p)
    E = torch.zeros(2 * ctx.G, dtype=torch.float64, device="cuda")
    E32 = torch.zeros(2 * ctx.G, dtype=torch.float32, device="cuda") if ctx.mixed else None
    rho = torch.zeros(ctx.G, dtype=torch.int64 if ctx.mixed else torch.float64, device="cuda")
    ctx.deposit(p, rho)
    ctx.field_solve(rho, E, E32)

    def best(per_call):
        times = []
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(0, steps, per_call):
                ctx.step(p, E, E32, per_call)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
        return min(times)

    single, paged = best(1), best(steps)
    ctx.sync()
    assert paged <= single, (paged, single)
