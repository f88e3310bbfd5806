"""apic_workspace_limit: the pages of long calls can be declined. A context without them needs the workspace of the
reordering step, stays inside it, and a long call equals single steps particle by particle; one that cannot allocate the
larger workspace runs without pages."""
import ctypes

import numpy as np
import pytest

import test_gpu_paged_step as paged
from test_gpu_paged_step import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

CFG = {"es": paged.CASES["2d_ragged"], "em": paged.CASES["em"], "3d": paged.CASES["3d"]}


def size(ctx):
    out = ctypes.c_size_t()
    ctx._check(ctx.L.apic_workspace_size(ctx.h, ctypes.byref(out)))
    return out.value


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("name", list(CFG))
def test_size_and_the_way_back(torch, name, precision):  # noqa: F811
    cfg = CFG[name]
    ctx = paged._context(cfg, cfg["n"], precision)
    full = size(ctx)
    state = (4 * (1 + cfg["dim"] + cfg["vdim"]) if precision == "mixed" else 8 * (cfg["dim"] + cfg["vdim"])) * cfg["n"]
    for limit, want_less in ((0, True), (2**64 - 1, False), (full - 1, True), (full, False)):
        ctx._check(ctx.L.apic_workspace_limit(ctx.h, limit))
        assert (size(ctx) < full) if want_less else (size(ctx) == full)
    ctx._check(ctx.L.apic_workspace_limit(ctx.h, 0))
    less = size(ctx)
    # the pages take what the header says: four times the state and 29 bytes per particle, where the step takes the
    # state and 5 (grids, tables and the pool's partly filled pages aside)
    assert 3 * state + 20 * cfg["n"] < full - less < 4 * state + 29 * cfg["n"] + 2 * (ctx.nbuckets * 128 * state // cfg["n"] + 4096 * 256)


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("how", ["declined", "no memory"])
def test_long_call_without_pages(torch, monkeypatch, how, precision):  # noqa: F811
    cfg = CFG["es"]
    pos, vel = paged._state(np.random.default_rng(3), 2, 2, cfg["cells"], cfg["n"], 1.0, False)
    one = paged._run(torch, cfg, pos, vel, precision, 1)
    made = paged._context
    kept = []

    def lean(c, n, prec):
        if how == "declined":
            ctx = made(c, n, prec)
            ctx._check(ctx.L.apic_workspace_limit(ctx.h, 0))
            # what lies behind the smaller workspace stays as it is
            ctx.ws = torch.full((size(ctx) + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        else:
            empty, asked = torch.empty, []

            def scarce(*a, **k):
                if k.get("dtype") is torch.uint8:
                    asked.append(a[0])
                    if len(asked) == 1:
                        raise torch.cuda.OutOfMemoryError("no memory for the larger workspace")
                return empty(*a, **k)
            monkeypatch.setattr(torch, "empty", scarce)
            ctx = made(c, n, prec)
            monkeypatch.setattr(torch, "empty", empty)
            assert len(asked) == 2 and asked[1] == size(ctx) < asked[0]
        kept.append(ctx)
        return ctx

    monkeypatch.setattr(paged, "_context", lean)
    many = paged._run(torch, cfg, pos, vel, precision, paged.STEPS)
    if how == "declined":
        assert torch.all(kept[0].ws[-4096:] == 0x5A)
    for a, b in ((one[0], many[0]), (one[2], many[2])):
        for k in a:
            if a[k] is None:
                continue
            if precision == "mixed":
                assert np.array_equal(a[k], b[k]), k     # reordered both times: the same slots too
            else:
                # sums of binary64 round by their order: 1e-16 amplified over nine steps by less than 1e4; the slots are
                # the same as long as no particle's tile differs by it
                assert np.max(np.abs(a[k] - b[k])) <= 1e-11 * max(1.0, np.max(np.abs(a[k]))), k


def test_a_gradient_run_keeps_no_room_for_pages(torch):  # noqa: F811
    """FieldEnergyRun steps in the adjoint workspace: its context asks for the least."""
    from paper_2608_15249_amd.adjoint import FieldEnergyRun
    kw = dict(dim=2, vdim=2, nx=32, ny=32, lx=32.0, ly=32.0, dt=0.1, n=20011, tile=(16, 16))
    run = FieldEnergyRun(nsteps=4, stride=2, **kw)
    full = paged._context(dict(dim=2, vdim=2, cells=(32, 32), tile=(16, 16)), 20011, "mixed")
    assert run.ctx.ws.numel() < full.ws.numel()
    full._check(full.L.apic_workspace_limit(full.h, 0))
    assert run.ctx.ws.numel() == size(full)
