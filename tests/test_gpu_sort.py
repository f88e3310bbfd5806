"""apic_sort_by_cell against numpy's stable argsort of the buckets: particle
arrays, permutation and bucket table exactly, at particle counts around the
chunk of the sort's workgroups, with one bucket, with bucket counts whose digits
are uneven, above the limit of two passes, clustered input, and without perm."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2608_15249_amd import apic
    apic.load_library()
    return t


CASES = [
    # dim, cells, tile, n, clustered
    (1, (61,), (8, 0), 1, False),
    (1, (4096,), (1, 0), 12289, False),
    (2, (64, 48), (64, 64), 5000, False),
    (2, (37, 29), (8, 8), 4095, False),
    (2, (64, 64), (4, 4), 4096, False),
    (2, (64, 64), (4, 4), 4097, True),
    (2, (300, 182), (16, 8), 50001, False),
    (2, (1024, 640), (2, 2), 300007, False),     # 163840 buckets: four passes
    (3, (20, 12, 18), (8, 4, 8), 30011, False),
    (3, (16, 16, 16), (2, 2, 2), 20000, True),
]


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dd_%d" % (c[0], c[3]))
@pytest.mark.parametrize("with_perm", [True, False])
def test_sort_is_stable_by_bucket(torch, case, precision, with_perm):
    from paper_2608_15249_amd import workloads as W
    from paper_2608_15249_amd.apic import Context, Particles
    dim, cells, tile, n, clustered = case
    vdim = {1: 1, 2: 2, 3: 3}[dim]
    rng = np.random.default_rng(n)
    c3 = cells + (1,) * (3 - dim)
    c = Context(dim=dim, vdim=vdim, nx=c3[0], ny=c3[1], nz=c3[2], lx=float(c3[0]), ly=float(c3[1]), lz=float(c3[2]),
                dt=0.1, n=n, precision=precision, tile=tile)
    pos = [np.mod(m * 0.5 + rng.normal(size=n), m) if clustered else rng.uniform(0.0, m, n) for m in cells]
    vel = [rng.normal(size=n) for _ in range(vdim)]
    p = Particles(c)
    if c.mixed:
        both = [W.to_cell_offset(x, 1.0, m) for x, m in zip(pos, cells)]
        idx = [b[0].astype(np.int64) for b in both]
        cell = W.pack_cell(both[0][0], both[1][0] if dim > 1 else None, both[2][0] if dim == 3 else None)
        src = dict(cell=cell, **{k: b[1] for k, b in zip(("ox", "oy", "oz"), both)})
    else:
        idx = [np.floor(x).astype(np.int64) % m for x, m in zip(pos, cells)]
        src = dict(zip(("x", "y", "z"), pos))
    src.update(zip(("vx", "vy", "vz"), vel))
    p.upload(**src)
    bucket, scale = np.zeros(n, dtype=np.int64), 1
    for a in range(dim):
        bucket += (idx[a] // c.tile[a]) * scale
        scale *= -(-cells[a] // c.tile[a])
    assert scale == c.nbuckets
    order = np.argsort(bucket, kind="stable")
    perm = torch.full((n,), -1, dtype=torch.int32, device="cuda") if with_perm else None
    before = p.download()
    c.sort_by_cell(p, perm=perm)
    c.sync()
    after = p.download()
    for k in src:
        assert np.array_equal(after[k], before[k][order]), k
    if with_perm:
        assert np.array_equal(perm.cpu().numpy(), order)
    assert np.array_equal(after["bucket_start"], np.searchsorted(bucket[order], np.arange(c.nbuckets + 1)))
