"""Chunk sizes of apic_sort_by_cell: the particle counts at which a workgroup's chunk changes and those around its ends, for
few and for many buckets, exactly against numpy's stable argsort; and a short sort costs less than a long one."""
import time

import pytest

from test_gpu_sort import test_sort_is_stable_by_bucket as check
from test_gpu_sort import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

SMALL, MEDIUM = 1 << 19, 1 << 23   # from these counts on a thread takes twice as many particles
FEW, MANY = ((64, 48), (4, 4)), ((1024, 1024), (4, 4))   # 192 and 65536 buckets: digits of 4 and of 8 bits
CASES = [(2, *b, n, False) for b in (FEW, MANY) for n in (511, 512, 513, 1024, 1025, SMALL - 1, SMALL, SMALL + 1)]
CASES += [(2, *b, n, False) for b in (FEW, MANY) for n in (MEDIUM - 1, MEDIUM)]
CASES += [(1, (61,), (8, 0), SMALL + 1023, False), (3, (16, 16, 16), (4, 4, 4), SMALL + 7, False)]


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dd_%d_in_%s" % (c[0], c[3], "x".join(map(str, c[1]))))
def test_sort_at_the_chunk_changes(torch, case, precision):  # noqa: F811
    check(torch, case, precision, case[3] % 2 == 1)


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_short_sorts_cost_less(torch, precision):  # noqa: F811
    """Ten thousand particles take less than 0.7 times the time of a million (0.9 times with one chunk size for all: three
    workgroups that rank sixteen particles per thread one after the other)."""
    from paper_2608_15249_amd.apic import Context, Particles

    def best(n):
        c = Context(dim=2, vdim=3, nx=512, ny=512, lx=512.0, ly=512.0, dt=0.1, n=n, precision=precision, tile=(32, 32))
        g = torch.Generator(device="cuda").manual_seed(1)
        x, y = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 512 for _ in range(2))
        v = torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
        p = Particles(c)
        c.import_state(p, x, y, v, v, v)
        c.sort_by_cell(p)
        graph, stream, out = torch.cuda.CUDAGraph(), torch.cuda.Stream(), []
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            c.sort_by_cell(p)
            with torch.cuda.graph(graph, stream=stream):
                for _ in range(10):
                    c.sort_by_cell(p)
        torch.cuda.synchronize()
        for _ in range(5):
            t = time.perf_counter()
            graph.replay()
            torch.cuda.synchronize()
            out.append(time.perf_counter() - t)
        c.sync()
        return min(out)

    short, long_ = best(10007), best(1000003)
    assert short < 0.7 * long_, (short, long_)
