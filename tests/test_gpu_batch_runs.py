"""A work item of the batched replicas is read in runs of four particles, what
is left one by one, and a particle may cross its grid several times in a step.
Items of every remainder, shorter than one run and longer than one round of the
workgroup, against the same plasma advanced alone: the same bits."""
import numpy as np
import pytest

from paper_2608_15249_amd import workloads as W

pytestmark = pytest.mark.gpu

STEPS = 3
COUNTS = (1, 2, 3, 4, 5, 255, 1023, 1024, 4096, 4099, 8193, 16387)


@pytest.mark.parametrize("speed", [1.0, 700.0])
def test_items_of_every_length(speed):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2608_15249_amd.sim import BatchSimulation, Simulation
    rng = np.random.default_rng(17)
    reps = [W.Replica(int(rng.integers(2, 90)), n, 0.02, 700 + i) for i, n in enumerate(COUNTS)]
    ws = [W.replica_workload(r) for r in reps]
    states = [(rng.uniform(0.0, w.Lx, w.n_particles), speed * rng.normal(size=w.n_particles)) for w in ws]
    bs = BatchSimulation(reps, states=states)
    bs.initialise()
    dg = bs.run(STEPS).cpu().numpy().reshape(STEPS, len(reps), 4)
    bs.batch.sync()
    for r, (w, (x, v)) in enumerate(zip(ws, states)):
        sim = Simulation(w, "mixed", state=(x, None, v, None, None), tile=(16, 0))
        sim.initialise()
        d1 = sim.run(STEPS).cpu().numpy().reshape(STEPS, 4)
        sim.ctx.sync()
        assert np.array_equal(bs.replica_field(r), sim.field()[0]), COUNTS[r]
        st = sim.state()
        a, b = bs.replica_state(r), (st["cell"], st["ox"], st["vx"])
        for p, q in zip([k[np.lexsort(a)] for k in a], [k[np.lexsort(b)] for k in b]):
            assert np.array_equal(p, q), COUNTS[r]
        assert np.array_equal(dg[:, r, :2], d1[:, :2]), COUNTS[r]
        # sums of n terms of one order of magnitude in two orders: n 2^-53 of the sum of their sizes
        assert np.allclose(dg[:, r, 2], d1[:, 2], rtol=1e-11, atol=0.0), COUNTS[r]
