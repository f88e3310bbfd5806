"""The 2D field solve on sides that are not powers of two (three launches, a line
transformed in one pass per factor, each output the sum of its terms): against
the oracle's solve of the same charge and the library-transform path on the same
input. Prime sides, sides of two nodes, odd numbers of rows, lines longer than a
workgroup, one side a power of two, the odd extension between walls, and the
fixed-point accumulation with its exact charge."""
import os

import numpy as np
import pytest

import oracle as O
from oracle import bounded as B

pytestmark = pytest.mark.gpu

SHAPES = [(2, 3), (3, 2), (61, 67), (300, 182), (64, 45), (45, 64), (77, 1001), (1000, 33), (720, 960), (127, 131)]

# the sums of a line have at most the sum of its factors in terms, below 400 here: four
# transforms of such sums round by less than 4 * 400 * 2^-53 = 2e-13 of the largest value
TOL = 1e-12


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    from paper_2608_15249_amd import apic
    apic.load_library()
    return t


def _ctx(nx, ny, precision, walls=False, library=False):
    from paper_2608_15249_amd.apic import Context
    old = os.environ.pop("APIC_FIELD_FFT", None)
    if library:
        os.environ["APIC_FIELD_FFT"] = "library"
    try:
        return Context(dim=2, vdim=2, nx=nx, ny=ny, lx=nx * 0.83, ly=ny * 1.21, dt=0.1, n=1024, precision=precision,
                       tile=(2, 2), walls=walls)
    finally:
        os.environ.pop("APIC_FIELD_FFT", None)
        if old is not None:
            os.environ["APIC_FIELD_FFT"] = old


def _solve(torch, c, rho):
    E = torch.zeros(2 * c.G, dtype=torch.float64, device="cuda")
    E32 = torch.zeros(2 * c.G, dtype=torch.float32, device="cuda") if c.mixed else None
    we = torch.zeros(1, dtype=torch.float64, device="cuda")
    dev = torch.from_numpy(rho.ravel().copy()).cuda()
    c.field_solve(dev, E, E32, we)
    c.sync()
    assert np.array_equal(dev.cpu().numpy(), rho.ravel())
    return E.cpu().numpy(), E32.cpu().numpy() if c.mixed else None, float(we.item())


@pytest.mark.parametrize("nx,ny", SHAPES)
def test_lines_of_any_length(torch, nx, ny):
    rng = np.random.default_rng(4000 + nx + 7 * ny)
    rho = rng.normal(size=(ny, nx)) + 0.3
    s = O.Setup(2, 2, nx, nx * 0.83, 1024, 0.1, ny=ny, Ly=ny * 1.21)
    Eo = np.stack(O.solve_field(s, rho))
    scale = np.max(np.abs(Eo))
    E, _, we = _solve(torch, _ctx(nx, ny, "fp64"), rho)
    El, _, wel = _solve(torch, _ctx(nx, ny, "fp64", library=True), rho)
    assert np.max(np.abs(E.reshape(2, ny, nx) - Eo)) <= TOL * scale
    assert np.max(np.abs(E - El)) <= TOL * scale
    assert abs(we / wel - 1) <= TOL


@pytest.mark.parametrize("nx,ny", [(3, 5), (96, 61), (300, 182)])
def test_fixed_point_sums(torch, nx, ny):
    rng = np.random.default_rng(5000 + nx)
    c, cl = _ctx(nx, ny, "mixed"), _ctx(nx, ny, "mixed", library=True)
    S = c.frac_bits
    I = rng.integers(0, 40 << (2 * S), size=(ny, nx), dtype=np.int64)
    s = O.Setup(2, 2, nx, nx * 0.83, 1024, 0.1, ny=ny, Ly=ny * 1.21)
    Eo = np.stack(O.solve_field(s, O.rho_from_quantised(s, I, S)))
    E, E32, we = _solve(torch, c, I)
    _, _, wel = _solve(torch, cl, I)
    assert np.max(np.abs(E.reshape(2, ny, nx) - Eo)) <= TOL * np.max(np.abs(Eo))
    assert np.array_equal(E32, E.astype(np.float32))
    assert c.charge_exact() == cl.charge_exact()
    assert abs(we / wel - 1) <= TOL


@pytest.mark.parametrize("nx,ny", [(3, 4), (45, 32), (150, 91)])
def test_odd_extension(torch, nx, ny):
    rng = np.random.default_rng(6000 + nx)
    b = B.Box(nx, nx * 0.83, ny, ny * 1.21, 1024, 0.1)
    rho = rng.normal(size=(ny, nx + 1))
    ext = np.zeros((ny, 2 * nx))
    ext[:, :nx + 1] = rho
    E, _, we = _solve(torch, _ctx(nx, ny, "fp64", walls=True), ext)
    El, _, wel = _solve(torch, _ctx(nx, ny, "fp64", walls=True, library=True), ext)
    Eo = B.solve_field(b, rho)
    Eg = E.reshape(2, ny, 2 * nx)[:, :, :nx + 1]
    scale = max(np.max(np.abs(e)) for e in Eo)
    for d in range(2):
        assert np.max(np.abs(Eg[d] - Eo[d])) <= TOL * scale
    assert np.max(np.abs(E - El)) <= TOL * scale
    assert abs(we / wel - 1) <= TOL
