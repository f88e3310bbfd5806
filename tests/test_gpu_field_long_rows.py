"""2D field solves with rows of 1024 points: many rows go through the library's transforms (the same bits as with
APIC_FIELD_FFT=library), few through the lines in LDS; both match the oracle."""
import numpy as np
import pytest

from test_gpu_field_dft import _ctx, _solve, test_lines_of_any_length as check
from test_gpu_field_dft import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("ny,library", [(748, False), (750, True), (960, True), (1023, True)])
def test_route_of_long_rows(torch, ny, library, walls):  # noqa: F811
    nx = 512 if walls else 1024   # between walls the rows are the odd extension
    rho = np.random.default_rng(ny).normal(size=(ny, 1024))
    E, _, we = _solve(torch, _ctx(nx, ny, "fp64", walls=walls), rho)
    L, _, wl = _solve(torch, _ctx(nx, ny, "fp64", walls=walls, library=True), rho)
    assert np.array_equal(E, L) == library
    assert np.max(np.abs(E - L)) <= 1e-12 * np.max(np.abs(L)) and abs(we / wl - 1) <= 1e-12


def test_long_rows_match_the_oracle(torch):  # noqa: F811
    check(torch, 1024, 960)
