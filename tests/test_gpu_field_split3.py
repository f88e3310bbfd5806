"""The 3D field solve on elongated grids, whose workgroups take from 4 to 16 lines each: against the oracle and the library's
transforms, as in test_gpu_field_fft3.py."""
import pytest

from test_gpu_field_fft3 import test_fused_solve_3d_fixed_point_accumulation as check_mixed
from test_gpu_field_fft3 import test_fused_solve_3d_fp64_matches_oracle_and_library as check_fp64
from test_gpu_field_fft3 import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

SHAPES = [(256, 64, 32), (64, 256, 32), (32, 64, 256), (128, 64, 16), (16, 32, 64), (4, 256, 256), (256, 4, 8)]


@pytest.mark.parametrize("nx,ny,nz", SHAPES)
def test_elongated_grids(torch, nx, ny, nz):  # noqa: F811
    check_fp64(torch, nx, ny, nz)
    check_mixed(torch, nx, ny, nz)
