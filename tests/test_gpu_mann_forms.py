"""The fused update pass where its waves change how they share the looks, against
the float64 oracle: 64-point rows past one block per CU and 128-point rows
past four, whose blocks stay on one look at a time (the latter with three blocks
per CU), grids just below those lines, and 32-point rows with two waves a
group.  Bound: as for the small scenes, 1e-5 after three iterations."""

import pytest

from test_gpu_slices import test_small_scene_runs_match_oracle as _run

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, nz, looks, radius, with_prior, range_support
    (64, 64, 129, 1, 16.0, True, 0),    # 1032 groups
    (64, 64, 128, 1, 16.0, False, 0),   # 1024
    (128, 64, 257, 1, 16.0, True, 0),   # 4112
    (128, 64, 256, 1, 16.0, False, 0),  # 4096
    (32, 256, 31, 9, 8.0, True, 0),     # 496, two waves a group
]


@pytest.mark.parametrize("nx,ny,nz,looks,radius,with_prior,K", CASES, ids=["%dx%dx%d_L%d" % c[:4] for c in CASES])
def test_update_pass_forms_match_oracle(nx, ny, nz, looks, radius, with_prior, K):
    _run(nx, ny, nz, looks, radius, with_prior, K, True)
