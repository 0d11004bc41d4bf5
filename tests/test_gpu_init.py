"""Initialisation against the float64 oracle at the edges of its launches:
look counts that the eight looks in flight do not divide, a voxel count whose
partial sums of the mean are added by a launch of their own, the 3D operator,
and the observation's norm added beside the average over the looks.

Bounds: mu carries the rounding of the two transforms (2 to 3 radix stages of
each, below 1e-6 of its norm), r their squares (twice that) and the float32
sum over the looks; 5e-6 covers both.  The norm is a sum in float64 of
float32 squares: 1e-6."""

import numpy as np
import pytest

import oracle
from helpers import rel_l2, report

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,looks,radius,with_prior,K", [
    (32, 32, 1, 1, 8.0, True, 0),
    (32, 64, 5, 9, 8.0, False, 0),
    (64, 32, 16, 17, 11.3, True, 9),
    (128, 64, 3, 7, 16.0, True, 0),
    (256, 256, 9, 2, 64.0, True, 0),   # 2304 partials of the mean
], ids=lambda v: str(v))
def test_init_edges(nx, ny, nz, looks, radius, with_prior, K):
    import torch
    import paper_2406_13651_amd as G
    rng = np.random.default_rng(3)
    shape = (looks, nz, ny, nx)
    y = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    mask = oracle.cylinder_mask(nz, ny, nx, radius, K) if K > 0 else oracle.pupil_mask(ny, nx, radius)
    g = G.ClampGPU(nx, ny, nz, looks, radius, 0.01, 1e-3, with_prior=with_prior, range_support=K)
    yt = torch.from_numpy(y).cuda()
    for _ in range(2):
        g.init(yt)
    torch.cuda.synchronize()
    st = oracle.clamp_init(y, mask, with_prior, 1.0)
    tag = "init %dx%dx%d L=%d K=%d" % (nx, ny, nz, looks, K)
    assert report(tag + " mu", rel_l2(g.mu.cpu().numpy(), st.mu), 5e-6) <= 5e-6
    assert report(tag + " r", rel_l2(g.r.cpu().numpy(), st.r), 5e-6) <= 5e-6
    assert report(tag + " w", rel_l2(g.w.cpu().numpy(), st.w), 5e-6) <= 5e-6
    assert report(tag + " |y|^2", rel_l2(g.ahy2.cpu().numpy(), st.ahy2), 1e-6) <= 1e-6
