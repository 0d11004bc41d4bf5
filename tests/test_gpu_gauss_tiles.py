"""The single-pass Gaussian prior against the oracle at the edges of its tiles:
one slice, fewer slices than taps, slice counts that a tile's slices do not
divide, the narrow and the wide tile, one tile in x and y and several.

Bound: three chains of seven float32 products and sums with weights that add
up to one, each rounding at most 2^-24 of the largest partial sum: below 21
roundings, 1.3e-6 in the worst case and 1e-6 in norm."""

import numpy as np
import pytest

import oracle
from helpers import rel_l2, report

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(32, 32, 1), (32, 64, 2), (64, 32, 3), (64, 64, 4), (192, 32, 5), (96 * 2, 64, 9),
                                      (128, 192, 37), (32, 512, 8)])
def test_gauss_tile_edges(nx, ny, nz):
    import torch
    import paper_2406_13651_amd._clamp as C
    import paper_2406_13651_amd as G
    g = G.ClampGPU(nx, ny, nz, 1, 8.0, 0.01, 1e-3, with_prior=True)
    x = np.random.default_rng(nx + ny + nz).uniform(0.0, 1.0, (nz, ny, nx)).astype(np.float32)
    xt = torch.from_numpy(x).cuda()
    out = torch.full_like(xt, float("nan"))
    C.clamp_prior_gauss(g.plan, 0, 1.0, xt, out, g.ws)
    torch.cuda.synchronize()
    ref = oracle.gaussian_smooth(x.astype(np.float64), 1.0)
    assert report("gauss %dx%dx%d" % (nx, ny, nz), rel_l2(out.cpu().numpy(), ref), 1e-6) <= 1e-6
