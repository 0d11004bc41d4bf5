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


@pytest.mark.parametrize("nx,ny,nz", [(512, 512, 16), (512, 512, 17), (192, 384, 63), (32, 512, 257)])
def test_gauss_deep_tiles(nx, ny, nz):
    """Volumes of 2^22 voxels and more: tiles of eight slices, slice counts
    that they divide and do not, both tile widths."""
    test_gauss_tile_edges(nx, ny, nz)


@pytest.mark.parametrize("scenes", [[(256, 256, 40), (128, 128, 101)], [(32, 512, 131), (192, 32, 5), (32, 512, 126)]],
                         ids=["wide", "narrow"])
def test_gauss_deep_tiles_in_a_batch(scenes):
    """A batch whose volumes of one tile width hold 2^22 voxels takes tiles of
    eight slices where each volume alone takes four: the same sums, so the
    prior agents' outputs are equal bit for bit."""
    import torch
    import paper_2406_13651_amd as G
    b = G.ClampBatchGPU([dict(nx=nx, ny=ny, nz=nz, looks=1, radius=8.0, sigma_w2=0.1, sigma2=1e-3)
                         for nx, ny, nz in scenes])
    gen = torch.Generator(device="cuda").manual_seed(5)
    ys = [torch.randn((1, nz, ny, nx), dtype=torch.complex64, device="cuda", generator=gen) for nx, ny, nz in scenes]
    b.init(ys)
    b.step()
    torch.cuda.synchronize()
    for i, (nx, ny, nz) in enumerate(scenes):
        g = G.ClampGPU(nx, ny, nz, 1, 8.0, 0.1, 1e-3, with_prior=True)
        g.init(ys[i])
        g.run(1)
        torch.cuda.synchronize()
        assert torch.equal(b.states[i]["r"][1], g.r[1])
        assert torch.equal(b.states[i]["w"], g.w)
