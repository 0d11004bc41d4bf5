"""The fused TV step at the edges of its tiling, against the float64 oracle:
one and several tiles per row (32- and 64-voxel tiles), one plane, depths the
plane walk does not divide, one and several steps (either buffer last), and
an image that starts at an odd float of its buffer.

Bound: a step rounds each dual component a few times (about 4 x 6e-8, |p| <=
1), the projection does not expand, and the output adds lam |div| <= 6 lam of
it, so `iters` steps stay below 4 * 6e-8 * 6 * 0.2 * iters of values near 0.5:
under 1e-5 for the 15 steps run here."""

import numpy as np
import pytest

import oracle
from helpers import rel_l2, report

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,iters,shift", [
    (32, 32, 1, 1, 0), (32, 64, 5, 2, 0), (64, 32, 17, 15, 0), (192, 96 * 2, 3, 3, 1), (384, 32, 33, 4, 3),
    (128, 512, 2, 5, 0), (512, 64, 18, 2, 1)])
def test_tv_tiles_match_oracle(nx, ny, nz, iters, shift):
    import torch
    from paper_2406_13651_amd import _clamp as C
    rng = np.random.default_rng(nx + 3 * ny + 7 * nz)
    x = (rng.uniform(0.0, 1.0, (nz, ny, nx)) + (rng.uniform(size=(nz, ny, nx)) > 0.9)).astype(np.float32)
    plan = C.clamp_plan_create([C.Scene(nx, ny, nz, 1, nx / 4.0)])
    ws = plan.workspace()
    buf = torch.zeros(2, x.size + 4, device="cuda")
    src, out = buf[0, shift:shift + x.size], buf[1, shift:shift + x.size]
    src.copy_(torch.from_numpy(x.ravel()))
    lam = float(np.float32(0.2))
    C.clamp_prior_tv(plan, 0, lam, iters, src, out, ws)
    torch.cuda.synchronize()
    want, _ = oracle.tv_prox(x.astype(np.float64), lam, iters)
    err = rel_l2(out.cpu().numpy().reshape(x.shape), want)
    assert report("tv tiles %dx%dx%d, %d steps" % (nx, ny, nz, iters), err, 1e-5) <= 1e-5
    assert float(buf[1, :shift].abs().sum()) == 0.0 and float(buf[1, shift + x.size:].abs().sum()) == 0.0
