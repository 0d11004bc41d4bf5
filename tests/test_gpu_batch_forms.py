"""Batches large enough that each wave of the fused update pass walks every
look of its rows (every row length), against single-scene calls of the same
scenes.  There up to four waves share the looks and hand r over through the
row buffers, and slices of 32 and 64 points take the one-launch passes, where
the batch takes the column, row and column passes.  All of them use the same
float32 operations in the same order, so every array of the state is equal bit
for bit; the float64 diagnostics differ by the order of their sums at most:
up to 1e5 positive terms added in runs, below 1e-14 relative."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ITERS = 3
ROWS_PER_WAVE = {32: 16, 64: 8, 128: 4, 192: 2, 256: 2, 384: 1, 512: 1}

# nx, ny, nz, looks, radius, with_prior: the last scene alone fills the chip
SCENES = {
    32: [(32, 32, 33, 6, 22.7, True), (32, 64, 3, 5, 8.0, True), (32, 512, 12, 9, 8.0, True),
         (32, 512, 26, 2, 8.0, False)],
    64: [(64, 64, 9, 7, 45.5, True), (64, 32, 5, 3, 15.9, False), (64, 64, 120, 2, 16.0, True)],
    128: [(128, 64, 3, 4, 16.0, True), (128, 128, 25, 2, 32.0, True)],
    192: [(192, 64, 5, 6, 101.5, True), (192, 192, 8, 3, 48.0, False)],
    256: [(256, 32, 3, 5, 8.0, True), (256, 128, 13, 2, 32.0, True)],
    384: [(384, 64, 5, 7, 193.0, True), (384, 192, 4, 3, 48.0, False)],
    512: [(512, 32, 5, 5, 8.0, True), (512, 128, 7, 2, 64.0, False)],
}


@pytest.mark.parametrize("nx", sorted(SCENES))
def test_full_batches_equal_single_scenes(nx):
    import torch
    import paper_2406_13651_amd as G
    scenes = SCENES[nx]
    groups = sum(s[1] * s[2] // ROWS_PER_WAVE[nx] for s in scenes)
    assert groups > 3 * torch.cuda.get_device_properties(0).multi_processor_count  # else four waves share
    b = G.ClampBatchGPU([dict(nx=s[0], ny=s[1], nz=s[2], looks=s[3], radius=s[4], sigma_w2=0.1, sigma2=1e-3,
                              with_prior=s[5]) for s in scenes])
    gen = torch.Generator(device="cuda").manual_seed(nx)
    ys = [torch.randn((s[3], s[2], s[1], s[0]), dtype=torch.complex64, device="cuda", generator=gen) for s in scenes]
    b.init(ys)
    for _ in range(ITERS):
        b.step()
    torch.cuda.synchronize()
    assert int(b.fault.item()) == 0
    for i, s in enumerate(scenes):
        g = G.ClampGPU(*s[:5], 0.1, 1e-3, with_prior=s[5])
        g.init(ys[i])
        g.run(ITERS)
        torch.cuda.synchronize()
        st = b.states[i]
        for name in ("mu", "r", "resid", "w", "wbar", "xbar"):
            assert torch.equal(st[name], getattr(g, name)), (s, name)
        np.testing.assert_allclose(st["diag"].cpu().numpy(), g.diag.cpu().numpy(), rtol=1e-14, atol=0)
        assert abs(b.conv[i].item() - g.conv_err()) <= 1e-14 * g.conv_err()
