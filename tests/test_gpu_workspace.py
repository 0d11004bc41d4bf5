"""The plan's workspace: what the forward agents need, with the TV agent's dual
fields inside it, and calls of different kinds taking turns on one workspace."""

import numpy as np
import pytest

import oracle
import synth
from helpers import rel_l2, report

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,looks,radius", [(256, 64, 8, 2, 16.0), (384, 192, 5, 3, 48.0), (64, 64, 6, 1, 1.0)])
def test_workspace_size(nx, ny, nz, looks, radius):
    """At most the two band buffers and A d of every look, a quarter of a look's
    bytes for the partial sums, and four floats a voxel; or the six floats a
    voxel of the dual fields where those are more."""
    from paper_2406_13651_amd import _clamp as C
    plan = C.clamp_plan_create([C.Scene(nx, ny, nz, looks, radius)])
    info, n = plan.info[0], nx * ny * nz
    tile = 8 if ny == 384 else 16
    band = looks * nz * ny * -(-info["B"] // tile) * tile * 8
    agents = 2 * band + looks * nz * info["P"] * 8 + looks * n * 2 + 16 * n + 8192
    assert plan.workspace().numel() <= max(agents, 24 * n + 1024)


@pytest.mark.parametrize("fused", [True, False])
def test_tv_prior_shares_the_agents_workspace(fused):
    """The TV agent's scratch and the forward agents' overlap: a run that
    alternates them against the oracle (float32 roundings of 3 iterations,
    below 1e-5 as without a TV agent)."""
    import torch
    import paper_2406_13651_amd as G
    spec = synth.SceneSpec("ws", 64, 32, 9, 2, 8.0, 10.0, 4, 0.05, 1, 3)
    _, y, s2w = synth.make_problem(spec, 0)
    f32 = lambda v: float(np.float32(v))
    lam = f32(0.05)
    g = G.ClampGPU(64, 32, 9, 2, 8.0, s2w, 1e-3, fused=fused, prior="tv", prior_weight=lam, tv_iters=3)
    g.init(torch.from_numpy(y).cuda())
    g.run(3)
    torch.cuda.synchronize()
    assert int(g.fault.item()) == 0
    mask = oracle.pupil_mask(32, 64, 8.0)
    st = oracle.clamp_init(y, mask, True, 1.0)
    for _ in range(3):
        h = oracle.clamp_iteration(st, y, mask, f32(s2w), f32(1e-3), 0.5, lambda v: oracle.tv_prox(v, lam, 3)[0])
    assert report("tv run wbar fused=%d" % fused, rel_l2(g.wbar.cpu().numpy(), h["wbar"]), 1e-5) <= 1e-5
    assert report("tv run mu fused=%d" % fused, rel_l2(g.mu.cpu().numpy(), st.mu), 1e-5) <= 1e-5


def test_cnn_training_workspace():
    """Bytes a voxel of a training step: the packed input, seven activations of
    32 channels and their ReLU patterns, the output (which its gradient
    replaces), the output gradient in 8 channels, two gradients of 32."""
    from paper_2406_13651_amd import _clamp as C
    v = 32 * 64 * 64
    per = (C.clamp_cnn_workspace_size(24, 32, 64, 64, True) - C.clamp_cnn_workspace_size(12, 32, 64, 64, True)) / (12 * v)
    assert per <= 16 + 7 * 64 + 7 * 4 + 4 + 16 + 2 * 64 + 0.01


def test_unet_training_workspace():
    """Bytes a voxel of a U-Net training step, level by level: z and the
    activation of four convolutions, the pooled tensor, skip sum and its
    gradient, three gradients; and a ReLU pattern for the layers whose
    backward-data product reads it (three at full resolution, two below)."""
    from paper_2406_13651_amd import _clamp as C
    v = 32 * 32 * 128
    per = (C.clamp_unet_workspace_size(24, 32, 32, 128, True) - C.clamp_unet_workspace_size(12, 32, 32, 128, True)) / (12 * v)
    levels = 1 + 1 / 8 + 1 / 64
    want = 16 + 4 + 16 + levels * (4 * 128 + 2 * 64 + 3 * 64) + 64 * (1 / 8 + 1 / 64 + 2 / 512)
    assert per <= want + 4 * (3 + 2 / 8 + 2 / 64) + 0.01
