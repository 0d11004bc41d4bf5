"""The short chains of small scenes against the float64 oracle, at the edges
of their tilings: the one-launch passes of a slice (32- and 64-point
transforms, equal and unequal lengths, pupils from three band columns to the
whole row, one slice, odd slice counts, the 3D operator), and the fused
update pass with one, two or four waves sharing a row group's looks (look
counts that the sharing does not divide), and the 192- and 384-point rows of
the split transform.  The forward agents alone and with
the Mann step fused in.

Bound: each iteration's arrays carry a few float32 roundings of the FFTs and
the pointwise steps (about 1e-7 each, the sums in float64); 3 iterations stay
below 1e-5."""

import numpy as np
import pytest

import oracle
import synth
from helpers import rel_l2, report

pytestmark = pytest.mark.gpu

TOL = 1e-5
ITERS = 3

CASES = [
    # nx, ny, nz, looks, radius, with_prior, range_support
    (32, 32, 1, 2, 1.0, True, 0),
    (32, 64, 3, 5, 8.0, True, 0),
    (64, 32, 5, 7, 15.9, False, 0),
    (64, 64, 9, 1, 16.0, True, 0),
    (64, 64, 2, 3, 45.5, True, 0),    # every row and column in the band
    (32, 32, 33, 6, 22.7, True, 0),   # every sample of a slice
    (64, 32, 16, 4, 8.0, True, 9),
    (64, 64, 130, 9, 16.0, False, 0),  # two waves per row group
    (128, 64, 3, 4, 16.0, True, 0),    # four waves, three-pass gradient
    (256, 32, 2, 3, 8.0, True, 0),
    (192, 32, 2, 6, 8.0, True, 0),     # rows that do not fill their threads
    (192, 64, 3, 4, 101.5, True, 0),   # the same with every sample of a row in the band
    (384, 32, 3, 5, 193.0, True, 0),
    (384, 64, 5, 1, 2.0, False, 0),
]


def f32(x):
    return float(np.float32(x))


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("nx,ny,nz,looks,radius,with_prior,K", CASES,
                         ids=["%dx%dx%d_L%d_R%g_prior%d_K%d" % c for c in CASES])
def test_small_scene_runs_match_oracle(nx, ny, nz, looks, radius, with_prior, K, fused):
    import torch
    import paper_2406_13651_amd as G
    spec = synth.SceneSpec("slices", nx, ny, nz, looks, radius, 10.0, 4, 0.05, 1, 3)
    r_true, y, s2w = synth.make_problem(spec, 0, range_support=K)
    g = G.ClampGPU(nx, ny, nz, looks, radius, s2w, 1e-3, with_prior=with_prior, range_support=K, fused=fused)
    g.init(torch.from_numpy(y).cuda())
    conv = []
    for _ in range(ITERS):
        g.iterate()
        conv.append(g.conv_err())
    torch.cuda.synchronize()
    assert int(g.fault.item()) == 0
    mask = oracle.cylinder_mask(nz, ny, nx, radius, K) if K > 0 else None
    st, hist = oracle.clamp_run(y, radius, f32(s2w), f32(1e-3), ITERS, with_prior=with_prior, mask=mask)
    tag = "%dx%dx%d L=%d R=%g K=%d fused=%d" % (nx, ny, nz, looks, radius, K, fused)
    assert report(tag + " wbar", rel_l2(g.wbar.cpu().numpy(), hist[-1]["wbar"]), TOL) <= TOL
    assert report(tag + " w", rel_l2(g.state_w().cpu().numpy(), st.w), TOL) <= TOL
    assert report(tag + " mu", rel_l2(g.mu.cpu().numpy(), st.mu), TOL) <= TOL
    ref = np.array([h["conv_err"] for h in hist])
    assert report(tag + " conv_err", rel_l2(np.array(conv), ref), TOL) <= TOL
    # diagnostics: h before and after of every look differ by gamma ||d||^2 / 2
    d = g.diag.cpu().numpy()
    want = 0.5 * d[:looks, G.DG_GAMMA] * d[:looks, G.DG_DD]
    got = d[:looks, G.DG_H0] - d[:looks, G.DG_H1]
    assert np.allclose(got, want, rtol=0, atol=2e-6 * np.abs(d[:looks, G.DG_H0]).max())
