"""Stage timing of calls that do a stage's work in another stage's launch: the
stage is counted once per call and has no time, and stages with a launch of
their own have some."""

import pytest

import synth

pytestmark = pytest.mark.gpu


def _timed(C, plan, step):
    import torch
    step()
    C.clamp_plan_set_timing(plan, True)
    step()
    torch.cuda.synchronize()
    C.clamp_plan_set_timing(plan, False)
    return C.clamp_plan_get_timing(plan)


@pytest.mark.parametrize("n,absorbed", [(32, {"col_inv", "col_fwd", "mace_step"}), (128, {"mace_step"})])
@pytest.mark.parametrize("batch", [False, True])
def test_absorbed_stages_have_no_time(n, absorbed, batch):
    import torch
    import paper_2406_13651_amd as G
    from paper_2406_13651_amd import _clamp as C
    spec = synth.SceneSpec("t", n, n, 4, 2, n / 4.0, 10.0, 4, 0.05, 1, 3)
    _, y, s2 = synth.make_problem(spec, 0)
    yt = torch.from_numpy(y).cuda()
    if batch:
        b = G.ClampBatchGPU([dict(nx=n, ny=n, nz=4, looks=2, radius=n / 4.0, sigma_w2=s2, sigma2=1e-3)])
        b.init([yt])
        st = _timed(C, b.plan, b.step)
        absorbed = {"mace_step"}  # a batch keeps the column passes' launches
    else:
        g = G.ClampGPU(n, n, 4, 2, n / 4.0, s2, 1e-3)
        g.init(yt)
        st = _timed(C, g.plan, g.iterate)
    for name, (ms, count) in st.items():
        assert count == 1, name
        assert (ms == 0.0) == (name in absorbed), (name, ms)
    assert absorbed <= set(st)
