"""GPU parity of the learned prior's gradients at the edges of the work split
of the one-channel weight gradients and of the ReLU patterns: rows that do not
fill a 16-row tile, a single slice, a single row, an odd number of 32-voxel
runs, several volumes.

Tolerance: every stored activation and gradient is rounded to bfloat16 on both
sides (relative 2^-9), and a rounding decided the other way by the float32
accumulation costs as much; through about 20 such stages (ten layers forward
and back) the errors add in squares to sqrt(20) 2^-9 = 8.7e-3 of a layer's
gradient at most, taken twice: 2e-2."""

import numpy as np
import pytest

from oracle import cnn as ocnn
from helpers import rel_l2, report
from test_gpu_cnn import C, _setup, bf16_params  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 1, 5, 32), (1, 3, 17, 96), (2, 2, 16, 64), (1, 9, 1, 32), (1, 17, 33, 32)])
def test_gradients_at_tile_edges(C, shape):  # noqa: F811
    net, params, x, t, torch = _setup(C, seed=11, shape=shape)
    xt, tt = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    grad = torch.full((C.CNN_PARAMS,), np.nan, dtype=torch.float32, device="cuda")
    ws = torch.full((C.clamp_cnn_workspace_size(*shape, True),), 255, dtype=torch.uint8, device="cuda")
    C.clamp_cnn_grad(net, xt, tt, loss, ws, grad=grad)
    torch.cuda.synchronize()
    _, ref = ocnn.loss_and_grads(x.astype(np.float64), t.astype(np.float64), bf16_params(params), act_round=True)
    g = grad.cpu().numpy().astype(np.float64)
    off = 0
    for l, (w, b) in enumerate(params):
        for name, n, want in (("dW", w.size, ref[l][0]), ("db", b.size, ref[l][1])):
            e = rel_l2(g[off:off + n], np.asarray(want).ravel())
            off += n
            report("cnn edge %s layer %d %s" % (name, l, shape), e, 2e-2)
            assert e <= 2e-2
