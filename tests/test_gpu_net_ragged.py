"""Weight gradients on grids that are no multiple of the MFMA kernel's 4 x 4 x 32 bricks, at any of the three levels.

Bars: the errors fall with D (the gradients sum BF16 products over more voxels), so each grid takes the table of the next
smaller one in test_gpu_net.
"""
import numpy as np
import pytest

from oracle import net as onet
from tests.gpu_util import rel_l2, requires_gpu, say, to_dev, to_np, torch
from tests.test_gpu_net import GRAD_BARS, GRAD_L2, cf_to_grid, max_rel, sample

pytestmark = [pytest.mark.gpu, requires_gpu]


# levels 12, 6, 3 / 24, 12, 6 / 36, 18, 9 / 40, 20, 10 / 60, 30, 15
@pytest.mark.parametrize("D,bars", [(12, 8), (24, 16), (36, 32), (40, 32), (60, 32)])
def test_ragged_gradient_matches_oracle(D, bars):
    from paper_1506_03737_amd import lpc
    say(f"net: ragged gradient D={D}")
    params = lpc.lpc_net_init(12)
    params[onet.layer_slices()["out"][0]] *= 10.0
    feat, target = sample(D, 2)
    grad = torch.empty(params.size, dtype=torch.float32, device="cuda")
    lpc.lpc_net_loss_grad(D, to_dev(params), to_dev(cf_to_grid(feat)), to_dev(cf_to_grid(target)), grad,
                          lpc.net_workspace(D))
    _, g = onet.loss_and_grad(params.astype(np.float64), feat.astype(np.float64), target.astype(np.float64))
    gg = to_np(grad).astype(np.float64)
    assert rel_l2(gg, g) < GRAD_L2[bars]
    for name, (ws_, bs, _, _, _) in onet.layer_slices().items():
        e = (rel_l2(gg[ws_], g[ws_]), max_rel(gg[ws_], g[ws_]), rel_l2(gg[bs], g[bs]), max_rel(gg[bs], g[bs]))
        assert all(v < b for v, b in zip(e, GRAD_BARS[bars][name])), (name, e)
