"""The bucket scan of the particle sort on either side of the line between its two forms (one workgroup up to 10240 buckets,
256^3, and three launches above): the deposit of what it sorted equals the oracle's integer density bit for bit."""
import numpy as np
import pytest

from oracle import pm as opm
from tests.gpu_util import requires_gpu, say, to_dev, to_np, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("nm", [250, 256, 270, 320])
def test_density_around_the_line(nm):
    from paper_1506_03737_amd import lpc
    say(f"sort scan: nm = {nm}")
    n, box = 30011, float(nm)
    pos = (np.random.default_rng(nm).random((3, n)) * 0.9999 * box).astype(np.float32)
    geom = lpc.geometry(2, nm, box)
    ws = lpc.workspace(geom, lpc.LPC_OP_PM_FORCE, n_particles=n)
    ws.fill_(255)
    grad = torch.empty((3, n), device="cuda")
    dens = torch.empty((nm,) * 3, dtype=torch.int64, device="cuda")
    for _ in range(2):
        lpc.lpc_pm_force(geom, lpc.stepping(), to_dev(pos), grad, ws, density_out=dens)
        assert np.array_equal(to_np(dens), opm.deposit_fixed(pos, nm, box))
