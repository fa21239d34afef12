"""The forms of the tile deposit: 256 and 1024 threads per tile, and tiles split over several workgroups when they hold many
more particles than the others (while there are slots for their chunks). The counts are integers, so every form gives the
oracle's density bit for bit, and the force is the same whether the deposit writes counts or the contrast."""
import numpy as np
import pytest

from oracle import pm as opm
from tests.gpu_util import requires_gpu, say, to_dev, to_np, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


def clump(seed, n, box, share, width, centre):
    """share of the particles in one Gaussian clump of the given width (in boxes) around centre, the rest uniform."""
    rng = np.random.default_rng(seed)
    k = int(share * n)
    inside = np.asarray(centre)[:, None] + width * rng.standard_normal((3, k))
    pos = np.concatenate([inside, rng.random((3, n - k))], axis=1) % 1.0 * box
    pos = pos.astype(np.float32)
    pos[pos >= box] = 0.0
    return pos[:, rng.permutation(n)]


@pytest.mark.parametrize("nm,n,share,width", [
    (8, 30000, 0.5, 0.05),       # one tile, no room for slots
    (20, 100003, 0.9, 0.01),     # more chunks than slots: the tile stays whole
    (36, 20000, 0.0, 0.1),       # uniform and sparse: nothing to split
    (32, 200001, 0.3, 0.1),      # many per tile: 1024 threads
    (64, 300007, 0.8, 0.005),    # a clump within a tile and over its faces
    (64, 2000003, 0.5, 0.02),    # 1024 threads and split tiles of more than 2^16 particles each
    (90, 250001, 0.9, 0.03),     # several split tiles, narrow last tiles
    (128, 150000, 0.99, 0.003),
])
def test_density_of_clumps(nm, n, share, width):
    from paper_1506_03737_amd import lpc
    box = 100.0
    for centre in ((0.5, 0.5, 0.5), (0.99, 0.02, 0.25)):
        say(f"deposit: nm = {nm}, n = {n}, clump of {share} within {width} at {centre}")
        pos = clump(nm + n, n, box, share, width, centre)
        pos_d = to_dev(pos)
        geom, step = lpc.geometry(2, nm, box), lpc.stepping()
        ws = lpc.workspace(geom, lpc.LPC_OP_PM_FORCE, n_particles=n)
        ws.fill_(255)
        dens = torch.empty((nm,) * 3, dtype=torch.int64, device="cuda")
        with_counts, without = torch.empty((3, n), device="cuda"), torch.empty((3, n), device="cuda")
        if opm.fixed_point_overflow(pos, nm, box):  # (90 % of 100003 particles around a node)
            for out in (dens, None):
                with pytest.raises(lpc.LpcError) as err:
                    lpc.lpc_pm_force(geom, step, pos_d, with_counts, ws, density_out=out)
                assert err.value.status == -5
            continue
        lpc.lpc_pm_force(geom, step, pos_d, with_counts, ws, density_out=dens)
        assert np.array_equal(to_np(dens), opm.deposit_fixed(pos, nm, box))
        for _ in range(2):
            lpc.lpc_pm_force(geom, step, pos_d, without, ws)
            assert torch.equal(with_counts, without)


@pytest.mark.parametrize("extra,overflow", [(0, False), (1, True)])
def test_overflow_of_a_split_tile(extra, overflow):
    """2^63 is reached by 32768 particles on a node; the tile holds 60000 more elsewhere and is split."""
    from paper_1506_03737_amd import lpc
    nm, box = 64, 64.0
    say(f"deposit: {32767 + extra} particles on a node of a split tile")
    rng = np.random.default_rng(4)
    pos = np.concatenate([np.full((3, 32767 + extra), 4.0), rng.uniform(6.0, 7.0, (3, 60000))], axis=1).astype(np.float32)
    assert opm.fixed_point_overflow(pos, nm, box) == overflow
    geom = lpc.geometry(2, nm, box)
    ws = lpc.workspace(geom, lpc.LPC_OP_PM_FORCE, n_particles=pos.shape[1])
    grad = torch.empty((3, pos.shape[1]), device="cuda")
    if overflow:
        with pytest.raises(lpc.LpcError) as err:
            lpc.lpc_pm_force(geom, lpc.stepping(), to_dev(pos), grad, ws)
        assert err.value.status == -5
    else:
        lpc.lpc_pm_force(geom, lpc.stepping(), to_dev(pos), grad, ws)
