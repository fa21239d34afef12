"""The strided FFT passes with run-time plans, whose first stage reads global memory and whose last stage writes it, and the
built-in tile widths at the edges of their rule.

Bars: those of the force against the FP64 oracle (relative L2 2e-5, max 2e-4 of the largest component), and between two
tilings of one mesh (2e-6, 2e-5; a width only decides how many transforms share a tile, and the chained x pass takes the same
transforms in another radix order). Batched boxes equal their single runs bit for bit.
"""
import numpy as np
import pytest

import synth
from oracle import pm as opm
from tests.gpu_util import rel_l2, requires_gpu, say, to_dev, to_np, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.fixture(autouse=True)
def builtin_tiling_after():
    yield
    from paper_1506_03737_amd import lpc
    lpc.lpc_fft_tiling_reset()


def force(lpc, pos_d, nm, box):
    n = pos_d.shape[1]
    geom = lpc.geometry(0, nm, box)
    ws = lpc.workspace(geom, lpc.LPC_OP_PM_FORCE, n_particles=n)
    grad = torch.empty((3, n), dtype=torch.float32, device="cuda")
    lpc.lpc_pm_force(geom, lpc.stepping(), pos_d, grad, ws)
    return to_np(grad)


# first and last radices: one stage (8, 12), 2..5 (10, 50), 4..5 (20), 4..4 (16), 12..3 (36), 12..5 (60), 8..12 (96), 4 4 8
# (128), 8..3 (72), 8..5 (200, 250: 2 5 5 5), with 8, 16 and 32 columns a tile (y pairs of 4, 8 and 16)
@pytest.mark.parametrize("cols", [8, 16, 32])
@pytest.mark.parametrize("nm", [8, 10, 12, 16, 20, 36, 50, 60, 72, 96, 128, 250])
def test_run_time_plans_match_oracle(nm, cols):
    from paper_1506_03737_amd import lpc
    say(f"fft plans: force at nm={nm}, {cols} columns")
    box = 200.0
    pos = synth.clustered_positions(3, 20011, box)
    lpc.lpc_fft_tiling_set(nm, dict(lpc.lpc_fft_tiling_default(nm), axis_cols=cols))
    g = force(lpc, to_dev(pos), nm, box)
    ref = opm.pm_force(pos.astype(np.float64), nm, box, deconv_power=1)
    assert rel_l2(g, ref) < 2e-5
    assert np.abs(g - ref).max() < 2e-4 * np.abs(ref).max()


@pytest.mark.parametrize("nm", [200, 216, 240, 250, 384, 400, 480, 500, 768, 800])
def test_builtin_widths_at_their_lines(nm):
    from paper_1506_03737_amd import lpc
    say(f"fft plans: built-in widths at nm={nm}")
    box = 500.0
    pos_d = to_dev(synth.clustered_positions(5, 200003, box))
    g = force(lpc, pos_d, nm, box)
    lpc.lpc_fft_tiling_set(nm, dict(z_rows=8, axis_cols=8, poisson_cols=4, c2r_rows=4))
    ref = force(lpc, pos_d, nm, box)
    assert rel_l2(g, ref) < 2e-6
    assert np.abs(g - ref).max() < 2e-5 * np.abs(ref).max()


def test_batch_of_both_x_passes_equals_single_runs():
    """64 and 90 take the plain x pass, 192 and 256 the chained one: one batch launches both."""
    from paper_1506_03737_amd import lpc
    from tests.test_gpu_batched import batched_run, box_ic, single_runs
    say("fft plans: one batch with chained and plain x passes")
    boxes = [(32, 64, 128.0, 21), (32, 192, 150.0, 22), (30, 90, 160.0, 23), (32, 256, 170.0, 24)]
    ics = [box_ic(n, L, seed) for (n, nm, L, seed) in boxes]
    a, step = synth.A_LIST[:4], lpc.stepping()
    ref = single_runs(lpc, ics, boxes, a, step)
    got, _, _, _ = batched_run(lpc, ics, boxes, a, step)
    for i, ((x, v), (xr, vr)) in enumerate(zip(got, ref)):
        assert np.array_equal(x, xr), f"box {i}: positions differ"
        assert np.array_equal(v, vr), f"box {i}: velocities differ"
