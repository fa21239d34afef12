"""The fused x pass on meshes with a compiled plan in its unchained form, whose instances carry no run-time stages, and next to
boxes without a compiled plan, where the instance carries both.

Bars as between two tilings of one mesh (test_gpu_fft_plans.py: relative L2 2e-6, max 2e-5 of the largest component); batched
boxes equal their single runs bit for bit."""
import numpy as np
import pytest

import synth
from tests.gpu_util import rel_l2, requires_gpu, say, to_dev
from tests.test_gpu_fft_plans import builtin_tiling_after, force  # noqa: F401

pytestmark = [pytest.mark.gpu, requires_gpu]


# 4 columns of 8 points; 8 of 8 and 12; 16 of 8, 12 and 16 points a thread (768 and 1024 hold no 16 columns)
@pytest.mark.parametrize("nm", [192, 256, 320, 384, 768])
def test_unchained_widths(nm):
    from paper_1506_03737_amd import lpc
    box = 300.0
    pos_d = to_dev(synth.clustered_positions(7, 100003, box))
    default = lpc.lpc_fft_tiling_default(nm)
    ref, widths = force(lpc, pos_d, nm, box), []
    for cols in (4, 8, 16):
        try:
            lpc.lpc_fft_tiling_set(nm, dict(default, poisson_cols=cols))
        except lpc.LpcError:
            continue  # not a width that this mesh takes
        widths.append(cols)
        g = force(lpc, pos_d, nm, box)
        assert rel_l2(g, ref) < 2e-6, cols
        assert np.abs(g - ref).max() < 2e-5 * np.abs(ref).max(), cols
    say(f"x pass: nm = {nm}, widths {widths}")
    assert 4 in widths and 8 in widths


def test_batch_with_and_without_compiled_plans():
    from paper_1506_03737_amd import lpc
    from tests.test_gpu_batched import batched_run, box_ic, single_runs
    say("x pass: a batch of 384 and 90, and of 384 alone")
    a, step = synth.A_LIST[:3], lpc.stepping()
    for boxes in ([(32, 384, 150.0, 31), (30, 90, 160.0, 32)], [(32, 384, 150.0, 31), (24, 384, 170.0, 33)]):
        ics = [box_ic(n, L, seed) for (n, nm, L, seed) in boxes]
        ref = single_runs(lpc, ics, boxes, a, step)
        got, _, _, _ = batched_run(lpc, ics, boxes, a, step)
        for i, ((x, v), (xr, vr)) in enumerate(zip(got, ref)):
            assert np.array_equal(x, xr) and np.array_equal(v, vr), i
