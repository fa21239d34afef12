"""The binning of lpc_power_spectrum where its runs and signs change: meshes whose half rows are not whole runs of 8, odd half
lengths, few and many bins (also more bins than modes), bins that end below, at and past the mesh's corner. Mode counts are
exact; bin means of k to 1e-12 (FP64 sums); P to 1e-6 of an FP64 transform of the same density (FP32 transforms: their
rounding of 1e-7 per value averages over the modes of a bin, but a bin may hold a single weak mode, so the bar is taken
against the largest P of the call)."""
import numpy as np
import pytest

import synth
from oracle import spectrum as ospec
from tests.gpu_util import requires_gpu, say, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("nm", [8, 10, 16, 18, 30, 50, 54, 100, 128])
@pytest.mark.parametrize("reach,bins", [(0.3, 1), (1.0, 7), (1.8, 300), (2.0, 2048)])
def test_bins(nm, reach, bins):
    from paper_1506_03737_amd import lpc
    say(f"power_spectrum: nm = {nm}, {bins} bins to {reach} of the Nyquist wavenumber")
    box, n = 3.0 * nm, 7 * nm * nm
    pos = synth.clustered_positions(nm + bins, n, box)
    geom = lpc.geometry(2, nm, box)
    ws = lpc.workspace(geom, lpc.LPC_OP_POWER_SPECTRUM, n_particles=n)
    ws.fill_(255)
    k_max = reach * np.pi * nm / box
    k, pk, cnt = lpc.lpc_power_spectrum(geom, to_dev(pos), k_max, bins, ws)
    kr, pr, cr = ospec.power_spectrum(pos, nm, box, k_max, bins)
    assert np.array_equal(cnt, cr)
    ok = cr > 0
    assert np.array_equal(np.isnan(pk), ~ok) and np.array_equal(np.isnan(k), ~ok)
    if ok.any():
        assert np.allclose(k[ok], kr[ok], rtol=1e-12)
        assert np.abs(pk - pr)[ok].max() <= 1e-6 * pr[ok].max()
