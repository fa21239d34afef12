"""The sum alpha (phi + fNL sum_g D^g[...]) of a non-Gaussian linear field is formed in more than FP32 and rounded once.

Two groups of terms that cancel, p - D^g p with g = 1e-13, and fNL = 3e8: a local kernel of fNL = 3000 is 13-110 % of the
Gaussian field (measured in test_gpu_png.py), so each group is 1e4 to 1e5 times it. k^g differs from 1 by less than 1e-12, so
what the groups leave is below 1e-6 of the field, and the fields are those of fNL = 0 to the bar of lpc_init_ic's fields,
1e-5 relative L2. Terms rounded to FP32 one by one would leave 1e4 x 2^-25 = 3e-4 or more.
"""
import pytest

import synth
from tests.gpu_util import requires_gpu, say, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


# the three tile forms of the x pass: 16 columns, 8 columns, 8 columns with 16 points per thread
@pytest.mark.parametrize("n_side", [32, 270, 540])
def test_cancelling_terms_leave_the_gaussian_field(n_side):
    from paper_1506_03737_amd import lpc
    say(f"png: cancelling terms, n_side = {n_side}")
    box = 8.0 * n_side
    geom, cosmo = lpc.geometry(n_side, 2 * n_side, box), lpc.cosmology(**synth.COSMOLOGY)
    ws = lpc.workspace(geom, lpc.LPC_OP_INIT_IC)
    terms = [(1.0, 0.0, 0.0, 0.0), (-1.0, 0.0, 0.0, 1e-13)]
    sets = []
    for f_nl in (0.0, 3e8):
        ps = lpc.ParticleSet.empty(n_side**3)
        lpc.lpc_init_ic_png(geom, cosmo, 5, synth.A_LIST[0], lpc.png(f_nl, terms=terms), ps, ws)
        sets.append(ps)
    for name in ("psi1", "psi2", "vel"):
        a, b = getattr(sets[1], name), getattr(sets[0], name)
        e = float(torch.linalg.vector_norm((a - b).double()) / torch.linalg.vector_norm(b.double()))
        say(f"  {name}: rel L2 {e:.2e}")
        assert e < 1e-5, name
