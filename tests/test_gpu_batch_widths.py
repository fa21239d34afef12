"""The c2r pass of a batch takes each box at its own tile width: one launch per distinct width, whatever the others are tuned
to, and the results of separate runs bit for bit (directly launched, recorded and replayed)."""
import numpy as np
import pytest

import synth
from tests.gpu_util import particle_set, requires_gpu, say, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]

MESHES = (32, 48, 64, 48, 90)


@pytest.fixture(autouse=True)
def builtin_tiling_after():
    yield
    from paper_1506_03737_amd import lpc
    lpc.lpc_profile_enable(False)
    lpc.lpc_fft_tiling_reset()


def particle_arrays(lpc, arrays):
    ps = particle_set(lpc, *arrays)
    return ps.pos, ps.vel


@pytest.mark.parametrize("widths,launches", [({}, 1), ({48: 4}, 2), ({48: 4, 64: 8}, 3), ({90: 8}, 2)])
def test_own_width(widths, launches):
    from paper_1506_03737_amd import lpc
    say(f"batched: c2r widths {widths}")
    for nm, rows in widths.items():
        lpc.lpc_fft_tiling_set(nm, dict(lpc.lpc_fft_tiling_get(nm), c2r_rows=rows))
    step, cosmo, a, box, n = lpc.stepping(), lpc.cosmology(**synth.COSMOLOGY), synth.A_LIST[:3], 90.0, 12**3
    rng = np.random.default_rng(3)
    inputs = [((rng.random((3, n)) * 0.999 * box).astype(np.float32), *rng.standard_normal((3, 3, n)).astype(np.float32))
              for _ in MESHES]
    geoms = [lpc.geometry(12, nm, box) for nm in MESHES]
    single = []
    for geom, arrays in zip(geoms, inputs):
        ps = particle_set(lpc, *arrays)
        lpc.lpc_cola_step(geom, cosmo, step, a, ps, lpc.workspace(geom, lpc.LPC_OP_COLA_STEP))
        single.append((to_np(ps.pos), to_np(ps.vel)))
    sets = [particle_set(lpc, *arrays) for arrays in inputs]
    entries = list(zip(geoms, sets))
    ws = lpc.workspace_batched(entries)
    for profiled in (True, False, False):
        for ps, arrays in zip(sets, inputs):
            for t, v in zip((ps.pos, ps.vel), particle_arrays(lpc, arrays)):
                t.copy_(v)
        lpc.lpc_profile_enable(profiled)
        lpc.lpc_profile_reset()
        lpc.lpc_cola_step_batched(entries, cosmo, step, a, ws)
        if profiled:
            assert lpc.lpc_profile_stats()["fft z c2r"][0] == launches * len(a)
        lpc.lpc_profile_enable(False)
        for i, (ps, (x, v)) in enumerate(zip(sets, single)):
            assert np.array_equal(to_np(ps.pos), x) and np.array_equal(to_np(ps.vel), v), i

