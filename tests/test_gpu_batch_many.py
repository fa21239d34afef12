"""lpc_cola_step_batched with as many boxes as its job tables have always held: 490 boxes of one size and of several sizes.
Bar: bit-for-bit equality with separate runs (as in test_gpu_batched.py), for the first, the last and some between."""
import numpy as np
import pytest

import synth
from tests.gpu_util import particle_set, requires_gpu, say, to_np

pytestmark = [pytest.mark.gpu, requires_gpu]

COUNT = 490


@pytest.mark.parametrize("meshes", [(8,), (8, 10, 12, 16, 18)], ids=["one-size", "several-sizes"])
def test_many_boxes(meshes):
    from paper_1506_03737_amd import lpc
    say(f"batched: {COUNT} boxes on meshes {meshes}")
    rng = np.random.default_rng(len(meshes))
    box, n, step, cosmo = 40.0, 27, lpc.stepping(), lpc.cosmology(**synth.COSMOLOGY)
    a = synth.A_LIST[:3]
    sets, entries, inputs = [], [], []
    for i in range(COUNT):
        pos = (rng.random((3, n)) * box).astype(np.float32)
        pos[pos >= box] = 0.0
        vel, psi1, psi2 = rng.standard_normal((3, 3, n)).astype(np.float32)
        inputs.append((pos, vel, psi1, psi2))
        sets.append(particle_set(lpc, *inputs[-1]))
        entries.append((lpc.geometry(3, meshes[i % len(meshes)], box), sets[-1]))
    lpc.lpc_cola_step_batched(entries, cosmo, step, a, lpc.workspace_batched(entries))
    for i in list(range(0, COUNT, 61)) + [COUNT - 1]:
        ps = particle_set(lpc, *inputs[i])
        geom = entries[i][0]
        lpc.lpc_cola_step(geom, cosmo, step, a, ps, lpc.workspace(geom, lpc.LPC_OP_COLA_STEP))
        assert np.array_equal(to_np(sets[i].pos), to_np(ps.pos)), i
        assert np.array_equal(to_np(sets[i].vel), to_np(ps.vel)), i
