"""The split form of the tile deposit: tiles that hold many more particles than the rest are worked on in chunks, whose counts
are added in slots of a workspace region of limited size.

Each test first works out, by the library's rule, how many tiles are past the trigger and how many slots and list entries
there are, and fails if its particles would not take the form that it is about. The counts are integers: the density equals
the oracle's bit for bit, also where slots or list entries run out, and the force is the same whether the deposit writes
counts or the contrast. A cell's count overflows at 2^63, which 32768 particles on its node reach and 32767 do not."""
import numpy as np
import pytest

from oracle import pm as opm
from tests.gpu_util import requires_gpu, say, to_dev, to_np, torch

pytestmark = [pytest.mark.gpu, requires_gpu]

TILE = (16, 8, 32)       # cells
CHUNK = 4096             # particles
SMALLEST = 1 << 17       # particles of a box that may be split


def split_plan(nm, n):
    """(slots, list entries, trigger) of lpc_pm_force: the space after the contrast in the 12 nm^3 bytes of the force mesh."""
    up = lambda b: (b + 255) // 256 * 256  # noqa: E731
    tiles = np.prod([-(-nm // t) for t in TILE])
    room = 12 * nm**3 - up(4 * nm**3)
    entries = room // 64
    slots = (room - up(8) - up(4 * tiles) - up(8 * entries) - 512) // (2 * 4096 * 8 + 4)
    return slots, entries, max(8192, 4 * n // tiles, min(n // 400, 65535))


def reach(pos, nm, box):
    """Particles that reach each tile, as the deposit counts them: its own and the boundary ones of its lower neighbours."""
    cell = (np.floor(pos.astype(np.float64) * (nm * 65536.0 / box)).astype(np.int64) >> 16) % nm
    grid = tuple(-(-nm // t) for t in TILE)
    tile = [cell[d] // TILE[d] for d in range(3)]
    last = [np.minimum(nm, (tile[d] + 1) * TILE[d]) - 1 for d in range(3)]
    edge = (cell[0] == last[0]) | (cell[1] == last[1]) | (cell[2] == last[2])
    own = np.zeros(grid, dtype=np.int64)
    np.add.at(own, tuple(tile), 1)
    bound = np.zeros(grid, dtype=np.int64)
    np.add.at(bound, tuple(t[edge] for t in tile), 1)
    total = own.copy()
    for q in range(1, 8):
        axes = [d for d in range(3) if q >> (2 - d) & 1]
        if all(grid[d] > 1 for d in axes):
            total += np.roll(bound, 1, axis=axes) if len(axes) == 1 else np.roll(bound, (1,) * len(axes), axis=axes)
    return total


def check(pos, nm, box):
    """Density and force of a particle set, from lpc_pm_force with and without the density output."""
    from paper_1506_03737_amd import lpc
    n = pos.shape[1]
    pos_d = to_dev(pos)
    geom, step = lpc.geometry(2, nm, box), lpc.stepping()
    ws = lpc.workspace(geom, lpc.LPC_OP_PM_FORCE, n_particles=n)
    ws.fill_(255)
    dens = torch.empty((nm,) * 3, dtype=torch.int64, device="cuda")
    with_counts, without = torch.empty((3, n), device="cuda"), torch.empty((3, n), device="cuda")
    lpc.lpc_pm_force(geom, step, pos_d, with_counts, ws, density_out=dens)
    assert np.array_equal(to_np(dens), opm.deposit_fixed(pos, nm, box))
    for _ in range(2):
        lpc.lpc_pm_force(geom, step, pos_d, without, ws)
        assert torch.equal(with_counts, without)


def shell(seed, count, tile, fill):
    """count positions (box = mesh side) spread over the boundary cells of the tile at `tile`, `fill` more over its inside."""
    rng = np.random.default_rng(seed)
    x = rng.random((3, count))
    lo = np.asarray(tile, dtype=np.float64)[:, None] * np.asarray(TILE)[:, None]
    axis = rng.integers(0, 3, count)
    x = x * np.asarray(TILE)[:, None]
    for d in range(3):
        x[d] = np.where(axis == d, TILE[d] - 1 + 0.999 * rng.random(count), x[d] * 0.999)
    inside = rng.random((3, fill)) * (np.asarray(TILE)[:, None] - 1.01)
    return (lo + np.concatenate([x, inside], axis=1)).astype(np.float32)


def test_clumps_with_room():
    """Several split tiles, next to whole ones, some of them past 2^16 particles and across narrow last tiles."""
    nm = 90
    rng = np.random.default_rng(1)
    parts = [rng.random((3, 60000)) * 0.9999 * nm]
    for k, centre in enumerate(((20.0, 30.0, 40.0), (88.0, 88.5, 89.0), (8.0, 60.0, 63.9))):
        parts.append(np.mod(np.asarray(centre)[:, None] + (0.8 + k) * rng.standard_normal((3, 90000)), 0.9999 * nm))
    pos = np.concatenate(parts, axis=1).astype(np.float32)
    pos = pos[:, rng.permutation(pos.shape[1])]
    assert not opm.fixed_point_overflow(pos, nm, float(nm))
    slots, entries, trigger = split_plan(nm, pos.shape[1])
    r = reach(pos, nm, float(nm))
    hot = r[r > trigger]
    say(f"deposit split: {hot.size} tiles past {trigger} of {slots} slots, most {hot.max()}")
    assert pos.shape[1] >= SMALLEST and 3 <= hot.size <= slots and hot.max() > 1 << 16
    check(pos, nm, float(nm))


@pytest.mark.parametrize("count,entries_run_out", [(1 << 18, False), (5_700_000, True)])
def test_slots_and_entries_run_out(count, entries_run_out):
    """The boundary particles of one tile reach eight: more tiles than slots, and with many particles more chunks than list
    entries. The tiles without a slot or entries stay whole."""
    nm = 40
    pos = shell(2, count - 4000, (0, 1, 0), 4000)
    slots, entries, trigger = split_plan(nm, count)
    r = reach(pos, nm, float(nm))
    hot = np.sort(r[r > trigger])
    say(f"deposit split: {hot.size} tiles past {trigger}, {slots} slots, {entries} entries")
    assert hot.size > slots
    assert (np.sum(-(-hot[:slots] // CHUNK)) > entries) == entries_run_out
    check(pos, nm, float(nm))


@pytest.mark.parametrize("node", [(4, 4, 4), (15, 7, 31)], ids=["inside", "corner"])
@pytest.mark.parametrize("others", [2000, 60000], ids=["below-2^16", "past-2^16"])
@pytest.mark.parametrize("on_node,overflow", [(32767, False), (32768, True)])
def test_overflow_of_chunks(node, others, on_node, overflow):
    nm = 64
    rng = np.random.default_rng(4)
    near = rng.uniform(6.0, 6.99, (3, others))  # in the first tile, sharing no cell with the node
    far = rng.uniform(33.0, 63.0, (3, SMALLEST))
    pos = np.concatenate([np.repeat(np.asarray(node, dtype=np.float64)[:, None], on_node, axis=1), near, far], axis=1)
    pos = pos.astype(np.float32)[:, rng.permutation(pos.shape[1])]
    expect_overflow(pos, nm, overflow, past=others > 1 << 15)


def test_overflow_that_wraps_to_zero():
    """65536 particles on a node: the 64-bit sum of the chunks' counts is 0 again, the sum of their high parts is not."""
    nm = 64
    rng = np.random.default_rng(5)
    pos = np.concatenate([np.full((3, 65536), 4.0), rng.uniform(33.0, 63.0, (3, SMALLEST))], axis=1)
    expect_overflow(pos.astype(np.float32)[:, rng.permutation(pos.shape[1])], nm, True, past=True)


def expect_overflow(pos, nm, overflow, past):
    from paper_1506_03737_amd import lpc
    n = pos.shape[1]
    slots, entries, trigger = split_plan(nm, n)
    r = reach(pos, nm, float(nm))
    hot = r[r > trigger]
    say(f"deposit split: {hot.size} of {slots} slots, first tile reached by {r[0, 0, 0]}, overflow {overflow}")
    assert n >= SMALLEST and r[0, 0, 0] > trigger and hot.size <= slots and (r[0, 0, 0] >= 1 << 16) == past
    geom, step = lpc.geometry(2, nm, float(nm)), lpc.stepping()
    ws = lpc.workspace(geom, lpc.LPC_OP_PM_FORCE, n_particles=n)
    grad = torch.empty((3, n), device="cuda")
    dens = torch.empty((nm,) * 3, dtype=torch.int64, device="cuda")
    for out in (None, dens):
        if overflow:
            with pytest.raises(lpc.LpcError) as err:
                lpc.lpc_pm_force(geom, step, to_dev(pos), grad, ws, density_out=out)
            assert err.value.status == -5
        else:
            lpc.lpc_pm_force(geom, step, to_dev(pos), grad, ws, density_out=out)
