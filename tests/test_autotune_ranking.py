"""The tuner ranks a pass's widths with the other passes at the widths that they will run at: a pass's time depends on what the
pass before it leaves in the caches. Stage times here are a made-up function of the tiling in effect; no GPU."""
import pytest


@pytest.fixture(autouse=True)
def builtin_tiling_after():
    yield
    from paper_1506_03737_amd import lpc
    lpc.lpc_fft_tiling_reset()


def test_pass_behind_another_is_ranked_at_the_picked_width(monkeypatch):
    import torch
    from paper_1506_03737_amd import autotune, lpc
    nm = 192
    seen = []

    def stage_ms(run, reps):
        t = lpc.lpc_fft_tiling_get(nm)
        seen.append(t)
        y = {8: 2.0, 16: 1.0, 32: 1.5}[t["axis_cols"]]
        # 4 rows are the fastest behind the slow y pass only
        c2r = {4: 0.8, 8: 1.0, 16: 1.2} if t["axis_cols"] == 8 else {4: 1.3, 8: 1.0, 16: 1.2}
        return {"fft z r2c": 1.0 / t["z_rows"], "fft y": y, "fft y inv": 2 * y,
                "fft x + poisson": {4: 3.0, 8: 1.0, 16: 2.0}[t["poisson_cols"]], "fft z c2r": c2r[t["c2r_rows"]]}

    monkeypatch.setattr(autotune, "_stage_ms", stage_ms)
    monkeypatch.setattr(lpc, "lpc_pm_force", lambda *a, **k: None)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    res = autotune.tune(nm, "cpu")
    assert res["tiling"] == {"z_rows": 32, "axis_cols": 16, "poisson_cols": 8, "c2r_rows": 8}
    assert lpc.lpc_fft_tiling_get(nm) == res["tiling"]
    assert {f: sorted(int(w) for w in v) for f, v in res["stage_ms"].items()} == \
        {f: sorted(w) for f, w in autotune.candidates(nm).items()}
    # while the c2r widths were timed, the y pass ran at its pick
    assert {t["axis_cols"] for t in seen[-len(res["stage_ms"]["c2r_rows"]):]} == {16}
