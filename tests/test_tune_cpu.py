"""The tile override (KB_TILE) and the planner-tuning script's fit, on the CPU."""
import numpy as np
import pytest

import paper_1805_09863_amd as kb
from paper_1805_09863_amd import tune_planner as tp


@pytest.fixture
def tile_env(monkeypatch):
    def set_tile(v):
        if v is None:
            monkeypatch.delenv("KB_TILE", raising=False)
        else:
            monkeypatch.setenv("KB_TILE", v)
    return set_tile


def _p(dt, N, H, V, aligned=True):
    p = kb.kbest_plan(dt, N, H, V, 5, aligned=aligned)
    return f"{p['kernel']} {p['tile_rows']}x{p['tile_words']}"


def test_tile_override_follows_the_path(tile_env):
    def ignored(tile, *step, **kw):
        # the choice, and its splits, are those made without the override
        tile_env(None)
        want = kb.kbest_plan(*step, 5, **kw)
        tile_env(tile)
        return kb.kbest_plan(*step, 5, **kw) == want

    tile_env(None)
    assert _p(kb.KB_BF16, 640, 1024, 60000) == "wide 256x256"
    tile_env("32x512")
    assert _p(kb.KB_BF16, 640, 1024, 60000) == "dma 32x512"
    assert _p(kb.KB_F32, 640, 1024, 60000) == "dma 32x512"
    assert _p(kb.KB_F32, 640, 1000, 60000) == "reg 32x512"
    tile_env("256x256")
    assert _p(kb.KB_BF16, 40, 1024, 50000) == "wide 256x256"
    assert ignored("256x256", kb.KB_F32, 320, 512, 30000)             # no 256 x 256 tile there
    assert ignored("256x256", kb.KB_F32, 320, 520, 30000)
    assert ignored("256x256", kb.KB_BF16, 640, 1024, 60000, aligned=False)
    assert ignored("256x256", kb.KB_BF16, 300, 128, 200)              # V < 256
    tile_env("64x128")
    assert _p(kb.KB_BF16, 640, 1024, 60000) == "dma 64x128"
    assert _p(kb.KB_F32, 640, 1024, 60000) == "dma 64x128"
    assert ignored("64x128", kb.KB_BF16, 640, 1000, 60000)            # the register-staged path has no such tile
    assert ignored("64x256", kb.KB_BF16, 640, 16, 60000)              # nor has the direct kernel this one
    tile_env("32x512")
    assert _p(kb.KB_BF16, 640, 16, 60000) == "reg 32x512"
    tile_env("128x256")
    assert _p(kb.KB_F32, 5, 256, 8000) == "few 8x64"                  # the few-row kernel keeps its steps
    for bad in ("64x64", "32x256x", "x", "", "256"):
        tile_env(bad)
        assert _p(kb.KB_BF16, 640, 1024, 60000) == "wide 256x256"


def test_small_tiles_only_one_per_split():
    # of several in turn they were slower than the model says; every path, row
    # and word count still has a tile, the narrowest vocabularies included
    for dt in (kb.KB_F32, kb.KB_BF16):
        for H in (16, 256, 500, 1024):
            for V in (1, 100, 130, 200, 3001, 30000, 50000, 90001):
                for N in (9, 24, 64, 100, 257, 300, 320, 640, 2560, 9000):
                    p = kb.kbest_plan(dt, N, H, V, 1)
                    assert p["tile_rows"] in (32, 64, 128, 256) and p["row_tiles"] == -(-N // p["tile_rows"])
                    if p["tile_words"] == 128 and p["tile_rows"] < 128:
                        assert p["tiles_per_split"] == 1


@pytest.mark.parametrize("dt,N,H,V,not_tile", [
    # shapes where one tile had been preferred against the measured times
    (kb.KB_F32, 320, 520, 30000, "32x256"), (kb.KB_F32, 160, 264, 60000, "32x256"),
    (kb.KB_F32, 160, 520, 60000, "32x256"), (kb.KB_BF16, 640, 1000, 90001, "256x128"),
    (kb.KB_BF16, 320, 1024, 50000, "64x128"), (kb.KB_BF16, 257, 1024, 50000, "64x128"),
    (kb.KB_BF16, 320, 512, 90000, "64x128")])
def test_choice_is_not_the_slow_tile(tile_env, dt, N, H, V, not_tile):
    tile_env(None)
    p = kb.kbest_plan(dt, N, H, V, 5)
    assert f"{p['tile_rows']}x{p['tile_words']}" != not_tile


def test_workspace_follows_the_override(tile_env):
    tile_env(None)
    a = kb.kbest_workspace_bytes(kb.KB_BF16, 3072, 1024, 90000, 12, 256)
    tile_env("32x128")
    b = kb.kbest_workspace_bytes(kb.KB_BF16, 3072, 1024, 90000, 12, 256)
    assert b != a   # 32-row tiles give other splits, hence other partials


def test_fit_recovers_the_model_and_evaluation_picks_it():
    rng = np.random.default_rng(0)
    truth = {"32x128": (8e-6, 3e-4, 25.0), "32x512": (7e-6, 3.3e-4, 20.0), "128x256": (5e-6, 4e-4, 15.0)}
    rows = []
    for H in (256, 512, 1024, 2048):
        for V in (8000, 30000, 60000):
            for N in (40, 100, 320, 1280):
                us = {}
                for t, (a, e, f) in truth.items():
                    r, w = tp.TILES[t]
                    us[t] = ((a * H + e) * tp.workgroup_words(N, V, r, w) + f) * (1 + 0.01 * rng.standard_normal())
                rows.append({"H": H, "V": V, "N": N, "us": us})
    model = tp.fit(rows, truth)
    for t, (a, e, f) in truth.items():
        assert model[t]["a"] == pytest.approx(a, rel=0.05) and model[t]["f"] == pytest.approx(f, rel=0.1)
        assert model[t]["mean_rel_err"] < 0.02
    ev = tp.evaluate(rows, model)
    assert ev["worst_ratio"] < 1.05 and ev["sum_us_model_choice"] <= 1.02 * ev["sum_us_best"]


def test_workgroup_words_matches_the_plan(tile_env):
    # the script's split rule, two 32 x 128 workgroups per CU on the DMA pipeline included
    for dt, path, N, H, V in ((kb.KB_F32, "f32", 320, 512, 30000), (kb.KB_F32, "f32reg", 320, 520, 30000),
                              (kb.KB_BF16, "bf16", 3072, 1024, 90000), (kb.KB_BF16, "bf16", 100, 256, 8000)):
        for tile in (None, "32x128", "32x256", "128x256"):
            tile_env(tile)
            p = kb.kbest_plan(dt, N, H, V, 5)
            t = f"{p['tile_rows']}x{p['tile_words']}"
            assert tp.workgroup_words(N, V, p["tile_rows"], p["tile_words"], tp.per_cu(path, t)) == \
                p["tile_rows"] * p["tile_words"] * p["tiles_per_split"]
