"""Measure every projection tile over a grid of step shapes and fit the
planner's cost model.

For each shape and each tile its path offers (forced with KB_TILE), the
projection kernel of kbest_step is timed with HIP events on its own stream
(median of the timed launches after warm-up), on three sets of operands in
turn: a decoder's other layers displace W from the caches between two of its
steps, and tiles that read W once per row tile look up to 20% better when the
256 MB memory-side cache holds it (bf16, 300 x 1000 x 49,999: 64 x 256 tiles 81
us of one set, 97 of three; 128 x 256 77 and 79).  Then, per tile, the model

    t = (a H + e) w + f        w = rows x words one workgroup covers
                                 = tile rows x tile words x tiles per split,
                                 doubled for a tile at two workgroups per CU
                                 whose grid exceeds 256 workgroups

is fitted by least squares on relative error and then refined for the
choices it leads to (refine), and the choice the model makes on each shape is compared with the fastest tile measured there, the
merge's growth with the splits (merge_us) added to both.  The
planner's tables in csrc/kbest_abi.hip come from this script's fits, one per
path (k = 5): --dtype f32 (aligned shapes, H 256-2048, multiples of 64, V
8k-60k, 40-1,280 rows: kF32DmaCosts), f32reg (H 264-2056: kF32Costs), bf16
(the DMA pipeline, H 512-2048, V 8k-90k, 12-2,560 rows: kBf16DmaCosts) and
bf16reg (H 500-2000, odd V of 8,001-90,001, 12-2,560 rows: kBf16Costs).

    python -m paper_1805_09863_amd.tune_planner --dtype bf16 --out gpurun_out/tune_bf16.json

Operands are drawn on the device (normal h, W scaled by 1/sqrt(H), small
uniform bias); times do not depend on their values beyond the candidate
work a flat prior gives.
"""
from __future__ import annotations

import argparse
import json
import os
import sys

import numpy as np
import torch

from paper_1805_09863_amd import binding
from paper_1805_09863_amd.hipevents import HipEvents

TILES = {  # KB_TILE value -> (rows, words) per tile
    "256x256": (256, 256), "128x256": (128, 256), "256x128": (256, 128),
    "32x512": (32, 512), "32x256": (32, 256), "32x128": (32, 128), "64x128": (64, 128),
    "64x256": (64, 256),
}
GRIDS = {
    "f32": dict(H=(256, 512, 1024, 2048), V=(8000, 30000, 60000),
                N=(40, 64, 100, 160, 240, 320, 480, 640, 960, 1280),
                tiles=("128x256", "256x128", "32x512", "32x256", "32x128", "64x128", "64x256")),
    "f32reg": dict(H=(264, 520, 1032, 2056), V=(8000, 30000, 60000),
                   N=(40, 64, 100, 160, 240, 320, 480, 640, 960, 1280),
                   tiles=("128x256", "256x128", "32x512", "32x256", "32x128", "64x256")),
    "bf16reg": dict(H=(500, 1000, 2000), V=(8001, 30001, 50001, 90001),
                    N=(12, 24, 40, 64, 100, 160, 240, 320, 480, 640, 960, 1280, 2560),
                    tiles=("128x256", "256x128", "32x512", "32x256", "32x128", "64x256")),
    "bf16": dict(H=(512, 1024, 2048), V=(8000, 30000, 50000, 90000),
                 N=(12, 24, 40, 64, 100, 160, 200, 240, 260, 280, 300, 320, 400, 480, 640, 960, 1280, 2560),
                 tiles=tuple(TILES)),
}


SETS = 3  # weight arrays that the timed steps take in turn


def per_cu(dtype, tile: str) -> int:
    """Workgroups one CU holds at once, as the planner counts them at k <= 8:
    two of the aligned paths' 32 x 128 and 64 x 128 tiles, one of every other."""
    return 2 if dtype in ("f32", "bf16") and tile in ("32x128", "64x128") else 1


def workgroup_words(N: int, V: int, rows: int, words: int, per: int = 1) -> int:
    """rows x words one workgroup covers, with the planner's split rule."""
    rt, nt = -(-N // rows), -(-V // words)
    P = max(1, min(per * 256 // rt, nt, 256))
    return rows * words * -(-nt // P)


def model_words(N: int, V: int, rows: int, words: int, per: int = 1) -> int:
    """The model's w: a workgroup's rows x words, doubled for a tile planned at
    two workgroups per CU once its grid (row tiles x splits) exceeds 256."""
    w = workgroup_words(N, V, rows, words, per)
    rt, nt = -(-N // rows), -(-V // words)
    tps = w // (rows * words)
    return w * (2 if per == 2 and rt * -(-nt // tps) > 256 else 1)


def planner_skips(N: int, V: int, tile: str, dtype) -> bool:
    """The planner uses the small tiles for one tile per split only."""
    rows, words = TILES[tile]
    if dtype is None or tile not in ("32x128", "64x128"):
        return False
    return workgroup_words(N, V, rows, words, per_cu(dtype, tile)) > rows * words


def merge_us(N: int, V: int, tile: str, dtype) -> float:
    """The planner's term for the merge of a step's splits (none for a bare model)."""
    if dtype is None:
        return 0.0
    rows, words = TILES[tile]
    tps = workgroup_words(N, V, rows, words, per_cu(dtype, tile)) // (rows * words)
    return 0.02 * max(0, -(-(-(-V // words)) // tps) - 64)


def ragged_us(N: int, V: int, tile: str, dtype, k: int = 5) -> float:
    """The planner's term for a last tile alone in its split with too few words
    for a threshold (none for a bare model)."""
    rows, words = TILES[tile]
    one = workgroup_words(N, V, rows, words, per_cu(dtype, tile)) == rows * words
    left = V % words
    return 0.2 * left if dtype is not None and one and left * 32 < k * words else 0.0


def measure(dtype: str, grid: dict, reps: int, log, sets: int = SETS, whole: bool = False) -> list:
    ev = HipEvents()
    code = binding.KB_BF16 if dtype.startswith("bf16") else binding.KB_F32
    want = {"bf16": ("wide", "dma"), "f32": ("dma",), "f32reg": ("reg",), "bf16reg": ("reg",)}[dtype]
    tdt = torch.bfloat16 if dtype.startswith("bf16") else torch.float32
    g = torch.Generator(device="cuda").manual_seed(7)
    rows = []
    for H in grid["H"]:
        for V in grid["V"]:
            W = [(torch.randn((H, V), generator=g, device="cuda") / H ** 0.5).to(tdt) for _ in range(sets)]
            b = (torch.rand(V, generator=g, device="cuda") - 0.5) * 0.2
            for N in grid["N"]:
                S = (N + 4) // 5
                h = torch.randn((N, H), generator=g, device="cuda").to(tdt)
                prev = torch.zeros(N, device="cuda")
                off = torch.tensor([min(i * 5, N) for i in range(S + 1)], dtype=torch.int32, device="cuda")
                out = tuple(torch.empty((S, 5), dtype=t, device="cuda")
                            for t in (torch.int32, torch.int32, torch.float32))
                rec = {"H": H, "V": V, "N": N, "whole": whole, "us": {}}
                for tile in grid["tiles"]:
                    os.environ["KB_TILE"] = tile
                    plan = binding.kbest_plan(code, N, H, V, 5)
                    if f"{plan['tile_rows']}x{plan['tile_words']}" != tile or plan["kernel"] not in want:
                        continue  # not on this path
                    ws = binding.workspace(binding.kbest_workspace_bytes(code, N, H, V, 5, S))
                    for i in range(sets):
                        binding.kbest_step(h, W[i], b, prev, off, 5, out=out, ws=ws)
                    torch.cuda.synchronize()
                    t = []
                    if whole:
                        for _ in range(max(3, reps // 5)):
                            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                            e0.record()
                            for i in range(5 * sets):
                                binding.kbest_step(h, W[i % sets], b, prev, off, 5, out=out, ws=ws)
                            e1.record()
                            e1.synchronize()
                            t.append(e0.elapsed_time(e1) * 1e3 / (5 * sets))
                    else:
                        pairs = [(ev.create(), ev.create()) for _ in range(reps)]
                        for i, (a, c) in enumerate(pairs):
                            binding.kbest_step(h, W[i % sets], b, prev, off, 5, out=out, ws=ws, events=(a, c))
                        torch.cuda.synchronize()
                        t = [ev.elapsed_ms(a, c) * 1e3 for a, c in pairs]
                        for a, c in pairs:
                            ev.destroy(a)
                            ev.destroy(c)
                    rec["us"][tile] = sorted(t)[len(t) // 2]
                    del ws
                os.environ.pop("KB_TILE", None)
                rows.append(rec)
                log(json.dumps(rec))
            del W, b
            torch.cuda.empty_cache()
    return rows


def fit(rows: list, tiles, dtype=None) -> dict:
    """(a, e, f) per tile: least squares on relative error, over the shapes
    that the planner may use the tile on, without a last tile that has a term of its own."""
    out = {}
    for tile in tiles:
        r, w = TILES[tile]
        pts = [x for x in rows if tile in x["us"] and not planner_skips(x["N"], x["V"], tile, dtype)
               and not ragged_us(x["N"], x["V"], tile, dtype)]
        if len(pts) < 3:
            continue
        pc = per_cu(dtype, tile)
        X = np.array([[x["H"] * model_words(x["N"], x["V"], r, w, pc), model_words(x["N"], x["V"], r, w, pc), 1.0]
                      for x in pts])
        y = np.array([x["us"][tile] for x in pts])
        c, *_ = np.linalg.lstsq(X / y[:, None], np.ones_like(y), rcond=None)
        err = np.abs(X @ c - y) / y
        out[tile] = {"a": float(c[0]), "e": float(c[1]), "f": float(c[2]),
                     "mean_rel_err": float(err.mean()), "max_rel_err": float(err.max())}
    return out


def evaluate(rows: list, model: dict, dtype=None) -> dict:
    """The model's choice on each shape against the fastest tile measured."""
    worst, tot_choice, tot_best, logs = 1.0, 0.0, 0.0, []
    for x in rows:
        cands = [t for t in model if t in x["us"] and not planner_skips(x["N"], x["V"], t, dtype)]
        if not cands:
            continue

        def pred(t):
            r, w = TILES[t]
            wg = model_words(x["N"], x["V"], r, w, per_cu(dtype, t))
            m = model[t]
            return (m["a"] * x["H"] + m["e"]) * wg + m["f"] + merge_us(x["N"], x["V"], t, dtype) + ragged_us(x["N"], x["V"], t, dtype)
        us = {t: u + merge_us(x["N"], x["V"], t, dtype) for t, u in x["us"].items()}
        choice, best = us[min(cands, key=pred)], min(us.values())
        tot_choice += choice
        tot_best += best
        worst = max(worst, choice / best)
        logs.append(np.log(choice / best))
    return {"sum_us_model_choice": tot_choice, "sum_us_best": tot_best, "worst_ratio": worst,
            "geomean_ratio": float(np.exp(np.mean(logs)))}


def refine(rows: list, model: dict, dtype, steps: int = 12000, seed: int = 0) -> dict:
    """The model's constants moved, by a random search from the fit, to where
    its choices lose least: the mean log of their ratio to the fastest tile,
    ratios above 1.06 again at half weight, a little for the worst one and for
    the distance from the fit."""
    tiles = list(model)
    n, m = len(rows), len(tiles)
    us, w, extra = np.full((n, m), np.inf), np.zeros((n, m)), np.zeros((n, m))
    for i, x in enumerate(rows):
        for k, t in enumerate(tiles):
            if t in x["us"]:
                us[i, k] = x["us"][t] + (0.0 if x.get("whole") else merge_us(x["N"], x["V"], t, dtype))
                w[i, k] = model_words(x["N"], x["V"], *TILES[t], per_cu(dtype, t))
                extra[i, k] = merge_us(x["N"], x["V"], t, dtype) + ragged_us(x["N"], x["V"], t, dtype)
                if planner_skips(x["N"], x["V"], t, dtype):
                    extra[i, k] = np.inf
    extra[np.isinf(us)] = np.inf
    H, best = np.array([x["H"] for x in rows], float), us.min(1)
    c0 = np.array([[model[t][q] for q in "aef"] for t in tiles])
    scale = np.abs(c0) + (0.0, 5e-5, 1.0)

    def objective(c):
        pred = (c[:, 0] * H[:, None] + c[:, 1]) * w + c[:, 2] + extra
        r = us[np.arange(n), pred.argmin(1)] / best
        return (np.log(r).mean() + 0.5 * np.maximum(0, r - 1.06).mean() + 0.01 * np.log(r.max())
                + 0.002 * (((c - c0) / scale) ** 2).mean())
    rng, c, least = np.random.default_rng(seed), c0, objective(c0)
    for _ in range(steps):
        d = c + scale * rng.standard_normal(c.shape) * rng.choice((.01, .03, .1)) * (rng.random(c.shape) < .25)
        if (d[:, 0] > 0).all() and (v := objective(d)) < least:
            c, least = d, v
    return {t: dict(model[t], a=float(c[k, 0]), e=float(c[k, 1]), f=float(c[k, 2])) for k, t in enumerate(tiles)}


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n\n")[0])
    ap.add_argument("--dtype", choices=tuple(GRIDS), required=True)
    ap.add_argument("--reps", type=int, default=15)
    ap.add_argument("--out", required=True, help="JSON: measured times, fitted constants, evaluation")
    ap.add_argument("--rows", help="comma-separated row counts in place of the grid's (e.g. 9,16,24,32)")
    ap.add_argument("--also", nargs="*", default=[],
                    help="JSON files of earlier runs whose rows join the refinement")
    ap.add_argument("--whole", action="store_true", help="time whole steps, the merge included")
    ap.add_argument("--sets", type=int, default=SETS, help="weight arrays the timed steps take in turn")
    ap.add_argument("--check", action="store_true",
                    help="no fit: compare the library's own choice (kb_kbest_plan) with the fastest tile")
    args = ap.parse_args()

    def log(msg):
        print(msg, file=sys.stderr, flush=True)
    grid = dict(GRIDS[args.dtype])
    if args.rows:
        grid["N"] = tuple(int(x) for x in args.rows.split(","))
    rows = measure(args.dtype, grid, args.reps, log, args.sets, args.whole)
    if args.check:
        code = binding.KB_BF16 if args.dtype.startswith("bf16") else binding.KB_F32
        for x in rows:
            p = binding.kbest_plan(code, x["N"], x["H"], x["V"], 5)
            x["planner"] = f"{p['tile_rows']}x{p['tile_words']}"
            if not args.whole:
                x["us"] = {t: u + merge_us(x["N"], x["V"], t, args.dtype) for t, u in x["us"].items()}
        res = {"dtype": args.dtype, "grid": {k: list(v) for k, v in grid.items()}, "rows": rows,
               "sum_us_planner": sum(x["us"][x["planner"]] for x in rows),
               "sum_us_best": sum(min(x["us"].values()) for x in rows),
               "worst_ratio": max(x["us"][x["planner"]] / min(x["us"].values()) for x in rows)}
        with open(args.out, "w") as f:
            json.dump(res, f)
        log(json.dumps({k: v for k, v in res.items() if k.startswith(("sum", "worst"))}))
        return
    model = fit(rows, grid["tiles"], args.dtype)
    for path in args.also:
        with open(path) as f:
            rows = rows + json.load(f)["rows"]
    model = refine(rows, model, args.dtype)
    res = {"dtype": args.dtype, "grid": {k: list(v) for k, v in grid.items()}, "rows": rows,
           "fit": model, "evaluation_of_the_planner_set": evaluate(rows, model, args.dtype)}
    with open(args.out, "w") as f:
        json.dump(res, f)
    for t, m in model.items():
        log(f"{t:8s} a={m['a']:.3e} e={m['e']:.3e} f={m['f']:.2f}  rel err mean {m['mean_rel_err']:.3f} "
            f"max {m['max_rel_err']:.3f}")
    log(json.dumps(res["evaluation_of_the_planner_set"]))


if __name__ == "__main__":
    main()
