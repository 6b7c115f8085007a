"""Fit the constants of the tile dispatcher's cost model (sk_default_tile, sk_plan_estimate_us) to timings.

Input: one sweep file per tile shape of an input width, made with

    python -m paper_2408_11417_amd.sweep --suite model --graph --tile 256,256,64 --out model_bf16_256,256,64.json
    python -m paper_2408_11417_amd.sweep --suite model --graph --dtype e4m3 --tile 256,256,128 --out model_e4m3_256,256,128.json

(the same sizes in every file; 16- and 8-bit files are fitted apart; without --graph the host's launch rate
hides the differences between the small sizes).  Such a file holds the time of every
schedule - whole tiles in waves, a Stream-K region of so many tiles, everything split - of the tile on every
size.  The model predicts each of them, and the dispatcher takes the tile of the smallest prediction, the
selector's fall-back the schedule.  The fit minimises the regret of that pick of tile and schedule (its time /
the time of the fastest of all tiles and schedules) by random local search over the constants on the sweep,
skinny and deep sizes that lie on the 16-byte grid; the others are only reported.  The constants are fitted for
the quality of the pick, not for predicting times: they need not be physical (several parameter sets pick equally well).

    python -m paper_2408_11417_amd.fit_tile_model model_bf16_*.json
    python -m paper_2408_11417_amd.fit_tile_model --check model_bf16_*.json       (the library's constants only, no fit)

Prints the regret by family of sizes, of the library's constants and of the fitted ones, and the latter in the
order they appear in csrc/streamk_plan.cpp.  CPU only.

How the library's constants came about: the 16- and the 8-bit ones each by such a fit over the same sizes, after
which the large 8-bit tile was given the large 16-bit one's constants (it moves the same bytes with twice the k at
twice the rate); level_us and the two exchange rates are those of the 16-bit fit for both; STAGED_TILE was chosen
by hand among 1.0 .. 2.0 by the picks on the odd sizes.
"""
import json
import math
import sys

import numpy as np

GRID = 256
# The constants as they stand in csrc/streamk_plan.cpp (tile_costs16, tile_costs8, MODEL_*).  The library's C++ code
# is what runs; schedule_us() below restates its formula, and tests/test_selector.py checks that predict() with
# these constants picks sk_default_tile's tile.
LIBRARY = {"bk": {(256, 256): 64, (256, 128): 64, (128, 128): 64, (64, 128): 64, (32, 128): 64, (16, 128): 64, (64, 64): 128, (32, 64): 64},
           "tflops": {(256, 256): 1590., (256, 128): 1307., (128, 128): 1062., (64, 128): 745., (32, 128): 478., (16, 128): 287.,
                      (64, 64): 500., (32, 64): 364.},
           "tile_us": {(256, 256): 10.40, (256, 128): 5.61, (128, 128): 4.33, (64, 128): 2.91, (32, 128): 2.73, (16, 128): 2.68,
                       (64, 64): 3.08, (32, 64): 2.76},
           "level_us": 1.68, "fetch_bytes_per_us": 107e3, "traffic_bytes_per_us": 6.953e6, "piece": 8}
LIBRARY8 = {"bk": {(256, 256): 128, (128, 256): 128, (128, 128): 128, (64, 128): 128, (32, 128): 128},
            "tflops": {(256, 256): 3180., (128, 256): 2821., (128, 128): 1919., (64, 128): 1467., (32, 128): 915.},
            "tile_us": {(256, 256): 10.40, (128, 256): 4.75, (128, 128): 2.61, (64, 128): 2.45, (32, 128): 2.48},
            "level_us": 1.68, "fetch_bytes_per_us": 107e3, "traffic_bytes_per_us": 6.953e6, "piece": 16}
STAGED_TILE = 1.6      # MODEL_STAGED_TILE: problems whose rows are off the 16-byte grid ("piece": elements of 16 bytes)


def cdiv(a, b):
    return -(-a // b)


def terms(bm, bn, bk, M, N, K, sk_tiles, piece):
    """What a schedule that splits sk_tiles of the tiles over the grid takes of each constant: MAC-loop flops, tile
    times, exchange levels, bytes of one owner's chain of fetches, bytes of all partial tiles together."""
    ipt, T = cdiv(K, bk), cdiv(M, bm) * cdiv(N, bn)
    flops = 2.0 * bm * bn * bk * GRID                    # of one k-iteration of every workgroup
    staged = STAGED_TILE if N % piece or K % piece else 1.0
    waves = cdiv(T - sk_tiles, GRID)
    if sk_tiles == 0:
        return waves * ipt * flops, waves * staged, 0.0, 0.0, 0.0
    iters = sk_tiles * ipt
    ipw = cdiv(iters, GRID)
    split_tiles = ipw % ipt != 0 and iters > ipw
    n_iter = waves * ipt + ipw
    n_tile = (waves + max(sk_tiles / GRID if split_tiles else ipw // ipt, 1.0)) * staged
    if not split_tiles:
        return n_iter * flops, n_tile, 0.0, 0.0, 0.0
    # partial tiles an owner (or a group leader) fetches one after the other: all of them up to 16
    # workgroups per tile, beyond that the two-level reduction with groups of 8; and all of them together
    split = max(ipt / ipw, 1.0)
    serial = split if split < 16 else 8 + split / 8
    others = cdiv(iters, ipw) - 1
    contributors = others - others // (ipt // math.gcd(ipt, ipw))
    return n_iter * flops, n_tile, 1.0 if split < 16 else 2.0, serial * bm * bn * 4, contributors * bm * bn * 8.0


def schedule_us(P, tile, M, N, K, sk_tiles):
    """Microseconds of one schedule of a tile shape (model_us in C++)."""
    flops, n_tile, levels, chain, traffic = terms(*tile, P["bk"][tile], M, N, K, sk_tiles, P["piece"])
    return (flops / (P["tflops"][tile] * 1e6) + n_tile * P["tile_us"][tile] + levels * P["level_us"] +
            chain / P["fetch_bytes_per_us"] + traffic / P["traffic_bytes_per_us"])


def predict(P, tile, M, N, K):
    """The cost model of sk_default_tile for one tile shape (microseconds): its cheapest schedule."""
    T = cdiv(M, tile[0]) * cdiv(N, tile[1])
    return min(schedule_us(P, tile, M, N, K, s) for s in (0, T, T % GRID))


class Timings:
    """Every timed (size, tile, schedule) as one row: its measured time and its terms of the model.  The model is
    linear in the constants' inverses, so a prediction of all rows is one matrix product."""

    def __init__(self, files, piece):
        self.tiles, sizes, rows = [], None, []
        for f in files:
            recs = json.load(open(f))["records"]
            bm, bn, bk = recs[0]["tile"]
            self.tiles.append((bm, bn, bk))
            these = [(r["M"], r["N"], r["K"]) for r in recs]
            assert sizes in (None, these), "the sweep files must cover the same sizes"
            sizes = these
            for j, r in enumerate(recs):
                for s, t in {s: t for s, t in zip(r["sk_tiles"], r["time_ns"])}.items():
                    rows.append((j, len(self.tiles) - 1, t / 1000.0) + terms(bm, bn, bk, *these[j], s, piece))
        self.sizes = sizes
        self.size, self.tile = np.array([r[0] for r in rows]), np.array([r[1] for r in rows])
        self.us = np.array([r[2] for r in rows])
        n = len(self.tiles)
        self.X = np.zeros((len(rows), 2 * n + 3))
        for i, r in enumerate(rows):
            self.X[i, r[1]], self.X[i, n + r[1]] = r[3] / 1e6, r[4]
            self.X[i, 2 * n:] = r[5:]
        order = np.argsort(self.size, kind="stable")
        for name in ("size", "tile", "us", "X"):
            setattr(self, name, getattr(self, name)[order])
        self.first = np.searchsorted(self.size, np.arange(len(sizes)))
        self.best = np.minimum.reduceat(self.us, self.first)

    def regret(self, constants):
        """Per size: the time of the schedule predicted fastest over the fastest time."""
        pred = self.X @ constants
        lowest = np.minimum.reduceat(pred, self.first)
        at_lowest = np.where(pred == lowest[self.size], self.us, np.inf)      # (ties are one schedule timed twice: the faster)
        return np.minimum.reduceat(at_lowest, self.first) / self.best

    def constants(self, P):
        shapes = [t[:2] for t in self.tiles]
        return np.array([1 / P["tflops"][t] for t in shapes] + [P["tile_us"][t] for t in shapes] +
                        [P["level_us"], 1 / P["fetch_bytes_per_us"], 1 / P["traffic_bytes_per_us"]])


def describe(r):
    return "%.3f (%.2f at most, %d of %d above 1.1)" % (math.exp(np.log(r).mean()), r.max(), (r > 1.1).sum(), len(r))


def main():
    from . import inputs
    check = "--check" in sys.argv[1:]
    files = [f for f in sys.argv[1:] if f != "--check"]
    if not files:
        raise SystemExit(__doc__)
    fp8 = json.load(open(files[0]))["dtype"] == "e4m3"
    library = LIBRARY8 if fp8 else LIBRARY
    T = Timings(files, library["piece"])
    family = {}
    for name, members in inputs.model_sizes().items():
        for size in members:
            family.setdefault(size, name)
    names = np.array([family.get(size, "other") for size in T.sizes])
    aligned = np.array([N % library["piece"] == 0 and K % library["piece"] == 0 for M, N, K in T.sizes])

    def report(label, constants):
        r = T.regret(constants)
        for name in dict.fromkeys(names):
            of = (names == name) & (aligned | np.char.startswith(names, "odd"))
            if of.any():
                print("  %s, %s sizes: %s" % (label, name, describe(r[of])))
    print("time of the pick of tile and schedule over the fastest of all, geometric mean:")
    report("the library's constants", T.constants(library))
    if check:
        return 0
    train = aligned & ~np.char.startswith(names, "odd")
    n = len(T.tiles)

    def score(constants):
        r = T.regret(constants)[train]
        return np.log(r).mean() + 0.5 * (r > 1.2).mean()
    start = np.array([1 / ((8.8 if fp8 else 4.4) * math.sqrt(t[0] * t[1])) for t in T.tiles] + [2.0 + t[0] * t[1] / 8e3 for t in T.tiles] +
                     [2.0, 1 / 80e3, 1 / 6e6])
    fits = []
    for seed in range(4):
        rng = np.random.default_rng(10 + seed)
        P, s = start.copy(), score(start)
        for _ in range(5000):
            Q = P.copy()
            Q[rng.integers(len(Q))] *= math.exp(rng.normal(0, 0.15))
            sq = score(Q)
            if sq < s:
                P, s = Q, sq
        fits.append((s, P))
        print("restart %d: score %.4f" % (seed, s))
    P = min(fits, key=lambda f: f[0])[1]
    report("fitted", P)
    for i, t in enumerate(T.tiles):
        print("  {%d, %d, %d, %.0f., %.2f}," % (*t, 1 / P[i], P[n + i]))
    print("  level %.2f us, one owner's chain %.4g bytes per us, all partial traffic %.4g bytes per us" % (P[-3], 1 / P[-2], 1 / P[-1]))
    return 0


if __name__ == "__main__":
    sys.exit(main())
