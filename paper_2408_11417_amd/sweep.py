"""Tuning sweep: time every scheduling policy on a list of GEMM shapes and record the winners.

This is the stand-in for the profiler run of the paper (Sec. 5.1): for each problem size all seven
Stream-K++ policies are launched with warm-up + timed repetitions (50 + 50 for short kernels, fewer
for long ones) and the mean kernel time is kept.  The output feeds `selector.py`, which builds the
Bloom filters (Sec. 4.2) from the winners and evaluates them on held-out shapes.

    python -m paper_2408_11417_amd.sweep --shapes 500 --seed 4 --out sweep_bf16.json

Needs a GPU.  Inputs are seeded synthetic matrices (bf16 unless --dtype says otherwise; 8-bit inputs give bf16
results), uniform in [-1, 1], carved out of two device pools that are filled once.
"""
import argparse
import json
import sys
import time

import numpy as np


def time_policy(sk, torch, plan, sets, stream, est_ms, graph=False):
    """Mean milliseconds per launch; repetitions follow the paper's 50 + 50 protocol for kernels up
    to 0.2 ms and shrink to >= 5 + 5 (about 20 ms of timed work) for longer ones.  `sets`: (A, B, D)
    pointer triples the launches rotate over, so that operands smaller than the 256 MB memory-side
    cache are not served from it launch after launch.  graph=True captures the timed launches into a
    HIP graph once and times a replay: kernels of a few microseconds are then not held up by the rate
    at which the host can enqueue them."""
    reps = 50 if est_ms <= 0.2 else max(5, int(20.0 / est_ms))
    launches = [sk.sk_gemm_bind(*ptrs, plan, stream) for ptrs in sets]     # arguments marshalled once
    for i in range(reps):
        assert launches[i % len(sets)]() == sk.SK_OK
    replay = None
    if graph:
        replay = torch.cuda.CUDAGraph()
        with torch.cuda.graph(replay):
            capture_stream = torch.cuda.current_stream().cuda_stream
            for i in range(reps):
                sk.sk_gemm(*sets[i % len(sets)], plan, capture_stream)
        replay.replay()                                  # one untimed replay
        torch.cuda.synchronize()

    def timed():
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        if replay is not None:
            replay.replay()
        else:
            for i in range(reps):
                launches[i % len(sets)]()
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1) / reps

    ms = timed()
    if ms > 1.5 * est_ms:
        # far above the single launch timed beforehand: something else held the machine up; once more
        ms = min(ms, timed())
    return ms, reps


def run(shapes, out_path, dtype_code=1, verbose=True, check_every=25, fixup=0, tile=None, dp_first=False, ascending=False, tile_order=None,
        graph=False, verify=None):
    """Time the seven policies on every shape; returns the records.  verify: optional callback
    verify(record, policy, A, B, D) called for every shape after the timing, with the fastest policy
    and host copies (numpy uint16 storage bits) of the operands of one launch of it and of its
    result - the hook through which a test compares the very launches that were timed with a
    reference of its own."""
    import torch
    import paper_2408_11417_amd as sk

    torch.cuda.set_device(0)
    stream = torch.cuda.current_stream().cuda_stream
    tdt = {sk.SK_BF16: torch.bfloat16, sk.SK_F16: torch.float16, sk.SK_FP8_E4M3: torch.float8_e4m3fn}[dtype_code]
    es = 1 if dtype_code == sk.SK_FP8_E4M3 else 2                       # bytes of an input element
    out_code, out_tdt = (sk.SK_BF16, torch.bfloat16) if es == 1 else (dtype_code, tdt)
    max_a = max(M * K for M, N, K in shapes)
    max_b = max(K * N for M, N, K in shapes)
    max_d = max(M * N for M, N, K in shapes)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1234)

    def pool(n):
        out = torch.empty(n, dtype=tdt, device="cuda")
        step = 1 << 26
        for i in range(0, n, step):
            m = min(step, n - i)
            out[i:i + m] = (torch.rand(m, device="cuda", generator=gen) * 2 - 1).to(tdt)
        return out

    # room for four copies of the largest operands, so that every size rotates over four sets
    # (at least 4 x the operand bytes between two uses of the same set: more than the 256 MB
    # memory-side cache holds for every operand above 64 MB, which is where that cache would matter)
    slack = 4 * 256
    pa, pb = pool(4 * max_a + slack), pool(4 * max_b + slack)
    pd = torch.empty(4 * max_d + slack, dtype=out_tdt, device="cuda")
    pd2 = torch.empty(max_d, dtype=out_tdt, device="cuda")
    ws_bytes = (256 + 64) * 256 * 256 * 4 + (1 << 16)      # 256 workgroups' partial tiles, and owners' where at least 4.5 share a tile
    if fixup:                                  # the atomic fix-up keeps an fp32 image of D in the workspace
        ws_bytes = max(ws_bytes, max_d * 4 + (1 << 16))
    ws = torch.empty(ws_bytes + 256, dtype=torch.uint8, device="cuda")
    ws_ptr = (ws.data_ptr() + 255) // 256 * 256

    records, t_start = [], time.time()
    for idx, (M, N, K) in enumerate(shapes):
        plans, infos = [], []
        for p in range(sk.SK_NUM_POLICIES):
            plan = sk.sk_plan(M, N, K, p, tile, 256, dtype_code, out_code, tile_order)
            sk.sk_plan_set_fixup(plan, fixup)
            if dp_first:
                sk.sk_plan_set_batch_order(plan, sk.SK_DATA_PARALLEL_FIRST)
            if ascending:
                sk.sk_plan_set_segment_order(plan, sk.SK_SEGMENTS_ASCENDING)
            assert sk.sk_workspace_bytes(plan) <= ws_bytes
            sk.sk_plan_set_workspace(plan, ws_ptr, ws_bytes)
            plans.append(plan)
            infos.append(sk.sk_plan_info(plan))
        # policies whose Stream-K region covers the same number of tiles are the same schedule
        by_sched, times, reps_used = {}, [0.0] * 7, [0] * 7
        dA, dB, dD = pa.data_ptr(), pb.data_ptr(), pd.data_ptr()
        # four operand sets carved out of the pools at 256-byte aligned offsets
        copies = 4
        step = lambda n, size: (n * size + 255) // 256 * 256
        assert step(M * K, es) * copies <= pa.numel() * es and step(K * N, es) * copies <= pb.numel() * es and step(M * N, 2) * copies <= pd.numel() * 2
        sets = [(dA + c * step(M * K, es), dB + c * step(K * N, es), dD + c * step(M * N, 2)) for c in range(copies)]
        for p in range(sk.SK_NUM_POLICIES):
            key = infos[p]["sk_tiles"]
            if key not in by_sched:
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                sk.sk_gemm(dA, dB, dD, plans[p], stream)          # first touch
                e0.record()
                sk.sk_gemm(dA, dB, dD, plans[p], stream)
                e1.record()
                e1.synchronize()
                by_sched[key] = time_policy(sk, torch, plans[p], sets, stream, e0.elapsed_time(e1), graph)
            times[p], reps_used[p] = by_sched[key]
        rec = {"M": M, "N": N, "K": K, "tile": [infos[0]["blk_m"], infos[0]["blk_n"], infos[0]["blk_k"]],
               "tiles": infos[0]["tiles"], "iters_per_tile": infos[0]["iters_per_tile"],
               "sk_tiles": [i["sk_tiles"] for i in infos], "time_ns": [int(round(t * 1e6)) for t in times],
               "reps": reps_used, "distinct_schedules": len(by_sched)}
        if check_every and idx % check_every == 0:
            # a log line, not a check: how far all-Stream-K and data-parallel results are apart (summation order only)
            sk.sk_gemm(dA, dB, pd.data_ptr(), plans[0], stream)
            sk.sk_gemm(dA, dB, pd2.data_ptr(), plans[6], stream)
            assert sk.sk_plan_check(plans[6], stream) == sk.SK_OK
            a, b = pd[:M * N].float(), pd2[:M * N].float()
            rec["dp_vs_allsk_maxdiff_over_rms"] = float((a - b).abs().max() / a.pow(2).mean().sqrt())
        if verify is not None:
            best = times.index(min(times))
            pd[:M * N].zero_()
            sk.sk_gemm(dA, dB, pd.data_ptr(), plans[best], stream)
            assert sk.sk_plan_check(plans[best], stream) == sk.SK_OK
            as_bits = lambda t, r, c: t[:r * c].view(torch.int16).cpu().numpy().view(np.uint16).reshape(r, c)
            verify(rec, best, as_bits(pa, M, K), as_bits(pb, K, N), as_bits(pd, M, N))
        records.append(rec)
        for plan in plans:
            sk.sk_plan_destroy(plan)
        if verbose and (idx % 10 == 0 or idx == len(shapes) - 1):
            best = min(times)
            print("[%4d/%d %6.0fs] %5dx%5dx%5d tile %s T=%d  best %.4f ms (%s) %.0f TFLOP/s  dp %.4f" % (
                idx + 1, len(shapes), time.time() - t_start, M, N, K, rec["tile"], rec["tiles"], best,
                sk.POLICY_NAMES[times.index(best)], 2.0 * M * N * K / best / 1e9, times[0]), flush=True)
        if out_path and (idx % 50 == 49 or idx == len(shapes) - 1):
            with open(out_path, "w") as f:
                json.dump({"dtype": {1: "bf16", 0: "f16", 2: "e4m3"}[dtype_code], "grid": 256,
                           "fixup": "atomic" if fixup else "flags", "dp_first": bool(dp_first),
                           "segment_order": "ascending" if ascending else "k_aligned",
                           "tile_order": {None: "default", 0: "row_major", 1: "grouped"}[tile_order],
                           "timing": "graph replay" if graph else "eager launches", "records": records}, f)
    return records


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--shapes", type=int, default=500)
    ap.add_argument("--seed", type=int, default=4)
    ap.add_argument("--out", default="sweep_bf16.json")
    ap.add_argument("--first", type=int, default=0, help="only the first N shapes (smoke runs)")
    ap.add_argument("--tile", default="", help="blk_m,blk_n,blk_k for every shape instead of the library's own choice")
    ap.add_argument("--skinny", action="store_true",
                    help="append the skinny family (M in 16..128, N = K in 4096, 8192; N = 16384, K = 4096) to the shapes")
    ap.add_argument("--dp-first", action="store_true",
                    help="data-parallel batches before the Stream-K work (the earlier hybrid of Sec. 3.2)")
    ap.add_argument("--suite", choices=("random", "paper", "model"), default="random",
                    help="random: log-uniform sizes (inputs.sweep_shapes); paper: a seeded sample of the power-of-two grid "
                         "of Sec. 5.1 (inputs.paper_suite); model: the sizes of the tile dispatcher's fit (inputs.model_sizes)")
    ap.add_argument("--dtype", choices=("bf16", "f16", "e4m3"), default="bf16")
    ap.add_argument("--tile-order", choices=("default", "row_major", "grouped"), default="default",
                    help="tile index -> tile grid position for every plan (default: the library's choice per schedule)")
    ap.add_argument("--graph", action="store_true",
                    help="time a HIP-graph replay of the launches instead of eager launches (no host launch floor)")
    ap.add_argument("--ascending", action="store_true",
                    help="Algorithm 1's order of a workgroup's Stream-K pieces instead of the k-aligned default")
    ap.add_argument("--fixup", choices=("flags", "atomic"), default="flags",
                    help="how split tiles are combined (atomic = Algorithm 1's accumulation into C)")
    args = ap.parse_args()
    from paper_2408_11417_amd import inputs
    if args.suite == "model":
        shapes = [size for family in inputs.model_sizes().values() for size in family]
    else:
        shapes = inputs.paper_suite(args.shapes, args.seed) if args.suite == "paper" else inputs.sweep_shapes(args.shapes, args.seed)
    if args.first:
        shapes = shapes[:args.first]
    if args.skinny:
        shapes += [(M, N, K) for M in (16, 32, 64, 128) for N, K in ((8192, 8192), (4096, 4096), (16384, 4096))]
    tile = tuple(int(v) for v in args.tile.split(",")) if args.tile else None
    run(shapes, args.out, dtype_code={"bf16": 1, "f16": 0, "e4m3": 2}[args.dtype], fixup=1 if args.fixup == "atomic" else 0, tile=tile, dp_first=args.dp_first, ascending=args.ascending,
        tile_order={"default": None, "row_major": 0, "grouped": 1}[args.tile_order], graph=args.graph)
    return 0


if __name__ == "__main__":
    sys.exit(main())
