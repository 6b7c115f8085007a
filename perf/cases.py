"""The GEMM calls whose speed this library is judged by, and how to make, run and check them.

Each case is one call D = A * B through the public entry points, as the README's program makes it: the
tile and the grid are the library's defaults, the scheduling policy is the one the selector falls back
to when nothing has been tuned (`selector.fallback_policy`), plan and workspace are kept by the caller,
and the launch goes through `sk_gemm_bind`, the form for programs that launch one problem many times.
"""
import math

import torch

import paper_2408_11417_amd as sk
from paper_2408_11417_amd import selector

IN = {"f16": (torch.float16, sk.SK_F16, 2), "bf16": (torch.bfloat16, sk.SK_BF16, 2), "e4m3": (torch.float8_e4m3fn, sk.SK_FP8_E4M3, 1)}
OUT = {"f16": (torch.float16, sk.SK_F16, 2), "bf16": (torch.bfloat16, sk.SK_BF16, 2), "f32": (torch.float32, sk.SK_F32, 4)}

# The most that a drawn case may cost: the largest listed case, 8192^3 in bf16.
MAX_FLOPS = 2.0 * 8192 ** 3
MAX_BYTES = 3 * 8192 * 8192 * 2


def _case(name, M, N, K, dtype="bf16", out="bf16", values="uniform"):
    return {"name": name, "M": M, "N": N, "K": K, "in": dtype, "out": out, "values": values}


def listed():
    return [
        # The smallest configuration the library is benchmarked on: one small fp16 product.  Launch latency and
        # the length of one workgroup's serial chain are all there is.
        _case("f16_512_cubed", 512, 512, 512, "f16", "f16"),
        # One token through one projection (a matrix-vector product, the smallest M of the paper's suite).
        _case("f16_decode_m1", 1, 4096, 4096, "f16", "f16", "weights"),
        # Decode of 16 and 128 tokens against an 8192 x 8192 weight (the skinny configuration's two ends).
        _case("bf16_decode_m16", 16, 8192, 8192, "bf16", "bf16", "weights"),
        _case("bf16_decode_m128", 128, 8192, 8192, "bf16", "bf16", "weights"),
        # The same decode step with 8-bit weights and activations.
        _case("fp8_decode_m64", 64, 8192, 8192, "e4m3", "bf16", "weights"),
        # The middle of the tuning sweep's range (64 .. 16384 in each dimension, multiples of 16): an everyday
        # product that is a fraction of one wave of large tiles.
        _case("bf16_middle", 1008, 1200, 1040),
        # Few tiles, deep K: a weight gradient, or an attention-score product with a long inner dimension,
        # accumulated in and returned as fp32.
        _case("f16_deep_k_f32_out", 256, 512, 16384, "f16", "f32", "normal"),
        # The wave-quantisation configuration: a little less than one wave of the largest tile.
        _case("bf16_wave_quantised", 3840, 4224, 4096, "bf16", "bf16", "normal"),
        # Sizes with no alignment at all (an odd vocabulary, an odd batch).
        _case("bf16_odd_sizes", 3841, 4225, 4097, "bf16", "bf16", "normal"),
        # Wide and shallow: a low-rank or per-head projection whose output is far larger than its inputs.
        _case("bf16_short_k", 8192, 8192, 512),
        # Prefill and training: large squares in 16 and in 8 bits.
        _case("fp8_8192_cubed", 8192, 8192, 8192, "e4m3", "bf16"),
        _case("bf16_8192_cubed", 8192, 8192, 8192),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _multiple(v, step):
    return max(step, (v + step // 2) // step * step)


def draw(rng):
    """One more call of the same ranges."""
    while True:
        kind = rng.choice(["sweep", "sweep", "sweep", "decode", "decode", "odd", "odd", "deep"])
        dtype = rng.choice(["bf16", "bf16", "f16"])
        values = rng.choice(["uniform", "normal"])
        if kind == "sweep":      # config 4's range, 16 and 8 bits
            dtype = rng.choice(["bf16", "f16", "e4m3"])
            M, N, K = (_multiple(_log_uniform(rng, 64, 16384), 16) for _ in range(3))
        elif kind == "decode":   # a few tokens against a weight matrix
            dtype, values = rng.choice(["bf16", "f16", "e4m3"]), "weights"
            M, N, K = rng.randint(1, 128), _multiple(_log_uniform(rng, 1024, 16384), 64), _multiple(_log_uniform(rng, 1024, 16384), 64)
            if N * K > 8192 * 8192:
                continue
        elif kind == "odd":      # any sizes at all
            M, N, K = (_log_uniform(rng, 64, 4400) for _ in range(3))
        else:                    # few tiles, deep K
            M, N, K = _multiple(_log_uniform(rng, 64, 1024), 16), _multiple(_log_uniform(rng, 64, 1024), 16), _multiple(_log_uniform(rng, 8192, 65536), 16)
        out = "bf16" if dtype == "e4m3" else dtype
        if rng.random() < 0.2:
            out = "f32"
        case = {"M": M, "N": N, "K": K, "in": dtype, "out": out, "values": values}
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


def _inputs(case, seed):
    dtype = IN[case["in"]][0]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))

    def matrix(rows, cols):
        if case["values"] == "uniform":
            x = torch.rand((rows, cols), generator=gen, device="cuda") * 2 - 1
        else:
            x = torch.randn((rows, cols), generator=gen, device="cuda")
            # "weights": the small weights of a projection, in 8 bits scaled to the middle of the format as
            # a quantiser would; "normal": unit variance of the result
            sigma = (0.02 if dtype != torch.float8_e4m3fn else 1.0) if case["values"] == "weights" else 1.0 / math.sqrt(case["K"])
            if dtype == torch.float8_e4m3fn and case["values"] == "normal":
                sigma = 1.0
            x = x * sigma
        return x.to(dtype)

    return matrix(case["M"], case["K"]), matrix(case["K"], case["N"])


def prepare(case, seed):
    M, N, K = case["M"], case["N"], case["K"]
    in_dtype, (out_torch, out_dtype, _) = IN[case["in"]][1], OUT[case["out"]]
    A, B = _inputs(case, seed)
    policy = selector.fallback_policy(M, N, K, sk.sk_default_tile(M, N, K, in_dtype), 256, in_dtype)
    plan = sk.sk_plan(M, N, K, policy, in_dtype=in_dtype, out_dtype=out_dtype)
    nbytes = sk.sk_workspace_bytes(plan)
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    sk.sk_plan_set_workspace(plan, (ws.data_ptr() + 255) // 256 * 256, nbytes)
    D = torch.empty((M, N), dtype=out_torch, device="cuda")
    launch = sk.sk_gemm_bind(A.data_ptr(), B.data_ptr(), D.data_ptr(), plan, torch.cuda.current_stream().cuda_stream)
    return State(A, B, D, ws, plan, launch)


class State:
    """Operands, result, workspace and plan of one problem; the plan goes with the object."""

    def __init__(self, A, B, D, ws, plan, launch):
        self.A, self.B, self.D, self.ws, self.plan, self.launch = A, B, D, ws, plan, launch

    def __del__(self):
        if self.plan is not None:
            sk.sk_plan_destroy(self.plan)
            self.plan = None


def run(state):
    status = state.launch()
    if status != sk.SK_OK:
        raise sk.StreamKError(status, "sk_gemm")
    return state.D


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    return {"bytes": (M * K + K * N) * IN[case["in"]][2] + M * N * OUT[case["out"]][2], "flops": 2.0 * M * N * K}


def tolerance(case):
    # Four times what this library's results are off from the 64-bit product (2-norm, and largest difference):
    # the rounding of the output where it is 16 bits wide, the order of the fp32 sums where it is not.
    return {"bf16": {"rel": 7e-3, "max": 1.6e-2}, "f16": {"rel": 9e-4, "max": 2e-3}, "f32": {"rel": 1e-5, "max": 1e-4}}[case["out"]]


def exact(case, seed):
    A, B = _inputs(case, seed)
    return A.double() @ B.double()
