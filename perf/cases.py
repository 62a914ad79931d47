"""Representative calls of the library, for timing and for comparing outputs.

Each case is one thing that a program using the library does over and over:
a training step of the attention, of the layer or of a whole block, a
ranking pass over candidates with and without cached histories, the linear
maps, the Stochastic Length sampler and the standalone time bucketisation.
A case is a dict of plain values; sequence lengths follow from the case
alone, the values of every input from the seed.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2402_17152_amd import hstu

TIME_ORIGIN = 1_700_000_000
GAP_MEAN_S = 600.0
RAB_STD = 0.02
LN_EPS = 1e-5
TIME_BUCKETS = 128
MAX_FLOPS = 4.0e11      # cost bound of a drawn case, below the largest listed one
MAX_BYTES = 4.0e8       # the same for the cases that only move data


def listed():
    """The calls in use, smallest to largest of each kind."""
    return [
        # The encoder's long histories: attention forward and backward at
        # length 8192 (the benchmark's default workload).
        {"name": "attn_step_8k", "op": "attn_step", "dtype": "bf16", "batch": 8, "dist": "uniform",
         "lo": 4096, "hi": 8192, "max_len": 8192, "heads": 4, "d_qk": 128, "d_v": 128,
         "targets": 0},
        # Attention of a batch of mostly short histories, inference only.
        {"name": "attn_fwd_short", "op": "attn_fwd", "dtype": "bf16", "batch": 32,
         "dist": "loguniform", "lo": 8, "hi": 1024, "max_len": 1024, "heads": 4, "d_qk": 64,
         "d_v": 64, "targets": 0},
        # One encoder layer of the training shape: skewed lengths up to 4096,
        # eight heads of 64, with the layer-norm gate, forward and backward.
        {"name": "layer_step_4k", "op": "layer_step", "dtype": "bf16", "batch": 64,
         "dist": "loguniform", "lo": 64, "hi": 4096, "max_len": 4096, "heads": 8, "d_qk": 64,
         "d_v": 64, "targets": 0},
        # The same layer with wide heads.
        {"name": "layer_step_wide", "op": "layer_step", "dtype": "bf16", "batch": 32,
         "dist": "loguniform", "lo": 64, "hi": 2048, "max_len": 2048, "heads": 4, "d_qk": 128,
         "d_v": 128, "targets": 0},
        # Ranking without a cache: histories and candidates in one
        # target-aware forward pass.
        {"name": "rank_full", "op": "attn_fwd", "dtype": "bf16", "batch": 16, "dist": "uniform",
         "lo": 3072, "hi": 3072, "max_len": 3072, "heads": 4, "d_qk": 128, "d_v": 128,
         "targets": 1024},
        # Ranking with cached histories: one microbatch of candidates.
        {"name": "rank_cached", "op": "cached", "dtype": "bf16", "batch": 16, "dist": "uniform",
         "lo": 1024, "hi": 2048, "max_len": 3072, "heads": 4, "d_qk": 128, "d_v": 128,
         "cand_lo": 64, "cand_hi": 64},
        # A whole block, x to x_next and back, on the short histories of
        # public recommendation data.
        {"name": "block_step_200", "op": "block_step", "dtype": "bf16", "batch": 64,
         "dist": "loguniform", "lo": 20, "hi": 200, "max_len": 200, "heads": 4, "d_qk": 64,
         "d_v": 64, "targets": 0, "d_model": 256},
        # The two linear maps at the training shape, forward and backward.
        {"name": "proj_fwd_60k", "op": "proj_fwd", "dtype": "bf16", "tokens": 60383,
         "d_model": 512, "heads": 8, "d_qk": 64, "d_v": 64},
        {"name": "proj_bwd_60k", "op": "proj_bwd", "dtype": "bf16", "tokens": 60383,
         "d_model": 512, "heads": 8, "d_qk": 64, "d_v": 64},
        # The smallest training step, in fp32: launches and latency count.
        {"name": "layer_step_fp32", "op": "layer_step", "dtype": "f32", "batch": 4,
         "dist": "uniform", "lo": 16, "hi": 128, "max_len": 128, "heads": 2, "d_qk": 32,
         "d_v": 32, "targets": 0},
        # Stochastic Length before a training step: sampling and the
        # gathers of the layer's inputs.
        {"name": "stochastic_length", "op": "sl", "batch": 64, "dist": "loguniform", "lo": 64,
         "hi": 4096, "max_len": 4096, "heads": 8, "d_qk": 64, "d_v": 64, "alpha": 1.6,
         "selection": "random"},
        # The bucket matrices of a batch of long histories.
        {"name": "bucketize_8k", "op": "bucketize", "batch": 8, "dist": "uniform", "lo": 4096,
         "hi": 8192, "max_len": 8192},
    ]


# ------------------------------------------------------------------ shapes

def _lengths(case):
    """Sequence lengths of a case: the same for every seed of its inputs."""
    rng = random.Random(f"{case['op']}/{case['batch']}/{case['lo']}/{case['hi']}")
    lo, hi = case["lo"], case["hi"]
    if case["dist"] == "uniform":
        return [rng.randint(lo, hi) for _ in range(case["batch"])]
    return [min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))
            for _ in range(case["batch"])]


def _targets(case, lengths):
    """Candidates per sequence, at most half of it."""
    return [min(case["targets"], n // 2) for n in lengths]


def _candidates(case):
    rng = random.Random(f"cand/{case['batch']}/{case['cand_lo']}/{case['cand_hi']}")
    return [rng.randint(case["cand_lo"], case["cand_hi"]) for _ in range(case["batch"])]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _shrink(case):
    """Halves the batch (or the tokens) until the case costs no more than
    the listed ones."""
    key = "tokens" if "tokens" in case else "batch"
    while case[key] > 1:
        w = work(case)
        light = case["op"] in ("sl", "bucketize")
        if w["bytes"] <= (MAX_BYTES if light else 2e9) and w["flops"] <= MAX_FLOPS:
            break
        case[key] //= 2
    return case


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    op = rng.choice(["attn_step", "attn_step", "attn_fwd", "attn_fwd", "layer_step", "layer_step",
                     "cached", "block_step", "proj_fwd", "proj_bwd", "sl", "bucketize",
                     "layer_step_f32", "attn_step_f32"])
    heads, d_qk, d_v = rng.choice([1, 2, 4, 8]), rng.choice([32, 64, 128]), 0
    d_v = d_qk if rng.random() < 0.7 else rng.choice([32, 64, 128])
    if op.endswith("_f32"):
        hi = _log_int(rng, 16, 384)
        return {"op": op[:-4], "dtype": "f32", "batch": _log_int(rng, 1, 8), "dist": "uniform",
                "lo": rng.randint(1, hi), "hi": hi, "max_len": hi + rng.randint(0, 16),
                "heads": rng.choice([1, 2, 4]), "d_qk": rng.choice([32, 64]),
                "d_v": rng.choice([32, 64]), "targets": rng.choice([0, 0, rng.randint(1, 32)])}
    if op in ("proj_fwd", "proj_bwd"):
        heads = max(heads, 64 // min(d_qk, d_v))
        return _shrink({"op": op, "dtype": "bf16", "tokens": _log_int(rng, 64, 65536),
                        "d_model": 64 * rng.randint(1, 16), "heads": heads, "d_qk": d_qk,
                        "d_v": d_v})
    if op == "cached":
        hi = _log_int(rng, 64, 4096)
        cand = _log_int(rng, 1, 1024)
        return _shrink({"op": op, "dtype": "bf16", "batch": _log_int(rng, 1, 64),
                        "dist": "uniform", "lo": max(1, hi // rng.randint(1, 8)), "hi": hi,
                        "max_len": hi + cand, "heads": heads, "d_qk": d_qk, "d_v": d_v,
                        "cand_lo": rng.randint(1, cand), "cand_hi": cand})
    hi = _log_int(rng, 64, 512 if op == "block_step" else 8192)
    case = {"op": op, "dtype": "bf16", "batch": _log_int(rng, 1, 64),
            "dist": rng.choice(["uniform", "loguniform"]), "lo": max(1, hi // rng.randint(1, 64)),
            "hi": hi, "max_len": hi + rng.randint(0, 64), "heads": heads, "d_qk": d_qk,
            "d_v": d_v, "targets": rng.choice([0, 0, _log_int(rng, 1, max(1, hi // 2))])}
    if op == "block_step":
        case["heads"] = max(heads, 64 // min(d_qk, d_v))
        case["d_model"] = 64 * rng.randint(1, 8)
    elif op == "sl":
        del case["targets"]
        case["alpha"] = round(rng.uniform(1.5, 1.9), 2)
        case["selection"] = rng.choice(["greedy", "random", "weighted"])
    elif op == "bucketize":
        for k in ("targets", "heads", "d_qk", "d_v", "dtype"):
            del case[k]
    return _shrink(case)


def _sl_parameters(case):
    L = int(math.floor(case["max_len"] ** (case["alpha"] / 2.0) + 1e-9))
    return L, float(case["max_len"]) ** case["alpha"]


def work(case):
    """Bytes (each input read once, each output written once) and flops
    (contractions of the pairs that the mask keeps) of one pass."""
    op = case["op"]
    e = 4 if case.get("dtype") == "f32" else 2
    if op in ("proj_fwd", "proj_bwd"):
        T, D = case["tokens"], case["d_model"]
        hv = case["heads"] * case["d_v"]
        F = 2 * hv + 2 * case["heads"] * case["d_qk"]
        weights = F * D + D * hv
        if op == "proj_fwd":   # x, residual, g in; z, z_pre, y out
            return {"bytes": 2 * (T * (3 * D + 2 * F + hv) + weights), "flops": 2 * T * weights}
        # dy, g, x, z_pre, dz, residual gradient in; dg, dx out; fp32 weight gradients out
        return {"bytes": 2 * T * (2 * hv + 4 * D + 2 * F) + 6 * weights,
                "flops": 4 * T * weights}
    lengths = _lengths(case)
    T = sum(lengths)
    if op == "bucketize":
        return {"bytes": sum(n * n for n in lengths) + 8 * T, "flops": 0}
    h, dqk, dv = case["heads"], case["d_qk"], case["d_v"]
    if op == "sl":
        L, num = _sl_parameters(case)
        kept = 0.0
        for n in lengths:
            p = 1.0 if n <= L else min(1.0, num / (n * n))
            kept += p * n + (1.0 - p) * L
        row = 4 * h * (dqk + dv) + 8
        return {"bytes": int(16 * T + kept * (2 * row + 16)), "flops": 0}
    if op == "cached":
        cand = _candidates(case)
        pairs = h * sum(c * (n + 1) for c, n in zip(cand, lengths))
        return {"bytes": 2 * h * (T * (dqk + dv) + 2 * sum(cand) * (dqk + dv)) +
                8 * (T + sum(cand)), "flops": 2 * pairs * (dqk + dv)}
    nts = _targets(case, lengths)
    pairs = h * sum((n - t) * (n - t + 1) // 2 + t * (n - t + 1) for n, t in zip(lengths, nts))
    fwd, bwd = 2 * pairs * (dqk + dv), 2 * pairs * (3 * dqk + 2 * dv)
    side = 8 * T + 4 * (2 * case["max_len"] - 1)
    if op == "attn_fwd":
        return {"bytes": e * T * h * (2 * dqk + 2 * dv) + side, "flops": fwd}
    if op == "attn_step":   # q, k, v, d_out in; out, dq, dk, dv out
        return {"bytes": e * T * h * (4 * dqk + 4 * dv) + 2 * side, "flops": fwd + bwd}
    # q, k, v, u, d_y in; y, dq, dk, dv, du and the fp32 attention output out
    layer = e * T * h * (4 * dqk + 6 * dv) + 4 * T * h * dv + 2 * side
    if op == "layer_step":
        return {"bytes": layer, "flops": fwd + bwd}
    D, hv = case["d_model"], h * dv
    weights = (2 * hv + 2 * h * dqk) * D + D * hv
    return {"bytes": layer + e * T * 4 * D + (e + 4) * weights,
            "flops": fwd + bwd + 6 * T * weights}


# ------------------------------------------------------------------ inputs

class _Inputs:
    """Seeded device arrays."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = torch.float32 if dtype == "f32" else torch.bfloat16

    def normal(self, *shape, std=1.0, dtype=torch.float32):
        return (torch.randn(*shape, generator=self.g, device="cuda") * std).to(dtype)

    def activations(self, *shape):
        """Values as the SiLU projection yields them."""
        return torch.nn.functional.silu(self.normal(*shape)).to(self.dtype)

    def timestamps(self, lengths, start=None):
        """Whole seconds, non-decreasing inside a sequence."""
        T = sum(lengths)
        gaps = torch.empty(T, device="cuda", dtype=torch.float64)
        gaps.exponential_(1.0 / GAP_MEAN_S, generator=self.g)
        total = torch.cumsum(gaps.floor().to(torch.int64), 0)
        first = _offsets(lengths)[:-1].clamp_(max=max(T - 1, 0))
        base = torch.repeat_interleave(total[first], _device(lengths))
        return total - base + (TIME_ORIGIN if start is None
                               else torch.repeat_interleave(start, _device(lengths)))

    def tables(self, max_len):
        return (self.normal(2 * max_len - 1, std=RAB_STD),
                self.normal(TIME_BUCKETS, std=RAB_STD))


def _device(xs):
    return torch.tensor(xs, dtype=torch.int64, device="cuda")


def _split(z, h, d_qk, d_v):
    """U, V, Q, K as [T, h, d] views of the fused projection output."""
    hv, hq = h * d_v, h * d_qk
    return (z[:, :hv].unflatten(1, (h, d_v)), z[:, hv:2 * hv].unflatten(1, (h, d_v)),
            z[:, 2 * hv:2 * hv + hq].unflatten(1, (h, d_qk)),
            z[:, 2 * hv + hq:].unflatten(1, (h, d_qk)))


def _offsets(lengths):
    out = [0]
    for n in lengths:
        out.append(out[-1] + n)
    return _device(out)


def _inputs(case, seed):
    """Every input of a case, and nothing of the library."""
    op = case["op"]
    r = _Inputs(seed, case.get("dtype", "bf16"))
    s = {}
    h, dqk, dv = case.get("heads"), case.get("d_qk"), case.get("d_v")
    if op in ("proj_fwd", "proj_bwd", "block_step"):
        D, hv = case["d_model"], h * dv
        F = 2 * hv + 2 * h * dqk
        s["w1"] = r.normal(F, D, std=D ** -0.5, dtype=r.dtype)
        s["b1"] = r.normal(F, std=0.1)
        s["w2"] = r.normal(D, hv, std=hv ** -0.5, dtype=r.dtype)
        s["b2"] = r.normal(D, std=0.1)
    if op in ("proj_fwd", "proj_bwd"):
        T = case["tokens"]
        s["x"], s["g"] = r.normal(T, D, dtype=r.dtype), r.normal(T, hv, dtype=r.dtype)
        if op == "proj_bwd":
            s["dy"] = r.normal(T, D, dtype=r.dtype)
            s["z_pre"] = r.normal(T, F, dtype=r.dtype)
            s["dz"] = [r.normal(T, h, d, dtype=r.dtype) for d in (dv, dv, dqk, dqk)]
        return s
    lengths = _lengths(case)
    T = sum(lengths)
    s["seq_offsets"], s["timestamps"] = _offsets(lengths), r.timestamps(lengths)
    if op == "bucketize":
        return s
    if op == "sl":
        s["u_keep"] = torch.rand(len(lengths), generator=r.g, device="cuda", dtype=torch.float64)
        s["e_rand"] = torch.empty(T, device="cuda", dtype=torch.float64)
        s["e_rand"].exponential_(generator=r.g)
        for name, d in (("q", dqk), ("k", dqk), ("v", dv), ("u", dv)):
            s[name] = r.activations(T, h, d)
        return s
    s["rab_pos"], s["rab_time"] = r.tables(case["max_len"])
    if op == "cached":
        cand = _candidates(case)
        last = s["timestamps"][s["seq_offsets"][1:] - 1]
        s["cand_offsets"], s["cand_ts"] = _offsets(cand), r.timestamps(cand, start=last + 60)
        s["k_cache"], s["v_cache"] = r.activations(T, h, dqk), r.activations(T, h, dv)
        C = sum(cand)
        s["q"], s["k"] = r.activations(C, h, dqk), r.activations(C, h, dqk)
        s["v"] = r.activations(C, h, dv)
        return s
    nts = _targets(case, lengths)
    s["num_targets"] = _device(nts) if case["targets"] else None
    if op in ("layer_step", "block_step"):
        s["ln_weight"] = 1.0 + r.normal(h * dv, std=0.1)
        s["ln_bias"] = r.normal(h * dv, std=0.1)
    if op == "block_step":
        s["x"], s["dy"] = r.normal(T, D, dtype=r.dtype), r.normal(T, D, dtype=r.dtype)
        return s
    if op == "layer_step":   # views of the fused projection output, as a layer has them
        z = r.activations(T, 2 * h * (dqk + dv))
        s["u"], s["v"], s["q"], s["k"] = _split(z, h, dqk, dv)
        s["d_y"] = r.normal(T, h * dv, dtype=r.dtype)
        return s
    s["q"], s["k"] = r.activations(T, h, dqk), r.activations(T, h, dqk)
    s["v"] = r.activations(T, h, dv)
    if op == "attn_step":
        s["d_out"] = r.normal(T, h, dv, dtype=r.dtype)
    return s


def prepare(case, seed):
    """The inputs and what a program keeps between calls: workspaces, and
    the output buffers of the inference calls and of the sampler."""
    s = _inputs(case, seed)
    op = case["op"]
    s["case"] = case
    h, dqk, dv = case.get("heads"), case.get("d_qk"), case.get("d_v")
    if op in ("attn_step", "attn_fwd", "layer_step", "block_step"):
        dtype = hstu.HSTU_F32 if case["dtype"] == "f32" else hstu.HSTU_BF16
        s["ws"] = hstu.workspace(hstu.make_problem(
            case["batch"], s["timestamps"].numel(), case["max_len"], h, dqk, dv, TIME_BUCKETS,
            dtype))
    if op in ("proj_fwd", "proj_bwd", "block_step"):
        s["proj_ws"] = hstu.proj_workspace(hstu.proj_problem(s["x"], h, dqk, dv), case["d_model"])
    if op == "attn_fwd":
        s["out"] = torch.empty_like(s["v"])
    elif op == "cached":
        s["out"] = torch.empty_like(s["v"])
        s["ws"] = hstu.cached_workspace(hstu.problem_for(
            s["q"], s["v"], s["cand_offsets"], case["max_len"], s["rab_time"]))
    elif op == "sl":
        s["subseq_len"] = hstu.hstu_sl_subseq_len(case["max_len"], case["alpha"])
        s["keep_numerator"] = hstu.hstu_sl_keep_numerator(case["max_len"], case["alpha"])
        s["mode"] = {"greedy": hstu.HSTU_SL_GREEDY, "random": hstu.HSTU_SL_RANDOM,
                     "weighted": hstu.HSTU_SL_WEIGHTED}[case["selection"]]
        s["ws"] = torch.empty(hstu.hstu_sl_workspace_bytes(case["batch"]), dtype=torch.uint8,
                              device="cuda")
        # Buffers of the full batch's size; rows past the kept tokens are not written.
        T = s["timestamps"].numel()
        s["out"] = (torch.zeros_like(s["seq_offsets"]),
                    torch.zeros(T, dtype=torch.int64, device="cuda"))
        s["kept"] = {n: torch.zeros_like(s[n]) for n in ("q", "k", "v", "u", "timestamps")}
    elif op == "bucketize":
        s["total_pairs"] = sum(n * n for n in _lengths(case))
        s["pair_offsets"] = hstu.hstu_pair_offsets(s["seq_offsets"])
        s["out"] = torch.empty(s["total_pairs"], dtype=torch.uint8, device="cuda")
    return s


# ------------------------------------------------------------------- passes

def run(s):
    """One pass through the public entry points."""
    return _RUN[s["case"]["op"]](s)


def _bias_args(s):
    return (s["seq_offsets"], s["timestamps"], s["rab_pos"], s["rab_time"], s["case"]["max_len"])


def _attn_fwd(s):
    return hstu.hstu_attn_fwd(s["q"], s["k"], s["v"], *_bias_args(s),
                              num_targets=s["num_targets"], out=s["out"], ws=s["ws"])


def _attn_step(s):
    out = hstu.hstu_attn_fwd(s["q"], s["k"], s["v"], *_bias_args(s),
                             num_targets=s["num_targets"], ws=s["ws"])
    grads = hstu.hstu_attn_bwd(s["q"], s["k"], s["v"], s["d_out"], *_bias_args(s),
                               num_targets=s["num_targets"], ws=s["ws"])
    return (out, *grads)


def _layer_fwd_bwd(s, u, v, q, k, d_y_of):
    kw = {"num_targets": s["num_targets"], "ln_weight": s["ln_weight"], "ln_bias": s["ln_bias"],
          "ws": s["ws"]}
    attn_out, y, mean, rstd = hstu.hstu_layer_fwd(q, k, v, u, *_bias_args(s), ln_eps=LN_EPS, **kw)
    grads = hstu.hstu_layer_bwd(q, k, v, u, attn_out, mean, rstd, d_y_of(y), *_bias_args(s), **kw)
    return y, grads


def _layer_step(s):
    y, grads = _layer_fwd_bwd(s, s["u"], s["v"], s["q"], s["k"], lambda y: s["d_y"])
    return (y, *grads)


def _block_step(s):
    c = s["case"]
    dims = (c["heads"], c["d_qk"], c["d_v"])
    z, z_pre = hstu.hstu_proj_in_fwd(s["x"], s["w1"], s["b1"], *dims)
    outer = {}

    def d_gated(y):
        outer["x_next"] = hstu.hstu_proj_out_fwd(y, s["w2"], s["b2"], s["x"], *dims)
        dg, outer["dw2"], outer["db2"] = hstu.hstu_proj_out_bwd(y, s["w2"], s["dy"], *dims,
                                                                ws=s["proj_ws"])
        return dg

    _, grads = _layer_fwd_bwd(s, *hstu.split_uvqk(z, *dims), d_gated)
    dq, dk, dv, du, dlw, dlb, drp, drt = grads
    dx, dw1, db1 = hstu.hstu_proj_in_bwd(s["x"], s["w1"], z_pre, du, dv, dq, dk, *dims,
                                         dx_add=s["dy"], ws=s["proj_ws"])
    return (outer["x_next"], dx, dw1, db1, outer["dw2"], outer["db2"], dlw, dlb, drp, drt)


def _cached(s):
    return hstu.hstu_attn_fwd_cached(
        s["q"], s["k"], s["v"], s["cand_offsets"], s["cand_ts"], s["k_cache"], s["v_cache"],
        s["seq_offsets"], s["timestamps"], s["rab_pos"], s["rab_time"], s["case"]["max_len"],
        out=s["out"], ws=s["ws"])


def _proj_fwd(s):
    c = s["case"]
    dims = (c["heads"], c["d_qk"], c["d_v"])
    z, z_pre = hstu.hstu_proj_in_fwd(s["x"], s["w1"], s["b1"], *dims)
    y = hstu.hstu_proj_out_fwd(s["g"], s["w2"], s["b2"], s["x"], *dims)
    return z, z_pre, y


def _proj_bwd(s):
    c = s["case"]
    dims = (c["heads"], c["d_qk"], c["d_v"])
    dg, dw2, db2 = hstu.hstu_proj_out_bwd(s["g"], s["w2"], s["dy"], *dims, ws=s["proj_ws"])
    dx, dw1, db1 = hstu.hstu_proj_in_bwd(s["x"], s["w1"], s["z_pre"], *s["dz"], *dims,
                                         dx_add=s["dy"], ws=s["proj_ws"])
    return dg, dw2, db2, dx, dw1, db1


def _sl(s):
    offs, gather = hstu.hstu_stochastic_length(
        s["seq_offsets"], s["timestamps"], s["subseq_len"], s["keep_numerator"], s["mode"],
        s["u_keep"], s["e_rand"], out=s["out"], ws=s["ws"])
    for n, dst in s["kept"].items():
        hstu.hstu_gather_rows(s[n], gather, offs[-1:], dst=dst)
    return (offs, gather, *s["kept"].values())


def _bucketize(s):
    return hstu.hstu_time_bucketize(s["seq_offsets"], s["timestamps"], TIME_BUCKETS,
                                    pair_offsets=s["pair_offsets"],
                                    total_pairs=s["total_pairs"], out=s["out"])


_RUN = {"attn_fwd": _attn_fwd, "attn_step": _attn_step, "layer_step": _layer_step,
        "block_step": _block_step, "cached": _cached, "proj_fwd": _proj_fwd,
        "proj_bwd": _proj_bwd, "sl": _sl, "bucketize": _bucketize}


def tolerance(case):
    """About four times the largest distance from 64-bit arithmetic, in
    2-norm, that any output showed over the listed and 40 drawn cases: 6.6e-7
    in fp32; 2.4e-3 in bf16 (1.7e-3 of it the rounding of the output), and
    6e-3 for a whole block, whose z, g and their gradients are rounded to
    bf16 on the way."""
    if case["op"] in ("sl", "bucketize"):
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 3e-6}
    return {"rel": 2.4e-2 if case["op"] == "block_step" else 1e-2}


# ---------------------------------------------------- the same in 64 bits

def _buckets64(dt):
    """floor(log2(max(|dt|, 1))), clamped (differences are below 2^53)."""
    x = dt.abs().clamp_(min=1).to(torch.float64)
    return (torch.frexp(x).exponent - 1).clamp_(max=TIME_BUCKETS - 1)


def _attention64(case, s, q, k, v, d_out=None):
    """Attention output [T, h, dv] and, for d_out, its gradients."""
    h, N = case["heads"], case["max_len"]
    lengths = _lengths(case)
    nts = _targets(case, lengths)
    f8 = {"dtype": torch.float64, "device": "cuda"}
    out = torch.zeros(v.shape, **f8)
    rp, rt = s["rab_pos"].double(), s["rab_time"].double()
    if d_out is not None:
        dq, dk, dv = (torch.zeros(t.shape, **f8) for t in (q, k, v))
        drp, drt = torch.zeros(2 * N - 1, **f8), torch.zeros(TIME_BUCKETS, **f8)
    o = 0
    for n, t in zip(lengths, nts):
        nh = n - t
        i = torch.arange(n, device="cuda")
        p = i.clamp(max=nh)
        ts = s["timestamps"][o:o + n]
        bkt = _buckets64(ts[:, None] - ts[None, :])
        bias = rp[(N - 1) + p[None, :] - p[:, None]] + rt[bkt.long()]
        keep = (i[None, :] <= i[:, None]) & ((i[None, :] < nh) | (i[None, :] == i[:, None]))
        total = None
        for a in range(h):
            qa, ka, va = (x[o:o + n, a].double() for x in (q, k, v))
            sc = qa @ ka.t() + bias
            sg = torch.sigmoid(sc)
            w = torch.where(keep, sc * sg, 0.0) / N
            out[o:o + n, a] = w @ va
            if d_out is None:
                continue
            ga = d_out[o:o + n, a].double()
            dv[o:o + n, a] = w.t() @ ga
            ds = torch.where(keep, (ga @ va.t()) * sg * (1.0 + sc * (1.0 - sg)), 0.0) / N
            dq[o:o + n, a] = ds @ ka
            dk[o:o + n, a] = ds.t() @ qa
            total = ds if total is None else total + ds
        if d_out is not None:
            for b in torch.unique(bkt).tolist():
                drt[b] += torch.where(bkt == b, total, 0.0).sum()
            # Candidates share position nh: their rows fold into one.
            m = nh + (1 if t else 0)
            if t:
                fold = torch.zeros(m, m, **f8)
                fold[:nh, :nh] = total[:nh, :nh]
                fold[nh, :nh] = total[nh:, :nh].sum(0)
                fold[nh, nh] = torch.diagonal(total[nh:, nh:]).sum()
                total = fold
            # Row i shifted by -i: one column per offset p(j) - p(i).
            skew = torch.zeros(m * (2 * m - 1), **f8)
            skew.as_strided((m, m), (max(2 * m - 2, 1), 1), m - 1).copy_(total)
            drp[N - m:N - m + 2 * m - 1] += skew.view(m, 2 * m - 1).sum(0)
        o += n
    return out if d_out is None else (out, dq, dk, dv, drp, drt)


def _layer64(case, s, u, v, q, k, d_y):
    """y and the layer's gradients, in the order of hstu_layer_bwd; d_y is a
    tensor or a function of y."""
    x = _attention64(case, s, q, k, v).flatten(1)
    T = x.shape[0]
    g, b, uu = s["ln_weight"].double(), s["ln_bias"].double(), u.reshape(T, -1).double()
    rstd = 1.0 / torch.sqrt(x.var(1, unbiased=False, keepdim=True) + LN_EPS)
    z = (x - x.mean(1, keepdim=True)) * rstd
    y = (z * g + b) * uu
    dy = (d_y(y) if callable(d_y) else d_y).double()
    du, dn = (z * g + b) * dy, dy * uu
    dlw, dlb = (dn * z).sum(0), dn.sum(0)
    dz = dn * g
    d_out = rstd * (dz - dz.mean(1, keepdim=True) - z * (dz * z).mean(1, keepdim=True))
    _, dq, dk, dv, drp, drt = _attention64(case, s, q, k, v, d_out.view(T, case["heads"], -1))
    return y, dq, dk, dv, du, dlw, dlb, drp, drt


def _block64(case, s):
    h, dqk, dv = case["heads"], case["d_qk"], case["d_v"]
    x, w1, w2, dy = (s[n].double() for n in ("x", "w1", "w2", "dy"))
    pre = x @ w1.t() + s["b1"].double()
    z = torch.nn.functional.silu(pre)
    keep = {}

    def d_gated(y):
        keep["x_next"] = y @ w2.t() + s["b2"].double() + x
        keep["dw2"] = dy.t() @ y
        return dy @ w2

    _, dq, dk, dv_, du, dlw, dlb, drp, drt = _layer64(
        case, s, *_split(z, h, dqk, dv), d_gated)
    dz = torch.cat([t.reshape(x.shape[0], -1) for t in (du, dv_, dq, dk)], 1)
    sg = torch.sigmoid(pre)
    dpre = dz * sg * (1.0 + pre * (1.0 - sg))
    return (keep["x_next"], dpre @ w1 + dy, dpre.t() @ x, dpre.sum(0), keep["dw2"], dy.sum(0),
            dlw, dlb, drp, drt)


def _cached64(case, s):
    N, h = case["max_len"], case["heads"]
    out = torch.zeros(s["v"].shape, dtype=torch.float64, device="cuda")
    rp, rt = s["rab_pos"].double(), s["rab_time"].double()
    o = c0 = 0
    for n, c in zip(_lengths(case), _candidates(case)):
        p = torch.arange(n, device="cuda")
        dt = s["cand_ts"][c0:c0 + c][:, None] - s["timestamps"][o:o + n][None, :]
        bias = rp[(N - 1) + p - n] + rt[_buckets64(dt).long()]
        for a in range(h):
            q, k, v = (s[x][c0:c0 + c, a].double() for x in ("q", "k", "v"))
            sc = q @ s["k_cache"][o:o + n, a].double().t() + bias
            own = (q * k).sum(1, keepdim=True) + rp[N - 1] + rt[0]
            out[c0:c0 + c, a] = (torch.nn.functional.silu(sc) @ s["v_cache"][o:o + n, a].double() +
                                 torch.nn.functional.silu(own) * v) / N
        o, c0 = o + n, c0 + c
    return out


def _proj64(case, s):
    x, g, w1, w2 = (s[n].double() for n in ("x", "g", "w1", "w2"))
    if case["op"] == "proj_fwd":
        pre = x @ w1.t() + s["b1"].double()
        return torch.nn.functional.silu(pre), pre, g @ w2.t() + s["b2"].double() + x
    dy, pre = s["dy"].double(), s["z_pre"].double()
    sg = torch.sigmoid(pre)
    dpre = torch.cat([t.flatten(1) for t in s["dz"]], 1).double() * sg * (1.0 + pre * (1.0 - sg))
    return dy @ w2, dy.t() @ g, dy.sum(0), dpre @ w1 + dy, dpre.t() @ x, dpre.sum(0)


def _sl64(case, s):
    L, num = _sl_parameters(case)
    u_keep = s["u_keep"].tolist()
    offs, picks, o = [0], [], 0
    for b, n in enumerate(_lengths(case)):
        if n <= L or u_keep[b] < num / (float(n) * float(n)):
            idx = torch.arange(n, device="cuda")
        else:
            ts, e = s["timestamps"][o:o + n], s["e_rand"][o:o + n]
            f = ts.max() - ts
            if case["selection"] == "greedy":
                key = f
            elif case["selection"] == "random" or int(f.sum()) == 0:
                key = e
            else:
                key = e / (f.sum() - f).double()
            # Equal keys: the later token first.
            order = torch.argsort(key.flip(0), stable=True)
            idx = (n - 1 - order[:L]).sort().values
        picks.append(idx + o)
        offs.append(offs[-1] + len(idx))
        o += n
    gather = torch.cat(picks)

    def padded(x):
        return torch.cat([x, x.new_zeros((o - x.shape[0],) + x.shape[1:])])

    return (_device(offs), padded(gather),
            *(padded(s[n][gather]) for n in ("q", "k", "v", "u", "timestamps")))


def _bucketize64(case, s):
    parts, o = [], 0
    for n in _lengths(case):
        ts = s["timestamps"][o:o + n]
        parts.append(_buckets64(ts[:, None] - ts[None, :]).to(torch.uint8).flatten())
        o += n
    return torch.cat(parts)


def exact(case, seed):
    """What run() returns for these inputs, in 64-bit arithmetic."""
    s = _inputs(case, seed)
    op = case["op"]
    if op == "attn_fwd":
        return _attention64(case, s, s["q"], s["k"], s["v"])
    if op == "attn_step":
        return _attention64(case, s, s["q"], s["k"], s["v"], s["d_out"])
    if op == "layer_step":
        return _layer64(case, s, s["u"], s["v"], s["q"], s["k"], s["d_y"])
    if op == "block_step":
        return _block64(case, s)
    if op == "cached":
        return _cached64(case, s)
    if op in ("proj_fwd", "proj_bwd"):
        return _proj64(case, s)
    return _sl64(case, s) if op == "sl" else _bucketize64(case, s)
