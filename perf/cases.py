"""Timed workloads of the hybrid delta attention library: what a program that uses it asks of it.

A case is a dict of plain values; `kind` names the call it makes:

    prefill   delta_attn_prefill over one batch of prompts
    append    a prompt fed in pieces to delta_attn_prefill_append (the cache is emptied first)
    generate  a prompt into a cache (delta_attn_prefill), then decode steps (delta_attn_decode)
    scan      delta_attn_delta_scan alone, with the reference keys

Shapes are those of the repository's own configurations (C1 .. C5: 32 query / 8 KV heads of 64, 20 / 5 heads of 128),
of its prompt-length sweep with the window of Eq. 5, and ragged sizes in between.  Inputs follow the recipe of
`workloads.py` - an AR(1) walk per channel with whole-vector jumps, a scale per head - drawn on the GPU from the seed.
"""
import math

import torch

from paper_2507_19608_amd import binding as da

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_MODES = {"gather": da.DA_SCORE_GATHER, "rebase": da.DA_SCORE_REBASE}
_WINDOWS = {"block": da.DA_WINDOW_BLOCK, "sliding": da.DA_WINDOW_SLIDING}


def _prefill(name, batch, hq, hkv, d, n, window, theta, p_jump=0.05, dtype="bf16", mode="gather", shape="block",
             kept=True):
    return {"name": name, "kind": "prefill", "batch": batch, "hq": hq, "hkv": hkv, "d": d, "n": n, "window": window,
            "theta": theta, "p_jump": p_jump, "dtype": dtype, "mode": mode, "shape": shape, "kept": kept}


def _generate(name, batch, hq, hkv, d, n, window, theta, steps, decode_window, p_jump=0.05, mode="gather"):
    return {"name": name, "kind": "generate", "batch": batch, "hq": hq, "hkv": hkv, "d": d, "n": n, "window": window,
            "theta": theta, "p_jump": p_jump, "dtype": "bf16", "mode": mode, "shape": "block", "steps": steps,
            "decode_window": decode_window}


def listed():
    return [
        # C1: one fp32 head, a numerics user's call; buffers are left to the binding
        _prefill("prefill_f32_256", 1, 1, 1, 64, 256, 32, 0.05, dtype="f32", kept=False),
        # a chat-sized prompt of odd length, window by Eq. 5, buffers left to the binding: the latency of one call
        _prefill("prefill_333", 1, 32, 8, 64, 333, 16, 0.1113, kept=False),
        # a batch of prompts of a few hundred tokens, the range the method is meant for
        _prefill("prefill_16x200", 16, 20, 5, 128, 200, 10, 0.1113),
        # C2 and C3: one prompt, the two model shapes
        _prefill("prefill_C2", 1, 32, 8, 64, 2048, 128, 0.1074),
        _prefill("prefill_C3_rebase", 1, 20, 5, 128, 4096, 256, 0.0938, mode="rebase"),
        # ragged prompts with the sliding band and bursty keys
        _prefill("prefill_2x5003_sliding", 2, 20, 5, 128, 5003, 250, 0.1562, p_jump=0.2, mode="rebase", shape="sliding"),
        # C5, the headline: four 8K prompts, default score mode
        _prefill("prefill_C5", 4, 20, 5, 128, 8192, 512, 0.1113),
        # two 4K prompts in pieces of 1024, as a server that mixes prefill and decode feeds them
        {"name": "append_2x4096", "kind": "append", "batch": 2, "hq": 20, "hkv": 5, "d": 128, "n": 4096, "piece": 1024,
         "window": 256, "theta": 0.1113, "p_jump": 0.05, "dtype": "bf16", "mode": "gather", "shape": "block"},
        # one user's answer: a short prompt and 64 tokens, where launches and host work count
        _generate("generate_512_64", 1, 32, 8, 64, 512, 32, 0.1133, 64, 128),
        # a few long contexts, each step reads a lot per sequence
        _generate("generate_4x6000_64", 4, 20, 5, 128, 6000, 256, 0.1113, 64, 256, mode="rebase"),
        # C4: a serving batch of 32, 2048 cached tokens and 256 steps
        _generate("generate_C4", 32, 32, 8, 64, 2048, 128, 0.1133, 256, 128),
        # the delta matrix alone (mask, counts and reference keys) of C5's keys
        {"name": "scan_C5", "kind": "scan", "batch": 4, "hq": 5, "hkv": 5, "d": 128, "n": 8192, "theta": 0.1113,
         "p_jump": 0.05, "dtype": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a call, a head shape and log-uniform sizes, cut to what the largest listed case costs."""
    kind = rng.choices(("prefill", "append", "generate", "scan"), (0.5, 0.15, 0.25, 0.1))[0]
    d = rng.choice((64, 128))
    hq, hkv = rng.choice(((32, 8), (20, 5), (8, 8), (12, 6), (16, 2)))
    c = {"kind": kind, "hq": hq, "hkv": hkv, "d": d, "dtype": "bf16", "p_jump": rng.choice((0.01, 0.05, 0.2)),
         "theta": 0.0 if rng.random() < 0.08 else round(rng.uniform(0.05, 0.23), 4)}
    batch = _log_int(rng, 1, 32)
    if kind == "scan":
        c["dtype"] = rng.choice(("bf16", "bf16", "f32"))
        c["hq"] = hkv
        c["n"] = _log_int(rng, 64, 16384)
        c["batch"] = max(1, min(batch, (1 << 25) // (hkv * c["n"] * d)))
        return c
    if kind == "prefill" and rng.random() < 0.12:      # fp32 users: small problems
        c.update(dtype="f32", hq=rng.choice((1, 4, 8)), hkv=1)
        n, batch = _log_int(rng, 64, 1024), min(batch, 2)
    else:
        n = _log_int(rng, 64, 8192)
    if rng.random() < 0.5:                             # half of the lengths are whole tiles, half are not
        n = max(64, n // 64 * 64)
    room = 1.5e11 if kind == "generate" else 5e11      # batch * hq * n^2 * d of C4 and C5, with some margin
    batch = max(1, min(batch, int(room / (c["hq"] * n * n * d))))
    gamma = max(1, min(512, int(0.05 * n)))            # Eq. 5
    window = rng.choice((gamma, 1 << rng.randint(4, 9)))
    c.update(batch=batch, n=n, window=window, mode=rng.choice(("gather", "gather", "rebase")),
             shape=rng.choice(("block", "block", "sliding")))
    if kind == "prefill":
        c["kept"] = rng.random() < 0.6
    elif kind == "append":
        c["window"] = min(window, 512)
        c["piece"] = max(64, _log_int(rng, max(64, n // 8), n))
    else:
        c["shape"] = "block"
        c["steps"] = _log_int(rng, 16, 128)
        # mostly the windows of the configurations; now and then the paper's own handful of tokens
        c["decode_window"] = rng.choice((64, 128, 128, 256, 512, 4))
    return c


def _stream(gen, batch, heads, n, d, p_jump, scaled):
    """x_t = 0.95 x_{t-1} + N(0, 0.1^2), or N(0, I) with probability p_jump (whole vector); scale U(0.5, 2) per head.
    The recurrence x_t = a_t x_{t-1} + b_t (a_t = 0 at a jump) is solved by doubling."""
    dev = "cuda"
    b = torch.randn(batch, heads, n, d, generator=gen, device=dev)
    jump = torch.rand(batch, heads, n, 1, generator=gen, device=dev) < p_jump
    jump[:, :, 0] = False
    b *= torch.where(jump, 1.0, 0.1)
    b[:, :, 0] *= 1.0 / math.sqrt(1.0 - 0.95 ** 2)
    a = torch.where(jump, 0.0, 0.95).to(torch.float32)
    step = 1
    while step < n:
        b = torch.cat((b[:, :, :step], torch.addcmul(b[:, :, step:], a[:, :, step:], b[:, :, :-step])), 2)
        a = torch.cat((a[:, :, :step], a[:, :, step:] * a[:, :, :-step]), 2)
        step *= 2
        if step >= 512:                                # 0.95^512 is below 1e-11: nothing further back is felt
            break
    if scaled:
        b *= 0.5 + 1.5 * torch.rand(batch, heads, 1, 1, generator=gen, device=dev)
    return b


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = _DTYPES[c["dtype"]]
    total = c["n"] + c.get("steps", 0)

    def tensor(heads):
        return _stream(gen, c["batch"], heads, total, c["d"], c["p_jump"], c["dtype"] == "bf16").to(dt)

    s = {"case": dict(c)}
    K = tensor(c["hkv"])
    if c["kind"] == "scan":
        s["K"] = K.contiguous()
        return s
    V, Q = tensor(c["hkv"]), tensor(c["hq"])
    n = c["n"]
    if c["kind"] == "append":
        cuts = list(range(0, n, c["piece"])) + [n]
        s["pieces"] = [tuple(t[:, :, i:j].contiguous() for t in (Q, K, V)) for i, j in zip(cuts, cuts[1:])]
        s["cache"] = da.Cache(c["batch"], c["hq"], c["hkv"], c["d"], n, max(c["window"], 128), c["theta"], dt)
        return s
    s["QKV"] = tuple(t[:, :, :n].contiguous() for t in (Q, K, V))
    # what a program that calls this more than once keeps: results and scratch
    if c["kind"] == "generate" or c["kept"]:
        q, k, _ = s["QKV"]
        p = da.make_params(q, k, c["window"], c["theta"], 0.0, _MODES[c["mode"]], _WINDOWS[c["shape"]])
        s["workspace"] = torch.empty(max(1, da.delta_attn_prefill_workspace_bytes(p)), dtype=torch.uint8, device="cuda")
        s["out"] = (torch.empty_like(q),
                    torch.empty(c["batch"], c["hkv"], n, c["d"] // 32, dtype=torch.int32, device="cuda"),
                    torch.empty(c["batch"], c["hkv"], dtype=torch.int64, device="cuda"))
    if c["kind"] == "generate":
        s["cache"] = da.Cache(c["batch"], c["hq"], c["hkv"], c["d"], total, c["decode_window"], c["theta"], dt)
        s["tokens"] = [tuple(t[:, :, i].contiguous() for t in (Q, K, V)) for i in range(n, total)]
        s["o"] = torch.empty(c["steps"], c["batch"], c["hq"], c["d"], dtype=dt, device="cuda")
        s["mask_rows"] = torch.empty(c["steps"], c["batch"], c["hkv"], c["d"] // 32, dtype=torch.int32, device="cuda")
        s["slots"] = list(zip(s["o"].unbind(0), s["mask_rows"].unbind(0)))
    return s


def run(state):
    s = state
    c = s["case"]
    if c["kind"] == "scan":
        return da.delta_attn_delta_scan(s["K"], c["theta"], want_khat=True)
    opts = {"score_mode": _MODES[c["mode"]], "window_mode": _WINDOWS[c["shape"]]}
    if c["kind"] == "append":
        s["cache"].reset()
        return [da.delta_attn_prefill_append(s["cache"], q, k, v, c["theta"], c["window"], **opts)
                for q, k, v in s["pieces"]]
    q, k, v = s["QKV"]
    if c["kind"] == "prefill":
        if not c["kept"]:
            return da.delta_attn_prefill(q, k, v, c["theta"], c["window"], **opts)
        return da.delta_attn_prefill(q, k, v, c["theta"], c["window"], workspace=s["workspace"], out=s["out"], **opts)
    s["cache"].reset()
    da.delta_attn_prefill(q, k, v, c["theta"], c["window"], cache=s["cache"], workspace=s["workspace"], out=s["out"],
                          **opts)
    for (q1, k1, v1), (o, row) in zip(s["tokens"], s["slots"]):
        da.delta_attn_decode(s["cache"], q1, k1, v1, out=o, mask_row=row)
    return s["out"], s["o"], s["mask_rows"]


def _kept_fraction(theta):
    """Share of delta entries that survive, from the thresholds tuned for the configurations (5 % jumps)."""
    points = ((0.0, 1.0), (0.0625, 0.59), (0.1113, 0.40), (0.2227, 0.20))
    for (t0, r0), (t1, r1) in zip(points, points[1:]):
        if theta <= t1:
            return r0 + (r1 - r0) * (theta - t0) / (t1 - t0)
    return points[-1][1]


def work(case):
    c = case
    b, hkv, d, n = c["batch"], c["hkv"], c["d"], c["n"]
    es = 2 if c["dtype"] == "bf16" else 4
    kept = _kept_fraction(c["theta"])
    keys = b * hkv * n * d
    if c["kind"] == "scan":
        return {"bytes": 2 * keys * es + keys / 8 + 8 * b * hkv, "flops": 2 * keys}
    hq, w = c["hq"], min(c["window"], n)
    byts = 2 * (b * hq * n * d + keys) * es + keys / 8 + 8 * b * hkv
    pairs = n * (n + 1) / 2
    inside = (n // w) * w * (w + 1) / 2 + (n % w) * (n % w + 1) / 2
    if c["shape"] == "sliding":
        inside = w * n - w * (w - 1) / 2
    # scores: all channels inside the window, the surviving entries outside; P V over every causal pair
    flops = 2 * b * hq * d * (inside + kept * (pairs - inside) + pairs)
    if c["kind"] == "generate":
        for t in range(n + 1, n + c["steps"] + 1):
            near = min(c["decode_window"], t)
            byts += b * hkv * (t * d * es + near * d * es + (t - near) * d * (1 / 8 + kept * es)) + 2 * b * hq * d * es
            flops += 4 * b * hq * d * t
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    if case["kind"] == "scan":
        return "exact"
    # masks and counts are whole numbers and have one right value; outputs are bf16 (probabilities too), or fp32 sums
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
