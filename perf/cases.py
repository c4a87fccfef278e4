"""Workloads by which the speed of the routed-LoRA path is compared between versions.

A case is one serving or prefill step of a program that uses this library: inputs, weights,
routing inputs, output buffers and workspace are in hand on the GPU, and `run` takes one batch
through the public calls of `binding`.  The value distributions are those of `workloads`
(x ~ N(0,1), W, A, G ~ N(0, 1/d_in), B ~ N(0, 1/rank), all bf16), the shapes those of the
configurations, tests and benchmarks of this repository, or sizes of the same kind.

`kind` says how a program drives the path:

  given    the target of every token is known (a request's adapter): molora_apply
  decode   the same for a decode step of an engine that keeps its weights packed:
           molora_shrink_base_small + molora_expand_small on packed W and B (molora_apply for
           sizes that these calls do not take)
  vocab    targets from the token ids, optionally times the request's adapter: gating,
           dispatch and shrink in one call, then the fused GEMM (for sizes that the one call
           does not take: gating + dispatch, then molora_apply_bucketed)
  gate     learned linear gate: molora_route, then molora_apply
  shared   one gate and one dispatch for the projections of an attention layer (one of width
           d_out, two of width d_kv), each with its own weights and adapters:
           molora_route, molora_bucket, molora_apply_bucketed three times
  mix      router MLP and weighted top-k mixture through a slot table: molora_route_mlp,
           molora_apply_mix
"""
import math

import numpy as np
import torch

from paper_2603_15965_amd import binding as mb
from paper_2603_15965_amd import workloads as wl

MLP_HIDDEN = 64  # hidden units of the router MLP


def listed():
    return [
        # smallest call: 256 tokens through a toy layer, four adapters of rank 8 (configuration 0)
        dict(name="tiny", kind="given", N=256, d_in=256, d_out=256, C=4, rank=8, routing="uniform"),
        # one decode step of a few concurrent requests, each with its own narrow adapter
        dict(name="decode_few", kind="given", N=7, d_in=4096, d_out=4096, C=16, rank=16, routing="zipf"),
        # decode step of a full batch, popularity-skewed adapters, packed weights (configuration 3)
        dict(name="decode_up8", kind="decode", N=64, d_in=4096, d_out=12288, C=16, rank=64, routing="zipf"),
        # a batch between decode and prefill (verification of drafts, short prompts; batch sweep)
        dict(name="batch_256", kind="given", N=256, d_in=4096, d_out=4096, C=8, rank=64, routing="uniform"),
        # a ragged chunk of prefill with request adapters times modality, ranks off the powers of two
        dict(name="chunk_compose", kind="vocab", N=1333, d_in=2048, d_out=6144, C=40, rank=24, routing="compose"),
        # interleaved text / image batch routed by vocabulary (configuration 1)
        dict(name="vocab_q17", kind="vocab", N=4096, d_in=2048, d_out=2048, C=2, rank=16, routing="vocab"),
        # learned gate in front of an up projection (configuration 2)
        dict(name="gate_up17", kind="gate", N=8192, d_in=2048, d_out=6144, C=8, rank=16, routing="gate"),
        # router MLP and top-2 mixture of the same layer (top-k ablation)
        dict(name="mix_top2", kind="mix", N=8192, d_in=2048, d_out=6144, C=8, rank=16, k=2, routing="mlp"),
        # many tenants: 256 adapters of rank 16 with a long tail of small groups (tiling ablation)
        dict(name="tenants_256", kind="given", N=4096, d_in=4096, d_out=4096, C=256, rank=16, routing="zipf"),
        # odd layer widths and an odd batch, no dimension a multiple of a tile
        dict(name="ragged", kind="gate", N=5003, d_in=2728, d_out=3176, C=13, rank=40, routing="gate"),
        # large prefill, q, k and v of one layer under one gate (configuration 4 shapes)
        dict(name="prefill8_qkv", kind="shared", N=16384, d_in=4096, d_out=4096, d_kv=1024, C=32, rank=32, routing="gate"),
        # large prefill, the longest reduction (configuration 4)
        dict(name="prefill8_down", kind="gate", N=16384, d_in=12288, d_out=4096, C=32, rank=32, routing="gate"),
    ]


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choice(["given", "given", "decode", "vocab", "vocab", "gate", "gate", "shared", "mix"])

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def width(lo, hi):  # layer widths: mostly multiples of 256, sometimes only of 8
        w = log_int(lo, hi)
        q = rng.choice([256, 256, 256, 64, 8])
        return min(hi, max(lo, (w + q // 2) // q * q))

    big = 2.0 * 16384 * 12288 * 4096  # flops of the largest listed case
    while True:
        c = dict(kind=kind, N=log_int(128, 16384), d_in=width(256, 12288), d_out=width(256, 12288))
        c["rank"] = rng.choice([8, 16, 16, 24, 32, 32, 40, 64, 64, 128])
        c["C"] = log_int(2, 64)
        if kind == "given":
            c["N"] = log_int(1, 16384)
            c["C"] = log_int(2, 256)
            c["routing"] = rng.choice(["uniform", "zipf", "runs", "one"])
        elif kind == "decode":
            c["N"] = rng.randint(1, 64)
            c["d_in"], c["d_out"] = width(1024, 12288), width(1024, 12288)
            c["rank"] = rng.choice([16, 32, 64, 64, 128])
            c["routing"] = rng.choice(["uniform", "zipf"])
        elif kind == "vocab":
            c["routing"] = rng.choice(["vocab", "compose"])
            c["C"] = 2 if c["routing"] == "vocab" else 2 * log_int(2, 32)
        elif kind == "shared":
            c["d_kv"] = max(256, c["d_out"] // rng.choice([1, 2, 4, 8]) // 8 * 8)
            c["routing"] = "gate"
        elif kind == "mix":
            c["k"] = rng.choice([1, 2, 2, 3])
            c["C"] = rng.randint(c["k"] + 1, {1: 64, 2: 16, 3: 8}[c["k"]])
            c["rank"] = rng.choice([8, 16, 32])
            c["routing"] = "mlp"
        else:
            c["routing"] = "gate"
        w = work(c)
        if w["flops"] <= big and w["bytes"] < 2e9:
            return c


def _outs(case):
    return [case["d_out"]] + ([case["d_kv"]] * 2 if case["kind"] == "shared" else [])


def _targets(case, seed):
    """Host-side routing input: int32 targets, or token ids (and request adapters)."""
    N, C = case["N"], case["C"]
    rng = np.random.Generator(np.random.PCG64(seed))
    how = case["routing"]
    if how == "uniform":
        return wl.uniform_targets(seed, N, C), None
    if how == "zipf":
        return wl.zipf_targets(seed, N, C, 1.1), None
    if how == "one":
        return np.full(N, rng.integers(0, C), dtype=np.int32), None
    if how == "runs":  # the tokens of a request follow one another and share its adapter
        lens = rng.geometric(1.0 / 64, size=N)
        who = rng.integers(0, C, size=N)
        return np.repeat(who, lens)[:N].astype(np.int32), None
    seqs = -(-N // 512)
    ids = wl.interleaved_token_ids(seed, seqs, 512, 32.0, wl.VOCAB_BREAKS)[:N]
    if how == "vocab":
        return ids, None
    lens = rng.geometric(1.0 / 128, size=N)  # "compose": requests of ~128 tokens, an adapter each
    who = rng.integers(0, C // 2, size=N)
    return ids, np.repeat(who, lens)[:N].astype(np.int32)


def prepare(case, seed):
    N, d_in, C, rank = case["N"], case["d_in"], case["C"], case["rank"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * std).to(torch.bfloat16)

    def i32(a):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()

    kind = case["kind"]
    s = dict(kind=kind, x=normal(N, d_in))
    pool = C + 4 if kind == "mix" else C  # a mixture's adapters lie in a pool with spare slots
    s["layers"] = []
    for d_out in _outs(case):
        s["layers"].append(dict(
            W=normal(d_in, d_out, std=d_in ** -0.5), A=normal(pool, d_in, rank, std=d_in ** -0.5),
            B=normal(pool, rank, d_out, std=rank ** -0.5),
            h=torch.empty((N, d_out), dtype=torch.float32, device="cuda")))
    first = s["layers"][0]
    d_out = case["d_out"]
    # buffers that a serving loop allocates once
    s["offsets"] = torch.empty(C + 1, dtype=torch.int32, device="cuda")
    s["perm"] = torch.empty(N, dtype=torch.int32, device="cuda")
    s["r"] = torch.empty(N, dtype=torch.int32, device="cuda")
    if kind == "mix":
        k = case["k"]
        s["k"] = k
        s["W1"] = normal(d_in, MLP_HIDDEN, std=d_in ** -0.5)
        s["W2"] = normal(MLP_HIDDEN, C, std=MLP_HIDDEN ** -0.5)
        s["b1"] = 0.1 * torch.randn(MLP_HIDDEN, generator=gen, device="cuda")
        s["b2"] = 0.1 * torch.randn(C, generator=gen, device="cuda")
        s["idx"] = torch.empty((N, k), dtype=torch.int32, device="cuda")
        s["w"] = torch.empty((N, k), dtype=torch.float32, device="cuda")
        s["slots"] = i32(np.random.Generator(np.random.PCG64(seed)).permutation(pool)[:C])
        lib = mb.load()
        nbytes = lib.molora_apply_mix_workspace_bytes(N, d_in, d_out, C, rank, k)
        s["workspace"] = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
        nbytes = lib.molora_route_mlp_workspace_bytes(N, MLP_HIDDEN)
        s["mlp_workspace"] = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
        return s
    s["workspace"] = mb.new_workspace(N, d_in, max(_outs(case)), C, rank)
    if kind in ("gate", "shared"):
        s["G"] = normal(d_in, C, std=d_in ** -0.5)
        return s
    ids, who = _targets(case, seed)
    if kind == "vocab":
        s["v"], s["adapter"] = i32(ids), None if who is None else i32(who)
        s["breaks"] = [int(b) for b in wl.VOCAB_BREAKS]
        s["n_adapters"] = C // 2
        s["one_launch"] = mb.molora_dense_shrink_supported(N, d_in, C, rank)
        if s["one_launch"]:
            s["t"] = torch.empty((N, 2 * C * rank), dtype=torch.bfloat16, device="cuda")
        return s
    s["r"] = i32(ids)
    if kind == "decode":
        s["packed"] = mb.molora_bucket_shrink_small_supported(N, d_in, C, rank) and mb.molora_pack_w_cols(d_out) > 0
        if s["packed"]:
            s["t"] = torch.empty((N, 2 * rank), dtype=torch.bfloat16, device="cuda")
            s["Wp"], s["Bp"] = mb.molora_pack_w(first["W"]), mb.molora_pack_b(first["B"])
    return s


def run(s):
    x, layer, kind = s["x"], s["layers"][0], s["kind"]
    W, A, B, h = layer["W"], layer["A"], layer["B"], layer["h"]
    if kind == "decode" and s["packed"]:
        offsets, perm, t, h = mb.molora_shrink_base_small(s["r"], x, s["Wp"], A, s["offsets"], s["perm"], s["t"], h,
                                                          packed=True)
        mb.molora_expand_small(s["Bp"], t, offsets, perm, h, packed=True)
        return {"h": h, "offsets": offsets, "perm": perm}
    if kind in ("given", "decode"):
        return {"h": mb.molora_apply(x, W, A, B, s["r"], h=h, workspace=s["workspace"])}
    if kind == "vocab" and s["one_launch"]:
        r, offsets, perm, t = mb.molora_gate_dispatch_shrink(s["v"], s["breaks"], x, A, s["adapter"], s["n_adapters"],
                                                             s["r"], s["offsets"], s["perm"], s["t"])
        return {"h": mb.molora_base_expand_dense(x, W, B, t, offsets, perm, h), "r": r, "offsets": offsets, "perm": perm}
    if kind == "vocab":
        r, offsets, perm = mb.molora_gate_dispatch(s["v"], s["breaks"], s["adapter"], s["n_adapters"], s["r"],
                                                   s["offsets"], s["perm"])
        h = mb.molora_apply_bucketed(x, W, A, B, offsets, perm, h=h, workspace=s["workspace"])
        return {"h": h, "r": r, "offsets": offsets, "perm": perm}
    if kind == "gate":
        r = mb.molora_route(x, s["G"], s["r"])
        return {"h": mb.molora_apply(x, W, A, B, r, h=h, workspace=s["workspace"]), "r": r}
    if kind == "shared":
        r = mb.molora_route(x, s["G"], s["r"])
        offsets, perm = mb.molora_bucket(r, A.shape[0], s["offsets"], s["perm"])
        hs = [mb.molora_apply_bucketed(x, p["W"], p["A"], p["B"], offsets, perm, h=p["h"], workspace=s["workspace"])
              for p in s["layers"]]
        return {"h": hs, "r": r, "offsets": offsets, "perm": perm}
    idx, w = mb.molora_route_mlp(x, s["W1"], s["b1"], s["W2"], s["b2"], s["k"], s["idx"], s["w"], s["mlp_workspace"])
    h = mb.molora_apply_mix(x, W, A, B, idx, w, s["slots"], h=h, workspace=s["workspace"])
    return {"h": h, "idx": idx, "w": w}


def work(case):
    """Bytes and flops of one pass: x, routing input, weights and the adapters in use read once,
    outputs written once; gate or router, shrink, base product and expand."""
    N, d_in, C, rank, kind = case["N"], case["d_in"], case["C"], case["rank"], case["kind"]
    k = case.get("k", 1)
    used = 1 if case["routing"] == "one" else min(C, N * k)
    nbytes = 2.0 * N * d_in
    flops = 0.0
    for d_out in _outs(case):
        nbytes += 2.0 * d_in * d_out + 2.0 * used * rank * (d_in + d_out) + 4.0 * N * d_out
        flops += 2.0 * N * d_in * d_out + 2.0 * N * k * rank * (d_in + d_out)
    if kind in ("gate", "shared"):
        nbytes += 2.0 * d_in * C + 4.0 * N
        flops += 2.0 * N * d_in * C
    elif kind == "mix":
        nbytes += 2.0 * MLP_HIDDEN * (d_in + C) + 8.0 * N * k
        flops += 2.0 * N * MLP_HIDDEN * (d_in + C)
    else:
        nbytes += 4.0 * N * (3 if case["routing"] == "compose" else 2 if kind == "vocab" else 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Targets, lists and selections are whole numbers and equal.  h: exact bf16 products summed in
    fp32, the low-rank intermediate carried in two bf16 halves.  Against the same sums in 64 bits
    (26 cases, 256 rows each) h is off by 1.5e-6 to 1.9e-6 (relative, 2-norm) and by at most
    1.6e-5 (largest, over the rms or the value); four times that.  (A mixture's weights are a
    fixed sequence of fp32 operations, exact on any implementation.)"""
    return {"rel": 7e-6, "max": 6.4e-5}
