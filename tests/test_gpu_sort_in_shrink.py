"""The dispatch step inside the shrink launch (65 .. 8192 tokens): molora_apply against the separate dispatch,
shrink and GEMM, which give the same bits, at the edges of its ranges: a token more or less than a wavefront's or a
workgroup's range, one to 1024 buckets (groups of 64 keys, ballots for up to three), row-item and streaming
shrink with and without K slices, runs of one target, empty buckets, tokens without adapter."""
import numpy as np
import pytest

from paper_2603_15965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d_in,C,rank", [
    (65, 4096, 8, 64),      # four K slices
    (127, 256, 63, 16),     # row items; the keys fill one group
    (256, 1024, 64, 72),    # two K slices, a second group of keys
    (600, 264, 1, 72),      # one bucket
    (1025, 264, 3, 32),     # four keys, by ballots
    (1100, 72, 4, 24),
    (2049, 520, 1024, 8),   # as many buckets as there can be
    (4095, 256, 300, 40),
    (4096, 1024, 16, 96),   # a full range of row items, two per lane short of ...
    (4097, 136, 200, 16),   # ... the first batch past it: a separate dispatch launch for row items
    (5003, 2728, 13, 40),
    (7800, 264, 6, 128),    # 496 workgroups
    (7900, 264, 6, 128),    # 504: a separate dispatch launch
    (8192, 512, 8, 16),
    (8192, 264, 65, 16),
    (8193, 512, 8, 16),     # separate launches
])
@pytest.mark.parametrize("how", ["level", "skewed", "runs", "one", "third", "none"])
def test_apply_equals_separate_launches(N, d_in, C, rank, how):
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"sort in shrink N={N} d_in={d_in} C={C} rank={rank} {how}", flush=True)
    d_out = 128
    if how in ("level", "third"):
        r = wl.uniform_targets(N + C, N, C)
    elif how == "skewed":
        r = wl.zipf_targets(N + C, N, C, 1.3)
    elif how == "runs":
        r = ((np.arange(N) // 97 * 7) % C).astype(np.int32)
    else:
        r = np.full(N, C - 1, dtype=np.int32)
    if how == "none":  # tokens without adapter alone but for two
        r[:] = -1
        r[[3, N - 1]] = 0
    else:
        r = r.copy()
        if how == "third":  # as many tiles of tokens without adapter as four buckets of eight have
            r[::3] = -1
        r[5::41] = -1
        r[7::43] = C
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + C)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)

    x, W, A, B = normal(N, d_in), normal(d_in, d_out), normal(C, d_in, rank), normal(C, rank, d_out)
    rd = gpu.dev_i32(r)
    nan = torch.full((N, d_out), float("nan"), device="cuda")
    ws = mb.new_workspace(N, d_in, d_out, C, rank)
    ws.fill_(0xff)  # nothing in it has to start at zero
    h = mb.molora_apply(x, W, A, B, rd, h=nan.clone(), workspace=ws)
    offsets, perm = gpu.check_bucket(r, C)
    ref = mb.molora_apply_bucketed(x, W, A, B, offsets, perm, h=nan.clone())
    torch.cuda.synchronize()
    assert bool(torch.isfinite(h).all())
    assert torch.equal(h, ref)


@pytest.mark.parametrize("N,d_in,C,rank,k,S,weights", [
    (1500, 256, 8, 16, 2, None, True),    # row items
    (300, 4096, 3, 64, 2, None, True),    # 9 tuples of 128 columns, K slices: weights in the reduction
    (8192, 128, 4, 8, 3, 7, False),       # a full range, no weights, slot table
    (700, 264, 6, 24, 1, None, False),    # one adapter per token, no weights
    (3000, 1024, 5, 32, 2, None, True),   # streaming
    (4200, 72, 30, 8, 2, None, True),     # past the range of row items: key and dispatch launches
])
def test_mixture_with_entries_out_of_range(N, d_in, C, rank, k, S, weights):
    """molora_apply_mix on the same launches, entries outside [0, C) at weight zero."""
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    from test_gpu_mix import mix_case
    print(f"mixture N={N} d_in={d_in} C={C} rank={rank} k={k} S={S} weights={weights}", flush=True)
    w, idx, wts, slots = mix_case(N + 17 * k, N, d_in, 136, C, rank, k, S, True, weights)
    h = mb.molora_apply_mix(gpu.dev_bf16(w.x), gpu.dev_bf16(w.W), gpu.dev_bf16(w.A), gpu.dev_bf16(w.B),
                            gpu.dev_i32(idx), None if wts is None else torch.from_numpy(wts).cuda(),
                            None if slots is None else gpu.dev_i32(slots), C=C)
    torch.cuda.synchronize()
    gpu.assert_h_close(h.cpu().numpy(), oracle.apply_mix(w.x, w.W, w.A, w.B, idx, wts, slots, C=C), "mixture")
