"""The dispatch step inside the launches of a batch of at most 64 tokens, with more buckets than tokens."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _inputs(N, d_in, C, rank):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N * 1000 + C)
    bf = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    return bf(N, d_in), bf(C, d_in, rank)


@pytest.mark.parametrize("N,C", [(1, 2), (2, 1024), (37, 38), (63, 64), (64, 65), (64, 127), (64, 128), (50, 1023), (64, 1024)])
@pytest.mark.parametrize("how", ["random", "one", "none", "last", "descending", "edges"])
def test_order(N, C, how):
    """offsets and perm are those of molora_bucket, t is that of molora_shrink."""
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"order N={N} C={C} {how}", flush=True)
    rng = np.random.default_rng(N + C)
    r = {"random": rng.integers(-1, C + 1, N), "one": np.full(N, C // 2), "none": np.full(N, -1), "last": np.full(N, C - 1),
         "descending": C - 1 - np.arange(N) % C, "edges": np.where(np.arange(N) % 3 == 0, 0, C - 1)}[how].astype(np.int32)
    x, A = _inputs(N, 136, C, 40)
    rd = gpu.dev_i32(r)
    offsets, perm, t = mb.molora_bucket_shrink_small(rd, x, A)
    o2, p2 = mb.molora_bucket(rd, C)
    t2 = mb.molora_shrink(x, A, o2, p2)
    torch.cuda.synchronize()
    assert torch.equal(offsets, o2) and torch.equal(perm, p2)
    n = int(o2[C])
    assert torch.equal(t[:n], t2[:n])


@pytest.mark.parametrize("C", [103, 300])  # a place for every bucket; for every token
def test_many_buckets_cost_no_more_than_few(C):
    """The same 44 rows of the same 40 adapters, named among 40 or among C: the same work (counting the
    targets one by one made the launch 1.6 times as long)."""
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    N, d_in, d_out, rank = 44, 1536, 536, 40
    x, A = _inputs(N, d_in, C, rank)
    W = torch.randn(d_in, d_out, device="cuda").to(torch.bfloat16)
    r = gpu.dev_i32(np.random.default_rng(1).integers(0, 40, N).astype(np.int32))
    h, perm = torch.empty(N, d_out, device="cuda"), torch.empty(N, dtype=torch.int32, device="cuda")
    t = torch.empty(N, 2 * rank, dtype=torch.bfloat16, device="cuda")

    def us(C):
        a, offsets = A[:C].contiguous(), torch.empty(C + 1, dtype=torch.int32, device="cuda")
        best = 1e9
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(50):
                mb.molora_shrink_base_small(r, x, W, a, offsets, perm, t, h)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end) * 20)
        return best

    few, many = us(40), us(C)
    print(f"40 buckets {few:.2f} us, {C} buckets {many:.2f} us", flush=True)
    assert many < 1.2 * few
