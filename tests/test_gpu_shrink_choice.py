"""Shrinks of more than 64 rows around the lines between row items, the streaming kernel and its K-split
form, and batches of 65 .. 512 tokens with a few narrow adapters (token-order intermediate read by
the streaming and the tiled GEMM)."""
import sys

import numpy as np
import pytest

from paper_2603_15965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d_in,d_out,C,rank,structure", [
    (65, 264, 72, 4, 128, "uniform"),       # wide: streams, one tile a bucket
    (1040, 1032, 136, 64, 72, "zipf"),      # 64 buckets, wide
    (1024, 3128, 136, 65, 16, "uniform"),   # one bucket too many for 16 rows each: row items
    (1200, 4104, 72, 16, 24, "uniform"),    # row items: too few tiles
    (200, 8200, 72, 37, 16, "zipf"),        # narrow, K in four slices
    (300, 4104, 72, 40, 64, "uniform"),     # K in two slices
    (130, 4304, 72, 111, 128, "zipf"),      # about a row per bucket, a wide A_c: streams
    (400, 1032, 72, 129, 128, "uniform"),   # ... more than 128 buckets: row items
    (2100, 4104, 72, 16, 64, "zipf"),       # streams, narrow, a K tail
    (130, 4096, 72, 3, 64, "uniform"),      # K in four slices
    (5003, 2728, 264, 13, 40, "zipf"),      # streams with a half-used column group
])
def test_shrink_choice(N, d_in, d_out, C, rank, structure):
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"shrink choice N={N} {d_in}->{d_out} C={C} rank={rank} {structure}", flush=True)
    sys.stdout.flush()
    w = wl.custom("shrink", N, d_in, d_out, C, rank, wl.BASE_SEED + 44000 + N + C, structure=structure)
    r = w.r.copy()
    r[5::23] = -1
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    rows = np.unique(np.concatenate([np.arange(0, N, 1 + N // 300), np.arange(N - 20, N)])).astype(np.int64)
    ref = oracle.apply_rows(w.x, w.W, w.A, w.B, r, rows)
    dev_rows = torch.from_numpy(rows).cuda()
    offsets, perm = mb.molora_bucket(gpu.dev_i32(r), C)
    for workspace in (None, "auto"):
        t = mb.molora_shrink(x, A, offsets, perm, workspace=workspace)
        h = mb.molora_base_expand(x, W, B, t, offsets, perm)
        torch.cuda.synchronize()
        gpu.assert_h_close(h[dev_rows].cpu().numpy(), ref, f"workspace={workspace}")
    # a workspace with no room for partial sums: offsets, perm and t alone
    r256 = lambda b: (b + 255) // 256 * 256
    assert C * rank > 64
    bare = torch.empty(r256(4 * (C + 1)) + r256(4 * N) + r256(4 * N * rank), dtype=torch.uint8, device="cuda")
    h = mb.molora_apply(x, W, A, B, gpu.dev_i32(r), workspace=bare)
    torch.cuda.synchronize()
    gpu.assert_h_close(h[dev_rows].cpu().numpy(), ref, "molora_apply, bare workspace")


@pytest.mark.parametrize("N,d_in,C,rank", [
    (300, 4096, 5, 64),      # K slices, or streaming without them
    (2100, 4096, 16, 64),    # streaming
    (700, 12288, 40, 24),    # row items or slices, a long pitch
    (1100, 1032, 9, 72),
])
def test_a_row_does_not_depend_on_its_neighbours(N, d_in, C, rank):
    """t of a token is the same bits whatever adapters the rest of the batch takes."""
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"row of t N={N} d_in={d_in} C={C} rank={rank}", flush=True)
    rng = np.random.default_rng(N)
    w = wl.custom("rows", N, d_in, 8, C, rank, wl.BASE_SEED + 47000 + N)
    x, A = gpu.dev_bf16(w.x), gpu.dev_bf16(w.A)
    r1 = w.r.copy()
    kept = rng.random(N) < 0.3
    r2 = np.where(kept, r1, rng.integers(0, max(1, C // 3), N)).astype(np.int32)  # the others move to the first buckets
    for workspace in (None, "auto"):
        rows = []
        for r in (r1, r2):
            offsets, perm = mb.molora_bucket(gpu.dev_i32(r), C)
            t = mb.molora_shrink(x, A, offsets, perm, workspace=workspace)
            by_token = torch.empty_like(t)
            by_token[perm.long()] = t
            rows.append(by_token[torch.from_numpy(kept).cuda()])
        assert torch.equal(rows[0], rows[1]), f"workspace={workspace}"


@pytest.mark.parametrize("N,d_in,d_out,C,rank,structure,stages", [
    (65, 8, 8, 5, 8, "uniform", 0),         # 0 stages: the streaming GEMM (up to 32 columns of adapters: test_gpu_one_launch.py)
    (256, 256, 256, 5, 8, "uniform", 0),
    (100, 2048, 4096, 8, 8, "zipf", 0),     # 256 KB of adapters
    (100, 2056, 4096, 8, 8, "zipf", 0),     # ... just above: separate launches
    (512, 1032, 520, 3, 16, "zipf", 0),     # 48 columns
    (300, 520, 2056, 2, 32, "uniform", 0),
    (512, 264, 12288, 4, 8, "uniform", 2),  # tiled: the token's own adapter, buckets more than one
    (65, 256, 11008, 4, 8, "zipf", 3),
    (322, 2048, 6144, 4, 8, "uniform", 4),
    (440, 520, 12288, 4, 16, "zipf", 2),
    (303, 1032, 12288, 2, 32, "uniform", 3),
])
def test_few_narrow_adapters(N, d_in, d_out, C, rank, structure, stages):
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    assert mb.molora_base_expand_tile(N, d_in, d_out, C, rank)[2] == stages
    print(f"few narrow adapters N={N} {d_in}->{d_out} C={C} rank={rank} {structure}", flush=True)
    sys.stdout.flush()
    w = wl.custom("dense", N, d_in, d_out, C, rank, wl.BASE_SEED + 45000 + N + C, structure=structure)
    r = w.r.copy()
    r[2::9] = -1
    r[3::31] = C
    rows = np.unique(np.concatenate([np.arange(0, N, 1 + N * d_out // 2000000), np.arange(N - 20, N)])).astype(np.int64)
    ref = oracle.apply_rows(w.x, w.W, w.A, w.B, r, rows)
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    rd = gpu.dev_i32(r)
    full = mb.new_workspace(N, d_in, d_out, C, rank)
    full.fill_(255)
    h = mb.molora_apply(x, W, A, B, rd, workspace=full)
    assert not bool((full == 255).all()), "the path that these sizes are for leaves offsets, perm and t there"
    h2 = torch.empty_like(h)
    mb.molora_apply_static(x, W, A, B, rd, h2)
    torch.cuda.synchronize()
    gpu.assert_h_close(h[torch.from_numpy(rows).cuda()].cpu().numpy(), ref, "one launch")
    assert torch.equal(h, h2), "on the library's scratch"
