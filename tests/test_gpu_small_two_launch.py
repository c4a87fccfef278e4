"""Batches of at most 64 tokens with adapters of rank 32 or less: two launches, K of the base projection
cut into slices, workgroups per bucket that has rows when there are more buckets than tokens."""
import sys

import numpy as np
import pytest

from paper_2603_15965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d_in,d_out,C,rank,structure,slices", [
    (1, 8, 8, 5, 8, "uniform", 1),           # the smallest call (up to 32 columns of adapters: test_gpu_one_launch.py)
    (64, 72, 136, 5, 8, "uniform", 1),       # one short piece of K: unsplit
    (64, 8, 8, 5, 8, "uniform", 1),
    (7, 2048, 4096, 16, 16, "zipf", 2),      # slices of two units
    (7, 4096, 4096, 16, 16, "zipf", 3),
    (32, 4096, 264, 8, 32, "uniform", 8),    # eight slices of one unit
    (33, 2728, 3176, 13, 24, "zipf", 3),     # slices that are no whole number of pieces, a K tail
    (64, 1032, 6088, 200, 16, "zipf", 2),    # more buckets than tokens, a full wavefront of them
    (64, 1032, 6152, 200, 16, "zipf", 1),    # ... and a column group too many for slices
    (5, 520, 72, 1024, 8, "uniform", 2),     # far more buckets than tokens
    (64, 264, 16320, 64, 16, "uniform", 1),  # no room for slices
    (40, 1096, 512, 3, 16, "none", 3),       # no token has an adapter
    (6, 1096, 512, 9, 16, "none", 3),        # ... and more buckets than tokens
])
def test_small_batch_narrow_adapters(N, d_in, d_out, C, rank, structure, slices):
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"two launches N={N} {d_in}->{d_out} C={C} rank={rank} {structure}", flush=True)
    sys.stdout.flush()
    w = wl.custom("small", N, d_in, d_out, C, rank, wl.BASE_SEED + 43000 + N + C,
                  structure="uniform" if structure == "none" else structure)
    r = w.r.copy()
    r[2::5] = -1
    r[4::7] = C
    if structure == "none":
        r[:] = -1
    ref = oracle.apply(w.x, w.W, w.A, w.B, r)
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    rd = gpu.dev_i32(r)
    # the size for another d_out has no room for the slices' sums; the exact room of this batch
    small = mb.new_workspace(N, d_in, 1 << 16, C, rank)
    planes = (4 * (slices - 1) * N * d_out + 255) // 256 * 256
    full = torch.full((small.numel() + planes,), 255, dtype=torch.uint8, device="cuda")
    assert mb.new_workspace(N, d_in, d_out, C, rank).numel() >= full.numel()
    h = mb.molora_apply(x, W, A, B, rd, workspace=full)
    torch.cuda.synchronize()
    assert not bool((full == 255).all()), "the path that these sizes are for leaves offsets, perm and t there"
    gpu.assert_h_close(h.cpu().numpy(), ref, "two launches")
    h2 = torch.empty_like(h)
    mb.molora_apply_static(x, W, A, B, rd, h2)
    torch.cuda.synchronize()
    assert torch.equal(h, h2), "on the library's scratch"
    h3 = mb.molora_apply(x, W, A, B, rd, workspace=small)
    torch.cuda.synchronize()
    gpu.assert_h_close(h3.cpu().numpy(), ref, "unsplit")
    # K in slices: the room is used (other bits), a byte less of it is not
    if slices > 1:
        assert not torch.equal(h, h3)
        h4 = mb.molora_apply(x, W, A, B, rd, workspace=full[:-1])
        torch.cuda.synchronize()
        assert torch.equal(h4, h3), "a workspace a byte short"
