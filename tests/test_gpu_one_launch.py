"""molora_apply in one launch (a small batch, C * rank <= 32) at its edges: rows short of a tile and tiles of 32
and 64 rows, K shorter than a step, of a ragged last step and of several rounds, columns short of a group, one to
four adapters, tokens without adapter; what a row's own adapter does not hold never reaches it."""
import numpy as np
import pytest

from paper_2603_15965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d_in,d_out,C,rank", [
    (1, 8, 8, 1, 8),
    (65, 8, 8, 1, 8),
    (31, 40, 24, 2, 16),
    (64, 72, 136, 4, 8),
    (33, 256, 264, 4, 8),
    (64, 2048, 96, 1, 32),       # two rounds of four steps for every wavefront
    (65, 1032, 520, 3, 8),       # ragged last step, a column group that no adapter fills
    (256, 256, 256, 4, 8),
    (511, 72, 512, 1, 24),       # 32-row tiles, one round of workgroups
    (17, 264, 72, 2, 8),         # nine steps: two in flight
    (130, 504, 328, 3, 8),
    (512, 136, 1024, 2, 16),     # 64-row tiles, a step per wavefront
    (480, 264, 1024, 4, 8),      # ... two
    (500, 504, 1000, 2, 16),
    (500, 712, 1000, 1, 16),     # ... three
    (512, 1160, 1024, 1, 32),    # ... five, in rounds of four
])
def test_one_launch(N, d_in, d_out, C, rank):
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"one launch N={N} {d_in}->{d_out} C={C} rank={rank}", flush=True)
    w = wl.custom("one", N, d_in, d_out, C, rank, wl.BASE_SEED + 44000 + N)
    r = w.r.copy()
    if N > 5:
        r[3::17] = -1
        r[5::23] = C
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    h = torch.full((N, d_out), float("nan"), device="cuda")
    ws = mb.new_workspace(N, d_in, d_out, C, rank)
    ws.fill_(0xa5)
    mb.molora_apply(x, W, A, B, gpu.dev_i32(r), h=h, workspace=ws)
    torch.cuda.synchronize()
    assert bool((ws == 0xa5).all()), "one launch needs no workspace; these sizes took another path"
    gpu.assert_h_close(h.cpu().numpy(), oracle.apply(w.x, w.W, w.A, w.B, r), "one launch")
    if C > 1:  # an infinity and a NaN in the other adapters change no bit of a row
        rows = np.flatnonzero(r == 1)
        A2, B2 = A.clone(), B.clone()
        A2[0, 0, 0], B2[0, rank - 1, d_out - 1] = float("inf"), float("nan")
        h2 = mb.molora_apply(x, W, A2, B2, gpu.dev_i32(r))
        torch.cuda.synchronize()
        sel = torch.from_numpy(rows).cuda()
        assert torch.equal(h2[sel], h[sel])
        none = torch.from_numpy(np.flatnonzero((r < 0) | (r >= C))).cuda()
        assert torch.equal(h2[none], h[none])


@pytest.mark.parametrize("N,d_in,d_out,C,rank", [
    (33, 256, 264, 4, 8),       # a step per wavefront
    (40, 264, 72, 2, 16),       # two, with wavefronts that have one or none, and a ragged last step
    (65, 1032, 520, 3, 8),      # five in rounds of four
    (300, 360, 2048, 1, 24),    # 64-row tiles
    (512, 1160, 1024, 1, 32),
])
def test_infinity_in_x(N, d_in, d_out, C, rank):
    """A token without adapter with an infinity in x has h = x W, infinities of the sign of W; no other row
    changes a bit."""
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"one launch, infinities N={N} {d_in}->{d_out} C={C} rank={rank}", flush=True)
    w = wl.custom("one", N, d_in, d_out, C, rank, wl.BASE_SEED + 44500 + N)
    r = w.r.copy()
    rows = np.array([1, 8, 17, N - 1])
    r[rows] = -1
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    W[W == 0] = 1.0
    rd = gpu.dev_i32(r)
    h = mb.molora_apply(x, W, A, B, rd)
    x2 = x.clone()
    at = [0, d_in - 1, d_in // 2 + 3, (d_in - 1) // 32 * 32 - 1]
    for row, k in zip(rows, at):
        x2[row, k] = float("-inf")
    h2 = mb.molora_apply(x2, W, A, B, rd)
    torch.cuda.synchronize()
    want = h.clone()
    for row, k in zip(rows, at):
        want[row] = torch.where(W[k] > 0, float("-inf"), float("inf"))
    assert torch.equal(h2, want)
