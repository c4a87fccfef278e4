"""molora_apply in one launch (a small batch, C * rank <= 32) at its edges: rows short of a tile and tiles of 32
and 64 rows, K shorter than a step, of a ragged last step and of several rounds, columns short of a group, one to
four adapters, tokens without adapter; what a row's own adapter does not hold never reaches it."""
import numpy as np
import pytest

from paper_2603_15965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d_in,d_out,C,rank", [
    (1, 8, 8, 1, 8),
    (31, 40, 24, 2, 16),
    (33, 256, 264, 4, 8),
    (64, 2048, 96, 1, 32),       # two rounds of four steps for every wavefront
    (65, 1032, 520, 3, 8),       # ragged last step, a column group that no adapter fills
    (256, 256, 256, 4, 8),
    (511, 72, 512, 1, 24),       # 32-row tiles, one round of workgroups
    (512, 136, 1024, 2, 16),     # 64-row tiles
    (500, 712, 1000, 1, 16),
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
    mb.molora_apply(x, W, A, B, gpu.dev_i32(r), h=h)
    torch.cuda.synchronize()
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
