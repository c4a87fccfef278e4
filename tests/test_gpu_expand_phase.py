"""The expand phase of the tiled GEMM at its edges: rank chunks of 32 and slabs of 16 rows (whole
and partial), one to hundreds of buckets per row tile (batches, their places, groups of 64),
consecutive and strided 32-row blocks, both tile heights, tokens without adapter."""
import sys

import numpy as np
import pytest

from paper_2603_15965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d_in,d_out,C,rank,structure", [
    (600, 64, 136, 1, 8, "uniform"),      # one K tile, one bucket, half a slab
    (513, 200, 264, 3, 24, "uniform"),    # rank 24: a whole and a half slab
    (700, 136, 128, 5, 40, "uniform"),    # two chunks, the second of half a slab
    (530, 128, 520, 2, 128, "uniform"),   # four chunks
    (900, 192, 256, 20, 64, "zipf"),      # several batches per chunk, strided blocks
    (1000, 320, 264, 300, 16, "zipf"),    # more than 64 buckets in a tile
    (777, 96, 200, 600, 8, "uniform"),    # about a row per bucket
    (1100, 72, 136, 130, 48, "zipf"),     # both: groups of 64 and two chunks
])
@pytest.mark.parametrize("tile_rows", [128, 256])
def test_expand_phase(N, d_in, d_out, C, rank, structure, tile_rows):
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"expand N={N} {d_in}->{d_out} C={C} rank={rank} {structure} tile_rows={tile_rows}", flush=True)
    sys.stdout.flush()
    w = wl.custom("expand", N, d_in, d_out, C, rank, wl.BASE_SEED + 41000 + N, structure=structure)
    r = w.r.copy()
    r[::37] = -1
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    offsets, perm = mb.molora_bucket(gpu.dev_i32(r), C)
    t = mb.molora_shrink(x, A, offsets, perm)
    h = mb.molora_base_expand(x, W, B, t, offsets, perm, tile_rows=tile_rows)
    torch.cuda.synchronize()
    gpu.assert_h_close(h.cpu().numpy(), oracle.apply(w.x, w.W, w.A, w.B, r), "expand phase")


@pytest.mark.parametrize("N,d_in,d_out,C,rank", [
    (4779, 80, 8, 2, 24),       # 64 x 128 tiles
    (2025, 72, 1992, 8, 24),    # 128 x 128, four stages
    (5909, 72, 648, 2, 16),     # 128 x 128, two workgroups per compute unit
    (8295, 72, 1048, 1, 16),    # 192 x 256
    (8111, 72, 1296, 6, 16),    # 256 x 256
    (8083, 72, 1848, 7, 8),     # 320 x 256
    (1155, 2088, 6304, 7, 16),   # 128 x 256
])
def test_tile_configurations(N, d_in, d_out, C, rank):
    """Shapes for which the cost rule picks each of the row-tile configurations, none of them a
    multiple of its tile."""
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"tile configurations N={N} {d_in}->{d_out} C={C} rank={rank}", flush=True)
    sys.stdout.flush()
    w = wl.custom("tiles", N, d_in, d_out, C, rank, wl.BASE_SEED + 42000 + N)
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    h = mb.molora_apply(x, W, A, B, gpu.dev_i32(w.r))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(0, N, 13), np.arange(max(0, N - 40), N)])).astype(np.int64)
    gpu.assert_h_close(h[torch.from_numpy(rows).cuda()].cpu().numpy(),
                       oracle.apply_rows(w.x, w.W, w.A, w.B, w.r, rows), "tile configurations")
