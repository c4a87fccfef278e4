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


@pytest.mark.parametrize("tile,N,d_in,d_out,C,rank", [
    ((64, 128, 3), 4779, 80, 8, 2, 24),
    ((64, 128, 3), 4418, 328, 8, 14, 8),
    ((64, 128, 3), 4159, 520, 8, 200, 64),        # strided blocks, two chunks
    ((128, 128, 4), 2025, 72, 1992, 8, 24),
    ((128, 128, 4), 8955, 456, 136, 1, 64),       # two chunks
    ((128, 128, 4), 6071, 520, 520, 200, 16),     # strided
    ((128, 128, 2), 5909, 72, 648, 2, 16),
    ((128, 128, 2), 8227, 392, 392, 14, 48),      # two chunks
    ((128, 128, 2), 5849, 328, 656, 200, 64),     # strided, two chunks
    ((128, 256, 3), 1155, 2088, 6304, 7, 16),
    ((128, 256, 3), 4739, 2760, 1424, 14, 40),    # two chunks
    ((128, 256, 3), 3766, 3080, 1984, 130, 40),   # strided, two chunks
    ((192, 256, 2), 8295, 72, 1048, 1, 16),
    ((192, 256, 2), 7261, 328, 1032, 14, 40),     # two chunks
    ((192, 256, 2), 5955, 392, 1296, 200, 8),     # strided
    ((192, 256, 2), 5408, 392, 1416, 200, 48),    # strided, two chunks
    ((256, 256, 2), 8111, 72, 1296, 6, 16),
    ((256, 256, 2), 8119, 392, 1288, 7, 40),      # two chunks
    ((256, 256, 2), 5429, 328, 2056, 200, 16),    # strided
    ((320, 256, 2), 8083, 72, 1848, 7, 8),
    ((320, 256, 2), 7948, 392, 1808, 40, 64),     # two chunks, several batches
    ((320, 256, 2), 5409, 328, 2976, 200, 16),    # strided
    ((320, 256, 2), 5637, 328, 2832, 200, 64),    # strided, two chunks
    ((320, 256, 2), 5003, 2728, 3176, 13, 40),    # a layer of a model
    ((192, 256, 2), 1333, 2048, 6144, 40, 24),
])
def test_tile_configurations(tile, N, d_in, d_out, C, rank):
    """Every row-tile configuration, taken by the cost rule and checked to be: one or two K tiles, five and
    more (the loops that refill their stages) in odd and even numbers with a K tail, consecutive
    and strided 32-row blocks, one and two chunks of the rank."""
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    assert mb.molora_base_expand_tile(N, d_in, d_out, C, rank) == tile
    print(f"tile configurations {tile} N={N} {d_in}->{d_out} C={C} rank={rank}", flush=True)
    sys.stdout.flush()
    w = wl.custom("tiles", N, d_in, d_out, C, rank, wl.BASE_SEED + 42000 + N)
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    h = mb.molora_apply(x, W, A, B, gpu.dev_i32(w.r))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(0, N, 13 if d_in < 1000 else 41), np.arange(max(0, N - 40), N)])).astype(np.int64)
    gpu.assert_h_close(h[torch.from_numpy(rows).cuda()].cpu().numpy(),
                       oracle.apply_rows(w.x, w.W, w.A, w.B, w.r, rows), "tile configurations")


@pytest.mark.parametrize("sizes", [
    [15, 1, 16, 17, 31, 33, 47, 32, 8, 24, 300, 16, 400, 48],   # consecutive blocks
    [16] * 30 + [15, 1, 17, 15, 31, 1, 33, 15],                 # strided ones
])
def test_bucket_edges_at_sixteen_rows(sizes):
    """Buckets that begin and end at, before and behind the 16-row halves of a block."""
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    N, C, rank = sum(sizes), len(sizes), 40
    print(f"bucket edges N={N} C={C}", flush=True)
    w = wl.custom("edges", N, 136, 264, C, rank, wl.BASE_SEED + 44700 + N)
    r = np.random.default_rng(N).permutation(np.repeat(np.arange(C, dtype=np.int32), sizes))
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    offsets, perm = mb.molora_bucket(gpu.dev_i32(r), C)
    t = mb.molora_shrink(x, A, offsets, perm)
    h = mb.molora_base_expand(x, W, B, t, offsets, perm, tile_rows=128)
    torch.cuda.synchronize()
    gpu.assert_h_close(h.cpu().numpy(), oracle.apply(w.x, w.W, w.A, w.B, r), "bucket edges")


@pytest.mark.parametrize("N,d_out", [
    (4096, 2048),    # 512 tiles: one whole round of runs, nothing left over
    (4100, 2056),    # 561: 49 left, not a multiple of the eight XCDs
    (16400, 1032),   # 1161: two whole rounds, 137 left
    (16300, 1024),   # 1024
])
def test_tile_numbering(N, d_out):
    """Output tiles of 128 x 128 past a whole round of runs over the XCDs: every row and column comes out."""
    import oracle
    import torch
    import gpu_helpers as gpu
    from paper_2603_15965_amd import binding as mb
    print(f"tile numbering N={N} d_out={d_out}", flush=True)
    w = wl.custom("rounds", N, 72, d_out, 5, 8, wl.BASE_SEED + 43000 + N)
    x, W, A, B = (gpu.dev_bf16(t) for t in (w.x, w.W, w.A, w.B))
    offsets, perm = mb.molora_bucket(gpu.dev_i32(w.r), 5)
    t = mb.molora_shrink(x, A, offsets, perm)
    h = torch.full((N, d_out), float("nan"), device="cuda")
    mb.molora_base_expand(x, W, B, t, offsets, perm, h, tile_rows=128)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(h).all())
    rows = np.arange(0, N, 31, dtype=np.int64)
    gpu.assert_h_close(h[torch.from_numpy(rows).cuda()].cpu().numpy(),
                       oracle.apply_rows(w.x, w.W, w.A, w.B, w.r, rows), "tile numbering")
