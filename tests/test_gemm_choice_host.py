"""The choice of the GEMM's kernel and tile, which is made on the host from the sizes (no GPU)."""
import pytest

from paper_2603_15965_amd import binding as mb


@pytest.mark.parametrize("N,d_in,d_out,C,rank", [
    (311, 256, 7168, 62, 128),    # 41 us, 64 in tiles of 64 x 128
    (528, 1664, 5120, 180, 128),  # 88 / 121
    (335, 1280, 6912, 130, 96),   # 58 / 82
    (683, 376, 3144, 189, 128),   # 68 / 92
    (64, 4096, 12288, 16, 64),    # one row tile
    (256, 4096, 4096, 8, 64),
])
def test_streams(N, d_in, d_out, C, rank):
    assert mb.molora_base_expand_tile(N, d_in, d_out, C, rank)[2] == 0


@pytest.mark.parametrize("tile,N,d_in,d_out,C,rank", [
    ((192, 256, 2), 1333, 2048, 6144, 40, 24),    # 55 us, 67 in tiles of 128 rows
    ((128, 256, 3), 4096, 2048, 2048, 2, 16),     # 35.5 us from HBM, 41 in tiles of 128 columns
    ((128, 128, 2), 4096, 1024, 2048, 2, 16),
    ((256, 256, 2), 8192, 2048, 6144, 8, 16),
    ((320, 256, 2), 5003, 2728, 3176, 13, 40),    # 109 us, 154 in tiles of 256 rows
    ((256, 256, 2), 16384, 12288, 4096, 32, 32),
])
def test_tiles(tile, N, d_in, d_out, C, rank):
    assert mb.molora_base_expand_tile(N, d_in, d_out, C, rank) == tile


@pytest.mark.parametrize("tile,N,d_in,d_out,C,rank", [
    ((64, 64, 0), 600, 328, 1000, 7, 24),
    ((64, 64, 0), 1500, 1096, 392, 5, 16),
    ((128, 128, 2), 2304, 192, 2560, 6, 16),
    ((192, 256, 2), 2500, 128, 4000, 9, 8),
    ((128, 128, 2), 3000, 3080, 2600, 5, 24),
    ((128, 128, 2), 1250, 3072, 6504, 12, 16),
    ((128, 128, 2), 4090, 1024, 2048, 3, 8),
    ((128, 256, 3), 4000, 3080, 1992, 5, 24),
    ((128, 256, 3), 1100, 3072, 3800, 12, 16),
    ((128, 256, 3), 4090, 4096, 2048, 3, 8),
    ((64, 64, 0), 1500, 520, 392, 4, 16),
    ((64, 32, 0), 700, 256, 264, 2, 32),
    ((64, 128, 3), 3000, 264, 520, 8, 8),
    ((192, 256, 2), 2500, 128, 4000, 3, 8),
    ((128, 128, 4), 384, 1024, 8192, 6, 16),
    ((128, 128, 4), 200, 4096, 12288, 16, 64),
    ((64, 64, 0), 576, 4096, 1024, 8, 32),
    ((64, 64, 0), 1500, 4104, 520, 5, 24),
    ((64, 128, 3), 2100, 128, 512, 37, 8),
])
def test_the_parity_tests_take_the_kernels_they_name(tile, N, d_in, d_out, C, rank):
    """A change of the costs moves these shapes: the labels in test_gpu_parity.py then follow."""
    assert mb.molora_base_expand_tile(N, d_in, d_out, C, rank) == tile


def test_sizes_without_a_tile():
    for bad in [(0, 64, 64, 4, 8), (16, 60, 64, 4, 8), (16, 64, 64, 0, 8), (16, 64, 64, 4, 12)]:
        with pytest.raises(mb.MoloraError):
            mb.molora_base_expand_tile(*bad)
