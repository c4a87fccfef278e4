"""Scratch and workspace sizes, which follow from the choice of kernels (host-side, no GPU)."""
import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2603_15965_amd import binding
    return binding.load()


# (N, d_in, C, rank): slices of K
@pytest.mark.parametrize("N,d_in,C,rank,slices", [
    (611, 12032, 37, 16, 4),   # 22.5 us in one launch, 13.0 in slices
    (761, 5248, 10, 40, 4),    # 15.9 / 10.8
    (402, 6400, 4, 40, 4),     # 17.4 / 11.1
    (220, 8960, 59, 40, 2),    # 22.6 / 17.5
    (1065, 1248, 5, 128, 0),   # 7.5 / 9.5
    (1638, 11224, 203, 96, 0),
    (16384, 4096, 32, 32, 0),
])
def test_long_chains_of_k_are_sliced(lib, N, d_in, C, rank, slices):
    assert lib.molora_shrink_workspace_bytes(N, d_in, C, rank) == (4 * N * rank * slices + 255) // 256 * 256
