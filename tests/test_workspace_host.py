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


def _sizes(rng):
    d_in = rng.choice([256, 1024, 2048, 4096, 5248, 8192, 12288, 14080])
    C = rng.choice([1, 2, 5, 16, 31, 32, 33, 60, 64, 65, 100, 127, 128, 200, 480, 700])
    return d_in, rng.choice([512, 2048, 4096, 8192, 12288]), C, rng.choice([8, 16, 32, 40, 64, 96, 128])


def test_a_workspace_for_the_largest_batch_takes_every_smaller_one(lib):
    """Neither size decreases with N.  (What a batch needs for itself does: 64 tokens cut K into slices,
    256 may not, and a decode step was refused a workspace sized for a batch of 256.)"""
    import random
    rng = random.Random(7)
    for _ in range(400):
        d_in, d_out, C, rank = _sizes(rng)
        k = rng.choice([1, 2])
        edges = [64 * m + o for m in range(1, 40) for o in (-1, 0, 1)]
        big = sorted(rng.randint(2049, 40000) for _ in range(60))
        Ns = sorted(set(list(range(1, 131)) + edges + [2047, 2048, 2049] + big))
        f = [lib.molora_apply_workspace_bytes(N, d_in, d_out, C, rank) for N in Ns]
        assert f == sorted(f), (d_in, d_out, C, rank)
        g = [lib.molora_apply_mix_workspace_bytes(N, d_in, d_out, C, rank, k) for N in Ns]
        assert g == sorted(g), (d_in, d_out, C, rank, k)


def test_room_for_the_slices_of_a_decode_step(lib):
    """A workspace for 256 tokens holds the plane of x W over K slices of any batch of up to 64: two planes
    at 7 x 4096 -> 4096, one at 64."""
    f = lib.molora_apply_workspace_bytes
    assert f(256, 4096, 4096, 16, 16) >= 2 * 7 * 4096 * 4 and f(256, 4096, 4096, 16, 16) >= 64 * 4096 * 4
    assert f(256, 4096, 4096, 16, 16) >= f(64, 4096, 4096, 16, 16)


def test_the_library_scratch_takes_a_batch_by_its_own_need(lib):
    """The size of a workspace for up to N tokens may exceed the library's scratch where N tokens alone fit
    it: those sizes are not refused for it (the call stops at its null pointers, or for want of a device)."""
    import ctypes
    N, d_in, d_out, C, rank = 33000, 8192, 64, 3, 32
    assert lib.molora_apply_workspace_bytes(N, d_in, d_out, C, rank) > lib.molora_static_workspace_bytes()
    r = ctypes.c_void_p(1 << 20)  # never read
    call = lambda n: lib.molora_apply_static(None, None, None, None, r, None, n, d_in, d_out, C, rank, None)
    assert call(N) != -3 and call(3 * N) == -3
