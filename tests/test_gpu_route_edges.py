"""The learned gate at the edges of its kernel: target counts around the 16-target blocks and the
passes, row lengths around the 32-k chunks, the 256-k rounds and the G slabs, C below and off the
multiples of 8, and values that the widening by matrix products must not touch or must not
spread: denormals, NaN and infinities."""
import sys

import numpy as np
import pytest

from paper_2603_15965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in", [8, 40, 536, 544, 552, 808])
@pytest.mark.parametrize("C", [2, 7, 9, 16, 20, 33, 40, 72, 129, 136])
def test_route_gate_edges(d_in, C):
    import oracle
    import torch
    from paper_2603_15965_amd import binding as mb
    N = 17 + 16 * (C % 5)
    print(f"route edges N={N} d_in={d_in} C={C}", flush=True)
    sys.stdout.flush()
    w = wl.custom("edge", N, d_in, 16, C, 8, 9200 + d_in + C, route="gate")
    rng = np.random.default_rng(d_in * 1000 + C)
    x, G = w.x.copy(), w.G.copy()
    for case in range(2):
        if case == 1:
            # a denormal everywhere but in the last column, whose logits decide only if they survive
            x[0, :] = 0x0001
            G[:, C - 1] = 0x7180                              # 2^100 (no product or sum overflows)
            x[N // 2, rng.integers(0, d_in)] = 0x7FC0         # NaN in one token
            x[N - 1, rng.integers(0, d_in)] = 0x7F80          # infinity in one token
            G[rng.integers(0, d_in), C // 2] = 0x7FC0         # NaN in one target's column
        r = mb.molora_route(mb.bf16_tensor(x), mb.bf16_tensor(G)).cpu().numpy()
        torch.cuda.synchronize()
        assert np.array_equal(r, oracle.route_gate(x, G)), f"case {case}"


@pytest.mark.parametrize("what", ["token", "target"])
def test_a_non_finite_value_does_not_stall_the_gate(what):
    """One NaN in x, or one infinity in G, where the chains are computed again: a few times the launch, not
    fifty (2 to 3 times measured; a term after another it was 16 to 68 times)."""
    import torch
    from paper_2603_15965_amd import binding as mb
    N, d_in, C = 8192, 4096, 32
    x, G = torch.randn(N, d_in, device="cuda").to(torch.bfloat16), torch.randn(d_in, C, device="cuda").to(torch.bfloat16)
    r = torch.empty(N, dtype=torch.int32, device="cuda")

    def us():
        best = 1e9
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(4):
                mb.molora_route(x, G, r)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end) * 250)
        return best

    us()
    clean = us()
    if what == "token":
        x[N // 2, d_in // 3] = float("nan")
    else:
        G[d_in // 2, C // 2] = float("inf")
    bad = us()
    print(f"{what}: {clean:.1f} us, {bad:.1f} us with a non-finite value", flush=True)
    assert bad < 6 * clean
