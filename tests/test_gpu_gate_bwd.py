"""Gate backward alone (moe_gate_bwd) at the edges of its token blocks, column blocks and expert blocks."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(T, M, E, k, seed, x_change=None, dtype=torch.float32):
    """dL and dWg of one partition, the same in float64, and the magnitudes that their roundings follow."""
    from paper_2506_22175_amd import binding as B
    cfg = B.make_config(T, M, 64, E, k, 1.0, 1, B.MOE_F32 if dtype == torch.float32 else B.MOE_BF16, grad_overwrite=1)
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((T, M), generator=g).to(dtype)
    if x_change:
        x_change(x)
    logits, dw = torch.randn((T, E), generator=g), torch.randn((T, k), generator=g)
    idx = torch.topk(logits, k, dim=1)[1].to(torch.int32)
    slot = torch.zeros((T, k), dtype=torch.int32)
    d = "cuda:0"
    dL = torch.full((T, E), float("nan"), device=d)
    dWg = torch.full((M, E), float("nan"), device=d)
    scratch = torch.full((B.moe_gate_scratch_bytes(cfg),), 255, dtype=torch.uint8, device=d)
    B.moe_gate_bwd(cfg, 0, x.to(d), logits.to(d), idx.to(d), slot.to(d), dw.to(d), None, dL, dWg, scratch)
    torch.cuda.synchronize()
    p = torch.softmax(logits.double(), 1)
    dp = torch.zeros((T, E), dtype=torch.float64).scatter_(1, idx.long(), dw.double())
    ref = p * (dp - (dp * p).sum(1, keepdim=True))
    mag = p * (dp.abs() + (dp * p).abs().sum(1, keepdim=True))
    return x.double(), dL.cpu().double(), dWg.cpu().double(), ref, mag


@pytest.mark.parametrize("T,M,E,k", [
    (1, 8, 1, 1),              # one token, one expert (no gradient)
    (33, 40, 5, 2),            # one token into a second block of 32; one column block and a piece
    (64, 32, 32, 1),           # whole blocks throughout
    (65, 264, 33, 3),          # one token into a second chunk, one expert into a second block
    (1000, 72, 64, 8),         # several chunks, the most experts and choices
])
def test_gate_backward_matches_float64(T, M, E, k):
    x, dL, dWg, ref, mag = _run(T, M, E, k, T + E)
    # exponentials, E sums and a division, each to a few roundings of 2^-24
    assert bool(((dL - ref).abs() <= mag * (E + 16) * 2.0 ** -24).all())
    # and T products of them, added in any order
    bound = x.abs().t() @ mag * (E + 16 + T) * 2.0 ** -24
    assert bool(((dWg - x.t() @ ref).abs() <= bound).all())


@pytest.mark.parametrize("T,M,E,k", [
    (1, 8, 16, 1), (64, 72, 17, 2), (65, 64, 32, 3), (129, 136, 33, 2), (200, 72, 40, 4), (1000, 264, 48, 8), (65, 72, 49, 2), (130, 72, 64, 8),
])
def test_bfloat16_gate_backward_matches_float64(T, M, E, k):
    """One expert into each further block of sixteen, and whole blocks."""
    x, dL, dWg, ref, mag = _run(T, M, E, k, T + E, dtype=torch.bfloat16)
    assert bool(((dL - ref).abs() <= mag * (E + 16) * 2.0 ** -24).all())
    # as above, with dL as two bfloat16 numbers, the second of which rounds what the first leaves to 2^-9 * 2^-9 of dL
    bound = x.abs().t() @ (mag * (E + 16 + T) * 2.0 ** -24 + dL.abs() * 2.0 ** -17)
    assert bool(((dWg - x.t() @ ref).abs() <= bound).all())


@pytest.mark.parametrize("T", [1, 9, 31, 40, 70])
def test_an_infinite_activation_of_the_last_token_stays_infinite(T):
    M, E = 40, 5

    def last(x):
        x[T - 1, 3], x[T - 1, 38] = float("inf"), -float("inf")
    x, dL, dWg, ref, mag = _run(T, M, E, 2, T, last)
    rest = [c for c in range(M) if c not in (3, 38)]
    assert bool((dWg[3] == dL[T - 1].sign() * float("inf")).all())
    assert bool((dWg[38] == -dL[T - 1].sign() * float("inf")).all())
    assert bool(torch.isfinite(dWg[rest]).all())
