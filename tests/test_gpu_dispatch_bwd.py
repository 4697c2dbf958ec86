"""Dispatch backward at the edges of its column slices, token groups and expert groups."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,M,E,k,n", [
    (37, 8, 1, 1, 1),          # one column unit, one expert
    (3, 264, 17, 3, 1),        # fewer tokens than a round; a ragged expert group; a second slice of 8 columns (f32)
    (260, 520, 32, 2, 2),      # one column unit into the second slice
    (4500, 520, 33, 2, 1),     # several rounds per wavefront; experts that leave a ragged group of four
    (514, 1040, 64, 8, 2),     # the most experts and choices
])
def test_dispatch_bwd_matches_a_float64_reference(dtype, T, M, E, k, n):
    from paper_2506_22175_amd import binding as B
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = B.make_config(T, M, 64, E, k, 1.0, n, B.MOE_BF16 if dtype == "bf16" else B.MOE_F32)
    Cp, Tp = B.moe_capacity(cfg), T // n
    g = torch.Generator().manual_seed(T + E)
    rows = torch.randn((n, E * Cp, M), generator=g).to(dt)
    Wg = (torch.randn((M, E), generator=g) * 0.02).to(dt)
    dL = torch.randn((T, E), generator=g)
    # every partition's kept rows go to different tokens; about a quarter of the choices are dropped
    slot = torch.full((T, k), -1, dtype=torch.int32)
    for p in range(n):
        perm = torch.randperm(E * Cp, generator=g)[:Tp * k].to(torch.int32)
        flat = torch.full((Tp * k,), -1, dtype=torch.int32)
        flat[:perm.numel()] = perm
        flat[torch.rand((Tp * k,), generator=g) < 0.25] = -1
        slot[p * Tp:(p + 1) * Tp] = flat.reshape(Tp, k)
    ref = dL.double() @ Wg.double().t()
    mag = dL.double().abs() @ Wg.double().abs().t()
    for p in range(n):
        for j in range(k):
            s = slot[p * Tp:(p + 1) * Tp, j].long()
            add = rows[p].double()[s.clamp(min=0)] * (s >= 0)[:, None]
            ref[p * Tp:(p + 1) * Tp] += add
            mag[p * Tp:(p + 1) * Tp] += add.abs()
    d = "cuda:0"
    dx = torch.full((T, M), float("nan"), dtype=dt, device=d)
    for p in range(n):
        B.moe_dispatch_bwd(cfg, p, rows[p].to(d), slot.to(d), dL.to(d), Wg.to(d), dx)
    torch.cuda.synchronize()
    err = (dx.cpu().double() - ref).abs()
    # float32: (E + k) roundings of 2^-24 of the running magnitude; bfloat16: one rounding of the result
    # (2^-8 of it) and, up to sixteen experts, 2^-16 of the gate term's products for the two-term split of dL
    bound = mag * ((E + k) * 2.0 ** -24)
    if dtype == "bf16":
        bound += ref.abs() * 2.0 ** -8 + (mag * 2.0 ** -16 if E <= 16 else 0.0)
    assert bool((err <= bound + 1e-30).all()), float((err - bound).max())


@pytest.mark.parametrize("dtype,E", [("bf16", 17), ("bf16", 33), ("bf16", 64), ("f32", 5), ("f32", 64)])
def test_gate_gradients_keep_their_bits_and_infinities(dtype, E):
    """Two experts with equal gate weights and gradients a and -a', a' the sixteen leading bits of a: what is left
    is the other bits.  (bfloat16 up to sixteen experts carries sixteen bits by contract.)"""
    from paper_2506_22175_amd import binding as B
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    T, M = 21, 520
    cfg = B.make_config(T, M, 64, E, 1, 1.0, 1, B.MOE_BF16 if dtype == "bf16" else B.MOE_F32)
    g = torch.Generator().manual_seed(E)
    Wg = torch.zeros((M, E), dtype=dt)
    Wg[:, 1] = (torch.rand((M,), generator=g) + 0.5).to(dt)
    Wg[:, E - 1] = Wg[:, 1]
    a = torch.rand((T,), generator=g) + 1.0
    dL = torch.zeros((T, E))
    dL[:, 1] = a
    dL[:, E - 1] = -(a * 2.0 ** 15).round() * 2.0 ** -15
    dL[3, 1], dL[T - 1, 1] = float("inf"), -float("inf")
    slot = torch.full((T, 1), -1, dtype=torch.int32)
    ref = dL[:, 1:2].double() * Wg[:, 1].double() + dL[:, E - 1:].double() * Wg[:, E - 1].double()
    d = "cuda:0"
    rows = torch.zeros((E * B.moe_capacity(cfg), M), dtype=dt, device=d)
    dx = torch.full((T, M), float("nan"), dtype=dt, device=d)
    B.moe_dispatch_bwd(cfg, 0, rows, slot.to(d), dL.to(d), Wg.to(d), dx)
    torch.cuda.synchronize()
    got = dx.cpu().double()
    infinite = torch.isinf(ref)
    assert bool((got[infinite] == ref[infinite]).all())
    # two products of magnitude below 3, each added with a rounding of 2^-24 of it; one rounding of the result
    bound = 2 * 3 * 2.0 ** -24 + (ref.abs() * 2.0 ** -8 if dtype == "bf16" else 0.0)
    err = (got - ref).abs()
    assert bool((err <= bound)[~infinite].all()), float((err - bound)[~infinite].max())
