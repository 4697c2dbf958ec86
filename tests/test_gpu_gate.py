"""The gate by itself at the edges of its kernels: tokens that end inside a wavefront's or a workgroup's set, around
the numbers at which a wavefront takes more of them, experts that do not fill a power of two, gate weights that are not
16-byte aligned, rows that end inside a span of 512, equal logits, infinities and NaN."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle
from paper_2506_22175_amd import binding as B

pytestmark = pytest.mark.gpu

D = "cuda:0"


@pytest.mark.parametrize("T,M,E,k,dtype", [
    (1, 8, 64, 8, "bf16"), (3, 520, 33, 2, "bf16"), (9, 1032, 64, 8, "f32"), (50, 512, 17, 3, "f32"), (17, 72, 32, 1, "bf16"),
    (2047, 136, 64, 2, "bf16"), (2049, 136, 64, 2, "bf16"), (4095, 72, 32, 2, "f32"), (4097, 72, 32, 2, "bf16"), (4097, 72, 27, 2, "f32"),
    (2050, 520, 48, 4, "f32"), (16385, 8, 32, 1, "f32"),
    (1, 8, 1, 1, "f32"), (15, 520, 4, 2, "bf16"), (8191, 24, 8, 2, "bf16"), (8193, 24, 7, 2, "f32"), (4095, 24, 16, 3, "f32"), (4097, 24, 11, 3, "bf16"),
])
@pytest.mark.parametrize("renorm", [0, 1])
def test_gate(T, M, E, k, dtype, renorm):
    """Logits, choices bit for bit; weights to float32 rounding of E exponentials and their sum."""
    if renorm and k == 1:
        pytest.skip("one choice: nothing to renormalise")
    dt, mt = (torch.bfloat16, B.MOE_BF16) if dtype == "bf16" else (torch.float32, B.MOE_F32)
    g = torch.Generator().manual_seed(T + E)
    x, Wg = torch.randn((T, M), generator=g).to(dt), (torch.randn((M, E), generator=g) * 0.2).to(dt)
    if E > 4:
        Wg[:, E // 2] = Wg[:, 1]                    # equal logits: the lower index wins
        Wg[:, E - 1] = Wg[:, 1]
    bias = None if renorm else torch.randn((E,), generator=g)
    if bias is not None and E > 4:
        bias[E // 2] = bias[E - 1] = bias[1]
    if T > 8:
        x[4, 0], x[6, 1] = float("inf"), float("nan")
    cfg = B.make_config(T, M, 8, E, k, 1.0, 1, mt, 0, gate_renormalize=renorm)
    ref, _, idx, w = moe_oracle.route(x.float().numpy(), Wg.float().numpy(), k, None if bias is None else bias.numpy(), bool(renorm))
    odd = torch.empty((M * E + 1,), dtype=dt, device=D)
    odd[1:] = Wg.reshape(-1).to(D)
    for weights in (Wg.to(D), odd[1:].view(M, E)):
        lo = torch.full((T, E), 7.0, device=D)
        ti, tw = torch.full((T, k), -9, dtype=torch.int32, device=D), torch.full((T, k), -9.0, device=D)
        B.moe_route(cfg, x.to(D), weights, None if bias is None else bias.to(D), lo, ti, tw)
        got = lo.cpu().numpy()
        assert np.array_equal(got, ref, equal_nan=True)
        assert np.array_equal(ti.cpu().numpy(), idx)
        fine = np.isfinite(ref).all(axis=1)
        assert fine.any()
        # expf within 2 units, logit - max rounded once (half a unit of a difference of up to 60), a sum of 64, a quotient
        assert np.abs(tw.cpu().numpy() / w - 1.0)[fine].max() <= 2.0 ** -23 * (60 + 64 + 6)


@pytest.mark.parametrize("T,E,k,dtype", [
    (300, 17, 2, "bf16"), (300, 32, 8, "f32"), (5000, 24, 1, "bf16"), (300, 33, 3, "f32"), (300, 64, 2, "bf16"), (3000, 64, 8, "f32"),
])
@pytest.mark.parametrize("odd", [None, float("inf"), float("nan")], ids=["finite", "infinite", "nan"])
def test_weights_are_the_same_bits_for_few_and_for_many_experts(T, E, k, dtype, odd):
    """Sixteen experts by themselves, where one lane adds up a token's exponentials in ascending order, and the same sixteen
    in the same order among experts whose logits are -infinity: those add zeros to the sum, so the weights are the same
    bits, for infinite and NaN logits too."""
    few, M = 16, 72
    dt, mt = (torch.bfloat16, B.MOE_BF16) if dtype == "bf16" else (torch.float32, B.MOE_F32)
    g = torch.Generator().manual_seed(T + E)
    x, Wg = torch.randn((T, M), generator=g).to(dt).to(D), (torch.randn((M, few), generator=g) * 0.2).to(dt)
    if odd is not None:
        Wg[3, 5] = odd
    place = torch.sort(torch.randperm(E, generator=g)[:few])[0]
    many, bias = torch.zeros((M, E), dtype=dt), torch.full((E,), -float("inf"))
    many[:, place], bias[place] = Wg, torch.randn((few,), generator=g)
    got = []
    for n, W, b in ((few, Wg, bias[place]), (E, many, bias)):
        cfg = B.make_config(T, M, 8, n, k, 1.0, 1, mt, 0)
        lo, ti, tw = torch.empty((T, n), device=D), torch.empty((T, k), dtype=torch.int32, device=D), torch.empty((T, k), device=D)
        B.moe_route(cfg, x, W.contiguous().to(D), b.contiguous().to(D), lo, ti, tw)
        got.append((lo.cpu(), ti.cpu().long(), tw.cpu()))
    (lo, ti, tw), (lo_many, ti_many, tw_many) = got
    assert np.array_equal(lo.numpy(), lo_many[:, place].numpy(), equal_nan=True)
    assert torch.equal(place[ti], ti_many)
    assert np.array_equal(tw.numpy(), tw_many.numpy(), equal_nan=True)


@pytest.mark.parametrize("T,M,E,dtype", [
    (4097, 1000, 7, "f32"), (16385, 40, 28, "bf16"), (24577, 72, 32, "bf16"), (8193, 504, 44, "bf16"), (12289, 72, 35, "bf16"), (8193, 72, 17, "f32"), (24577, 40, 24, "f32"),
    (4097, 504, 33, "f32"), (6145, 384, 60, "f32"), (24577, 40, 48, "f32"), (20481, 504, 64, "f32"), (1000, 4096, 20, "f32"), (701, 8192, 28, "bf16"),
])
def test_gate_of_many_tokens_is_that_of_its_pieces(T, M, E, dtype):
    """Around the numbers of tokens from which a wavefront takes more of them and the gate weights stay in LDS, with gate
    weights read by eights and one by one: the same bits as for 600 tokens at a time."""
    dt, mt = (torch.bfloat16, B.MOE_BF16) if dtype == "bf16" else (torch.float32, B.MOE_F32)
    g, k, piece = torch.Generator(D).manual_seed(T + E), 3, 600
    x, Wg = torch.randn((T, M), generator=g, device=D).to(dt), (torch.randn((M, E), generator=g, device=D) * 0.2).to(dt)
    bias = torch.randn((E,), generator=g, device=D)

    def gate(rows):
        n = rows.shape[0]
        cfg = B.make_config(n, M, 8, E, k, 1.0, 1, mt, 0)
        out = torch.empty((n, E), device=D), torch.full((n, k), -9, dtype=torch.int32, device=D), torch.empty((n, k), device=D)
        B.moe_route(cfg, rows, Wg, bias, *out)
        return out
    whole = gate(x)
    for t in range(0, T, piece):
        for a, b in zip(whole, gate(x[t:t + piece].contiguous())):
            assert torch.equal(a[t:t + piece], b)
