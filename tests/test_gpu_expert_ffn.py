"""The expert FFN alone (moe_expert_ffn_fwd, moe_expert_ffn_bwd) at the edges of the GEMM tiles: rows per
expert around multiples of the tile heights, dimensions that end inside a tile or inside a k step, experts
without rows.  Padding rows hold NaN and must stay out of every result."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}          # max|gpu - ref| / max|ref|, as everywhere in these tests


def _run(dtype, M, H, counts, Cp, seed, recompute, overwrite):
    from paper_2506_22175_amd import binding as B
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    E = len(counts)
    cfg = B.make_config(E * Cp, M, H, E, 1, 1.0, 1, B.MOE_BF16 if dtype == "bf16" else B.MOE_F32, 0, overwrite)
    assert B.moe_capacity(cfg) == Cp
    g = torch.Generator().manual_seed(seed)
    d = "cuda:0"
    x = torch.randn((E * Cp, M), generator=g).to(dt)
    dy = torch.randn((E * Cp, M), generator=g).to(dt)
    W1 = (torch.randn((E, M, H), generator=g) * 0.05).to(dt)
    W2 = (torch.randn((E, H, M), generator=g) * 0.05).to(dt)
    w = torch.rand((E * Cp,), generator=g) * 0.5 + 0.1
    old1, old2 = torch.randn((E, M, H), generator=g), torch.randn((E, H, M), generator=g)
    for e in range(E):
        for t in (x, dy):
            t[e * Cp + counts[e]:(e + 1) * Cp] = float("nan")
        w[e * Cp + counts[e]:(e + 1) * Cp] = float("nan")
    nan = lambda *s, dtype=dt: torch.full(s, float("nan"), dtype=dtype, device=d)  # noqa: E731
    Z, A, DO, dZ, dDI = nan(E * Cp, H), nan(E * Cp, H), nan(E * Cp, M), nan(E * Cp, H), nan(E * Cp, M)
    parts = B.moe_dw_parts(cfg)
    dw_part = nan(E * Cp, parts, dtype=torch.float32)
    dW1, dW2 = (nan(E, M, H, dtype=torch.float32), nan(E, H, M, dtype=torch.float32)) if overwrite else (old1.to(d), old2.to(d))
    c = torch.tensor([counts], dtype=torch.int32, device=d)
    xd, dyd, W1d, W2d, wd = (t.to(d) for t in (x, dy, W1, W2, w))
    B.moe_expert_ffn_fwd(cfg, 0, xd, c, W1d, W2d, None if recompute else Z, A, DO)
    B.moe_expert_ffn_bwd(cfg, 0, int(recompute), xd, Z, dyd, c, wd, W1d, W2d, dZ, dDI, dW1, dW2, dw_part)
    torch.cuda.synchronize()
    got = {n: t.double().cpu() for n, t in (("DO", DO), ("dDI", dDI), ("dW1", dW1), ("dW2", dW2))}
    got["dw"] = dw_part.double().cpu().sum(1)
    ref = {n: torch.full_like(t, float("nan")) for n, t in got.items()}
    for e in range(E):
        q = slice(e * Cp, e * Cp + counts[e])
        xe, dye, we = x[q].double(), dy[q].double(), w[q].double()[:, None]
        w1, w2 = W1[e].double(), W2[e].double()
        z = xe @ w1
        cdf = 0.5 * (1 + torch.erf(z / math.sqrt(2)))
        a = z * cdf
        G = dye @ w2.t()
        dz = we * G * (cdf + z * torch.exp(-z * z / 2) / math.sqrt(2 * math.pi))
        ref["DO"][q], ref["dDI"][q], ref["dw"][q] = a @ w2, dz @ w1.t(), (a * G).sum(1)
        ref["dW1"][e] = xe.t() @ dz + (0 if overwrite else old1[e].double())
        ref["dW2"][e] = (we * a).t() @ dye + (0 if overwrite else old2[e].double())
    for n in ref:
        live = ~torch.isnan(ref[n])
        assert bool(torch.isfinite(got[n][live]).all()), n
        if n in ("DO", "dDI"):
            assert bool(torch.isnan(got[n][~live]).all()), n + ": a padding row was written"
        err = (got[n][live] - ref[n][live]).abs().max() / ref[n][live].abs().max()
        assert err <= TOL[dtype], (n, float(err))


@pytest.mark.parametrize("recompute,overwrite", [(0, 1), (1, 0)])
@pytest.mark.parametrize("M,H,counts,Cp", [
    (8, 8, (1, 0, 3), 3),                       # one k step that is nearly empty, an expert without rows
    (40, 72, (31, 32, 33, 64), 65),             # around 32 and 64 rows; k and columns end inside a step
    (136, 200, (63, 65, 128, 129), 130),
    (264, 328, (257, 1, 0, 255), 260),          # one row into a second tile of 256
], ids=["min", "rows32", "rows64", "rows256"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_expert_ffn_at_tile_edges(dtype, M, H, counts, Cp, recompute, overwrite):
    _run(dtype, M, H, counts, Cp, 11, recompute, overwrite)
