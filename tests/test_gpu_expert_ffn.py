"""The expert FFN alone (moe_expert_ffn_fwd, moe_expert_ffn_bwd) at the edges of the GEMM tiles: rows per
expert around multiples of the tile heights, dimensions that end inside a tile or inside a k step, experts
without rows.  Padding rows hold NaN and must stay out of every result."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}          # max|gpu - ref| / max|ref|, as everywhere in these tests


def _run(dtype, M, H, counts, Cp, seed, recompute, overwrite, mean=None, tiles=None):
    """mean: rows per expert when all are loaded alike (the capacity unless given); tiles: the output tiles, by GEMM,
    that the case is meant to be computed in."""
    from paper_2506_22175_amd import binding as B
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    E = len(counts)
    cfg = B.make_config(E * (mean or Cp), M, H, E, 1, Cp / (mean or Cp), 1, B.MOE_BF16 if dtype == "bf16" else B.MOE_F32, 0, overwrite)
    assert B.moe_capacity(cfg) == Cp
    for gemm, tile in (tiles or {}).items():
        assert B.moe_gemm_tile(cfg, 0, gemm) == tile, gemm
    d = "cuda:0"
    g = torch.Generator(d).manual_seed(seed)
    x = torch.randn((E * Cp, M), generator=g, device=d).to(dt)
    dy = torch.randn((E * Cp, M), generator=g, device=d).to(dt)
    W1 = (torch.randn((E, M, H), generator=g, device=d) * 0.05).to(dt)
    W2 = (torch.randn((E, H, M), generator=g, device=d) * 0.05).to(dt)
    w = torch.rand((E * Cp,), generator=g, device=d) * 0.5 + 0.1
    old1, old2 = torch.randn((E, M, H), generator=g, device=d), torch.randn((E, H, M), generator=g, device=d)
    for e in range(E):
        for t in (x, dy):
            t[e * Cp + counts[e]:(e + 1) * Cp] = float("nan")
        w[e * Cp + counts[e]:(e + 1) * Cp] = float("nan")
    nan = lambda *s, dtype=dt: torch.full(s, float("nan"), dtype=dtype, device=d)  # noqa: E731
    Z, A, DO, dZ, dDI = nan(E * Cp, H), nan(E * Cp, H), nan(E * Cp, M), nan(E * Cp, H), nan(E * Cp, M)
    parts = B.moe_dw_parts(cfg)
    dw_part_and_behind = nan(E * Cp + 256, parts, dtype=torch.float32)      # a tile is at most 256 rows high
    dw_part = dw_part_and_behind[:E * Cp]
    dW1, dW2 = (nan(E, M, H, dtype=torch.float32), nan(E, H, M, dtype=torch.float32)) if overwrite else (old1.to(d, copy=True), old2.to(d, copy=True))
    c = torch.tensor([counts], dtype=torch.int32, device=d)
    xd, dyd, W1d, W2d, wd = (t.to(d) for t in (x, dy, W1, W2, w))
    B.moe_expert_ffn_fwd(cfg, 0, xd, c, W1d, W2d, None if recompute else Z, A, DO)
    B.moe_expert_ffn_bwd(cfg, 0, int(recompute), xd, Z, dyd, c, wd, W1d, W2d, dZ, dDI, dW1, dW2, dw_part)
    torch.cuda.synchronize()
    got = {n: t.double() for n, t in (("DO", DO), ("dDI", dDI), ("dW1", dW1), ("dW2", dW2))}
    got["dw"] = dw_part.double().sum(1)
    kept = torch.zeros((E * Cp + 256,), dtype=torch.bool, device=d)
    for e in range(E):
        kept[e * Cp:e * Cp + counts[e]] = True
    assert bool(torch.isnan(dw_part_and_behind[~kept]).all()), "row dots of a padding row, or past the buffer, were written"
    old1, old2 = old1.to(d), old2.to(d)
    ref = {n: torch.full_like(t, float("nan")) for n, t in got.items()}
    for e in range(E):
        q = slice(e * Cp, e * Cp + counts[e])
        xe, dye, we = xd[q].double(), dyd[q].double(), wd[q].double()[:, None]
        w1, w2 = W1d[e].double(), W2d[e].double()
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


LARGE, HALF, SMALL, FLAT = (256, 256), (256, 128), (128, 128), (64, 128)       # the bfloat16 GEMM's tiles
GEMMS = ("first", "second", "recompute", "dgelu", "dgrad", "dW2", "dW1")


# sizes that the larger bfloat16 tiles are chosen for (the small ones too, for single GEMMs), with last tile rows of
# one row, of a few blocks of 64, of half a tile and one row more, and full ones
@pytest.mark.parametrize("M,H,counts,Cp,tiles", [
    (1024, 4096, (1024, 1023, 897, 896, 641, 129, 64, 0), 1024,
     dict(first=LARGE, second=HALF, dgelu=LARGE, dgrad=HALF, dW2=LARGE, dW1=LARGE)),
    (1024, 4096, (1024, 1025, 960, 1088, 1153, 1152, 897, 0), 1160, dict.fromkeys(GEMMS, LARGE)),
    (520, 4104, (4096, 4097, 4225, 4224), 4300,
     dict(first=LARGE, second=LARGE, dgelu=SMALL, dgrad=LARGE, dW2=SMALL, dW1=SMALL)),
], ids=["half_size", "last_rows", "whole"])
def test_expert_ffn_in_large_tiles(M, H, counts, Cp, tiles):
    _run("bf16", M, H, counts, Cp, 5, 0, 0, tiles=tiles)


# every tile with every epilogue of the expert FFN (256 x 128 accumulates over several partitions only: see the
# layer's tests), dimensions and loads that end inside a tile
@pytest.mark.parametrize("M,H,counts,Cp,mean,recompute,overwrite,tiles", [
    (784, 1312, (160, 1, 0, 128, 129, 64, 65, 32, 33, 127, 160, 96, 97, 31, 130, 159), 160, 128, 1, 0,
     dict(first=HALF, recompute=HALF, second=SMALL, dgelu=FLAT, dgrad=SMALL)),
    (1544, 1544, (1500, 1281), 1500, None, 1, 1,
     dict(first=SMALL, second=HALF, recompute=HALF, dgelu=HALF, dgrad=HALF, dW2=HALF, dW1=HALF)),
    (1544, 1544, (1409, 897), 1500, None, 0, 0, dict(second=HALF, dgelu=HALF, dgrad=HALF, dW2=SMALL, dW1=SMALL)),
    (768, 1032, (700, 513, 640, 641, 1, 0, 257, 384, 385, 128, 129, 639, 577, 576, 512, 64), 700, None, 1, 1,
     dict.fromkeys(GEMMS, LARGE)),
    (768, 1032, (700, 513, 640, 641, 1, 0, 257, 384, 385, 128, 129, 639, 577, 576, 512, 64), 700, None, 0, 0,
     dict.fromkeys(GEMMS, LARGE)),
    (136, 136, (1030, 1025, 1024, 129, 0, 1, 897, 961), 1030, None, 1, 1, dict.fromkeys(GEMMS, SMALL)),
    (136, 136, (1030, 1025, 1024, 129, 0, 1, 897, 961), 1030, None, 0, 0, dict.fromkeys(GEMMS, SMALL)),
    (136, 264, (100,), 100, None, 1, 0, dict.fromkeys(GEMMS[:5], FLAT)),
], ids=["half_gelu", "half", "half_tails", "large_store", "large_add", "small_store", "small_add", "flat"])
def test_expert_ffn_in_every_tile_shape(M, H, counts, Cp, mean, recompute, overwrite, tiles):
    _run("bf16", M, H, counts, Cp, 13, recompute, overwrite, mean, tiles)


# backward's last three GEMMs share a launch where their tiles go together (the tests above: two workgroups per CU, and
# 256 x 256 with 256 x 256 and 256 x 128): flat input-gradient tiles beside large ones, and tiles that do not go together
@pytest.mark.parametrize("recompute,overwrite", [(0, 1), (1, 0)])
@pytest.mark.parametrize("M,H,E,Cp,dgrad,dw", [
    (136, 3080, 16, 70, FLAT, LARGE),
    (136, 520, 64, 257, HALF, LARGE),
    (136, 1032, 32, 257, SMALL, LARGE),         # one workgroup per CU and two: the input gradient by itself
    (1032, 264, 16, 129, HALF, SMALL),
], ids=["flat_large", "half_large", "small_large", "half_small"])
def test_last_gradients_in_one_launch(M, H, E, Cp, dgrad, dw, recompute, overwrite):
    counts = tuple((0, Cp, 1, 64, 65, Cp - 1, 33)[e % 7] for e in range(E))
    dw = dw if overwrite else SMALL              # sums that are added to go into smaller tiles at these sizes
    _run("bf16", M, H, counts, Cp, 17, recompute, overwrite, tiles=dict(dgrad=dgrad, dW2=dw, dW1=dw))


# more rows than the hidden dimension: the weight gradients' tiles come first in that launch
@pytest.mark.parametrize("recompute,overwrite", [(0, 1), (1, 0)])
@pytest.mark.parametrize("M,H,counts,Cp", [(24, 40, (300, 0, 257, 64, 1), 300), (136, 72, (700, 65, 0), 700)], ids=["thin", "wide"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_last_gradients_with_more_rows_than_columns(dtype, M, H, counts, Cp, recompute, overwrite):
    _run(dtype, M, H, counts, Cp, 23, recompute, overwrite)


# 64 x 64 tiles of the second layer: few rows against a long reduction that ends inside a step, columns inside a tile
@pytest.mark.parametrize("M,H,counts,Cp", [
    (296, 1592, (1, 0, 18, 17, 64, 65, 33, 128), 128), (8, 1024, (1, 3), 3), (72, 4104, (129,), 129), (136, 1288, (64, 63, 31, 32), 64),
], ids=["many", "min", "one", "k_tail"])
def test_expert_ffn_in_the_smallest_tiles(M, H, counts, Cp):
    _run("bf16", M, H, counts, Cp, 19, 1, 1, tiles=dict(second=(64, 64)))


# float gradients of more than 2 GiB per expert, with columns that end inside a tile: the offset that stands for "out
# of range" is then smaller than the gradients (the reference takes some 40 GB)
@pytest.mark.parametrize("overwrite", [0, 1])
def test_expert_ffn_with_gradients_above_two_gib(overwrite):
    _run("bf16", 24008, 24008, (5,), 8, 3, 0, overwrite)


# experts smaller than the 256 x 256 tile that they are multiplied in: the tile's last rows belong to the experts
# behind (the last expert's to nobody), whichever rows of theirs hold something
@pytest.mark.parametrize("recompute,overwrite", [(0, 1), (1, 0)])
def test_expert_ffn_with_experts_smaller_than_their_tile(recompute, overwrite):
    counts = tuple([1, 10, 64, 65, 0, 127, 128, 140] + [129 + 5 * e % 12 for e in range(55)] + [129])
    _run("bf16", 768, 3072, counts, 140, 7, recompute, overwrite, tiles=dict.fromkeys(GEMMS[:5], LARGE))


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


# 256 x 256 tiles multiply with another shape of the matrix instruction than the smaller ones: the same products in the same
# order, so that a result does not depend on the tiles that a schedule gives it.  Rows and tiles of 32 k in odd and even
# numbers, dimensions that end inside a step, experts without rows.
@pytest.mark.parametrize("M,H,counts,Cp,mean,overwrite,gemms", [
    (768, 1032, (700, 513, 640, 641, 1, 0, 257, 384, 385, 128, 129, 639, 577, 576, 512, 64), 700, 8, 0, GEMMS),
    (1024, 1032, (65, 33, 32, 225, 256, 700, 0, 449), 700, 100, 1, GEMMS[5:]),
], ids=["all_add", "weight_gradients_store"])
def test_expert_ffn_is_the_same_in_large_and_small_tiles(M, H, counts, Cp, mean, overwrite, gemms):
    from paper_2506_22175_amd import binding as B
    E, d, dt = len(counts), "cuda:0", torch.bfloat16
    g = torch.Generator(d).manual_seed(29)
    x, dy = (torch.randn((E * Cp, M), generator=g, device=d).to(dt) for _ in range(2))
    W1 = (torch.randn((E, M, H), generator=g, device=d) * 0.05).to(dt)
    W2 = (torch.randn((E, H, M), generator=g, device=d) * 0.05).to(dt)
    w = torch.rand((E * Cp,), generator=g, device=d)
    old1, old2 = torch.randn((E, M, H), generator=g, device=d), torch.randn((E, H, M), generator=g, device=d)
    c = torch.tensor([counts], dtype=torch.int32, device=d)
    kept = torch.cat([torch.arange(e * Cp, e * Cp + r, device=d) for e, r in enumerate(counts)])
    padding = torch.ones((E * Cp,), dtype=torch.bool, device=d)
    padding[kept] = False
    for t in (x, dy, w):
        t[padding] = float("nan")
    got = []
    for rows, large in ((Cp, True), (mean, False)):
        cfg = B.make_config(E * rows, M, H, E, 1, Cp / rows, 1, B.MOE_BF16, 0, overwrite)
        assert B.moe_capacity(cfg) == Cp
        assert all((B.moe_gemm_tile(cfg, 0, gemm) == LARGE) == large for gemm in gemms)
        nan = lambda *s, dtype=dt: torch.full(s, float("nan"), dtype=dtype, device=d)  # noqa: E731
        Z, A, DO, dZ, dDI = nan(E * Cp, H), nan(E * Cp, H), nan(E * Cp, M), nan(E * Cp, H), nan(E * Cp, M)
        dW1, dW2 = (nan(E, M, H, dtype=torch.float32), nan(E, H, M, dtype=torch.float32)) if overwrite else (old1.clone(), old2.clone())
        B.moe_expert_ffn_fwd(cfg, 0, x, c, W1, W2, Z, A, DO)
        B.moe_expert_ffn_bwd(cfg, 0, 0, x, Z, dy, c, w, W1, W2, dZ, dDI, dW1, dW2, None)
        torch.cuda.synchronize()
        got.append({"DO": DO[kept], "dZ": dZ[kept], "dDI": dDI[kept], "dW1": dW1, "dW2": dW2})
    for name, value in got[0].items():
        assert bool(torch.isfinite(value).all()) and torch.equal(value, got[1][name]), name
    empty = counts.index(0)
    if overwrite:
        assert not bool(got[0]["dW1"][empty].any()) and not bool(got[0]["dW2"][empty].any())
    else:
        assert torch.equal(got[0]["dW1"][empty], old1[empty]) and torch.equal(got[0]["dW2"][empty], old2[empty])
