"""GEMM forms that only the layer calls reach - the scattered store of the fused combine, rows gathered from the
input, weight gradients over several partitions at once - in every tile shape of the bfloat16 GEMM."""
import numpy as np
import pytest

from paper_2506_22175_amd import binding as B
from paper_2506_22175_amd import runner, synth

pytestmark = pytest.mark.gpu

LARGE, HALF, SMALL, FLAT = (256, 256), (256, 128), (128, 128), (64, 128)


def _relerr(a, ref):
    assert np.isfinite(a).all()
    return np.abs(a - ref).max() / np.abs(ref).max()


@pytest.mark.parametrize("T,M,H,E,n,second,first", [
    (11200, 768, 1032, 16, 1, LARGE, LARGE),        # 700 rows per expert and less
    (1280, 2056, 264, 16, 1, LARGE, FLAT),          # 80: the tile is three times as high as an expert
    (6000, 1544, 1544, 2, 2, HALF, SMALL),
    (2048, 784, 1312, 16, 1, SMALL, HALF),
    (8240, 136, 136, 8, 1, SMALL, SMALL),
    (404, 136, 264, 4, 2, FLAT, FLAT),
], ids=["large", "large_few_rows", "half", "half_gathered", "small", "flat"])
def test_scattered_and_gathered_rows(T, M, H, E, n, second, first):
    """k = 1, mode 0: the fused combine gives the plain one's result up to the rounding that it saves, zeros for dropped
    tokens (the gate is skewed enough to have some); gathering the first GEMM's rows changes no bit."""
    cf = 1.25 if first == HALF else 1.0
    s = synth.custom_shape(T, M, H, E, 1, cf, dtype="bf16", x_std=1.0, w_std=0.05, zipf_s=1.2, zipf_tau=0.5,
                           name="k1")
    d = synth.make_inputs(s, seed=17)
    cfg = B.make_config(T, M, H, E, 1, cf, n, B.MOE_BF16, 0, 1, fuse_combine=1)
    assert B.moe_gemm_tile(cfg, 0, "second") == second and B.moe_gemm_tile(cfg, 0, "first") == first
    # (two streams: one partition per launch, whose tiles the above are)
    two = dict(grad_overwrite=1, gemm_free_cus=8 if n > 1 else 0)
    plain = runner.run_layer_step(s, d, n, 0, **two)
    fused = runner.run_layer_step(s, d, n, 0, fuse_combine=1, **two)
    gathered = runner.run_layer_step(s, d, n, 0, fuse_combine=1, fuse_gather=1, **two)
    for k_ in ("y", "dx", "dWg", "dW1", "dW2", "slot", "counts"):
        assert np.array_equal(gathered[k_], fused[k_]), k_
    dropped = (fused["slot"] < 0).all(axis=1)
    assert dropped.any() and not dropped.all()
    assert np.all(fused["y"][dropped] == 0.0) and np.all(np.abs(fused["y"][~dropped]).max(axis=1) > 0.0)
    # row by row: both round w * row to bfloat16 (2^-8 of it), the plain combine after a rounding of the row
    scale = np.abs(plain["y"]).max(axis=1, keepdims=True)
    assert np.all(np.abs(fused["y"] - plain["y"]) <= 2.0 ** -6 * scale)
    for k_ in ("dW1", "dW2"):
        assert np.array_equal(fused[k_], plain[k_]), k_


@pytest.mark.parametrize("M,H,E,mean,cf,G,overwrite,tile", [
    (136, 2832, 6, 1787, 1.0, 8, 0, HALF),
    (136, 2832, 6, 1787, 1.0, 8, 1, HALF),
    (136, 3232, 5, 131, 1.25, 8, 1, HALF),          # ranges of a step of 64 and a few rows more
    (264, 1032, 4, 700, 1.0, 3, 0, SMALL),
    (768, 1032, 16, 700, 1.0, 3, 0, LARGE),
    (768, 1032, 16, 700, 1.0, 3, 1, LARGE),         # experts without a row in any partition of a group, ranges of a few rows
], ids=["half_add", "half_store", "half_short_ranges", "small_add", "large_add", "large_store"])
def test_weight_gradients_over_several_partitions(M, H, E, mean, cf, G, overwrite, tile):
    """Skewed loads: ranges of every length between partitions without a row for the expert.  One reduction over a
    group's rows gives what adding partition by partition gives, up to the rounding of float sums."""
    n = 8
    T = n * E * mean
    s = synth.custom_shape(T, M, H, E, 1, cf, dtype="bf16", x_std=1.0, w_std=0.05, zipf_s=1.2, zipf_tau=2.0 if M < 200 else 3.0, name="skew")
    d = synth.make_inputs(s, seed=19)
    last = (n - 1) // G * G
    cfg = B.make_config(T, M, H, E, 1, cf, n, B.MOE_BF16, 0, overwrite, wgrad_group=G)
    for gemm in ("dW1", "dW2"):
        assert B.moe_gemm_tile(cfg, 0, gemm) == tile and B.moe_gemm_tile(cfg, n - 1, gemm) == B.moe_gemm_tile(cfg, last, gemm)
    one = runner.run_layer_step(s, d, n, 0, grad_overwrite=overwrite)
    group = runner.run_layer_step(s, d, n, 0, grad_overwrite=overwrite, wgrad_group=G)
    c = one["counts"]
    assert (c == 0).any() and (c % 64 != 0).any()
    if tile == LARGE:
        tiles = (c + 31) // 32
        assert (c[:G].sum(axis=0) == 0).any() and (c[c > 0] < 32).any() and (tiles % 2 == 1).any() and ((tiles > 0) & (tiles % 2 == 0)).any()
    for k_ in ("y", "dx", "counts", "slot"):
        assert np.array_equal(group[k_], one[k_]), k_
    # the terms of an element are alike in size and of either sign: r of them sum to about sqrt(r) of one and round
    # to 2^-24 of a partial sum each, at most r^1.5 of that in all; a row lost or counted twice would show as 1/sqrt(r)
    r = int(c.sum(axis=0).max())
    for k_ in ("dW1", "dW2"):
        assert _relerr(group[k_], one[k_]) <= max(1e-5, r ** 1.5 * 2.0 ** -24 / 8), k_


@pytest.mark.parametrize("M,H", [(768, 1032), (1032, 1288)])
@pytest.mark.parametrize("overwrite", [0, 1])
def test_weight_gradients_do_not_depend_on_the_partitions(M, H, overwrite):
    """Every partition's rows of an expert are whole tiles of 32 k, in odd and even numbers and none, so that one reduction over
    eight partitions adds the same products in the same order as one over all rows at once.  The other GEMMs take different
    tiles for the two."""
    E, n = 16, 8
    rows = np.array([0, 32, 64, 96, 128, 160, 192, 224, 0, 32, 320, 96, 128, 32, 416, 128])
    T = n * int(rows.sum())
    s = synth.custom_shape(T, M, H, E, 1, 416 / 128, dtype="bf16", x_std=1.0, w_std=0.05, name="blocks")
    d = synth.make_inputs(s, seed=31)
    rng = np.random.default_rng(31)
    counts = np.stack([np.roll(rows, p) for p in range(n)])
    chosen = np.concatenate([rng.permutation(np.repeat(np.arange(E), counts[p])) for p in range(n)])
    d["x"][:, :E] = 8.0 * np.eye(E, dtype=np.float32)[chosen]
    d["Wg"][:E] = 4.0 * np.eye(E, dtype=np.float32)
    got = []
    for parts, group in ((n, 8), (1, 0)):
        cfg = B.make_config(T, M, H, E, 1, 416 / 128, parts, B.MOE_BF16, 0, overwrite, wgrad_group=group)
        assert all(B.moe_gemm_tile(cfg, parts - 1, gemm) == LARGE for gemm in ("dW1", "dW2"))
        got.append(runner.run_layer_step(s, d, parts, 0, grad_overwrite=overwrite, wgrad_group=group))
    assert np.array_equal(got[0]["counts"], counts) and np.array_equal(got[1]["counts"][0], counts.sum(axis=0))
    for k_ in ("y", "dx", "dW1", "dW2"):
        assert np.isfinite(got[0][k_]).all() and np.array_equal(got[0][k_], got[1][k_]), k_
