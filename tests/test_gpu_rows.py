"""Slot assignment and the row permutations by themselves, at the edges of their launches: assignments around the number
that one kernel counts by itself, workgroups of 1024 tokens that end early, every number of choices, rows that end
inside a wavefront's piece; and the whole step with its combine in backward's dispatch."""
import numpy as np
import pytest
import torch

from paper_2506_22175_amd import binding as B

pytestmark = pytest.mark.gpu

D = "cuda:0"


def _choices(T, E, k, seed):
    """k different experts per token, the low ones more often."""
    rng = np.random.default_rng(seed)
    p = 1.0 / (np.arange(E) + 1.0)
    return np.argsort(-(np.log(p) + rng.gumbel(size=(T, E))), axis=1)[:, :k].astype(np.int32)


def _slots(idx, n, E, Cp):
    """Choice-major, then token order, inside each partition."""
    T, k = idx.shape
    Tp = T // n
    slot, counts = np.full((T, k), -1, np.int32), np.zeros((n, E), np.int32)
    for p in range(n):
        for j in range(k):
            for t in range(p * Tp, (p + 1) * Tp):
                e = idx[t, j]
                if counts[p, e] < Cp:
                    slot[t, j] = e * Cp + counts[p, e]
                    counts[p, e] += 1
    return slot, counts


@pytest.mark.parametrize("T,n,E,k", [
    (1, 1, 1, 1), (63, 1, 3, 2), (64, 1, 64, 8), (384, 1, 9, 8), (385, 1, 9, 8), (1023, 1, 33, 3), (1024, 1, 33, 3),
    (1025, 1, 33, 3), (3072, 1, 64, 1), (3073, 1, 64, 1), (6144, 2, 64, 1), (5120, 1, 2, 2), (9000, 3, 17, 4),
    (33000, 1, 16, 2),
])
def test_slots(T, n, E, k):
    cfg = B.make_config(T, 8, 8, E, k, 0.75, n, B.MOE_BF16, 0)
    Cp = B.moe_capacity(cfg)
    idx = _choices(T, E, k, T + E)
    ref, counts = _slots(idx, n, E, Cp)
    assert (ref < 0).any() or k == E
    w = np.random.default_rng(1).random((T, k), dtype=np.float32)
    ti, tw = torch.from_numpy(idx).to(D), torch.from_numpy(w).to(D)
    slot, c = torch.full((T, k), -9, dtype=torch.int32, device=D), torch.full((n, E), -9, dtype=torch.int32, device=D)
    slot_w = torch.full((n * E * Cp,), -1.0, device=D)
    scratch = torch.full((B.moe_slot_scratch_bytes(cfg),), 0xFF, dtype=torch.uint8, device=D)
    B.moe_assign_slots(cfg, ti, tw, slot, c, slot_w, scratch)
    assert np.array_equal(slot.cpu().numpy(), ref) and np.array_equal(c.cpu().numpy(), counts)
    want = np.full((n * E * Cp,), -1.0, np.float32)
    part = np.arange(T)[:, None] // (T // n) * (E * Cp) + ref
    want[part[ref >= 0]] = w[ref >= 0]
    assert np.array_equal(slot_w.cpu().numpy(), want)


@pytest.mark.parametrize("M", [8, 520, 2056])
@pytest.mark.parametrize("k", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_dispatch_with_row_dots(dtype, k, M):
    """Rows land bit for bit and nowhere else; the dots are float sums of M products: M units of rounding at most."""
    T, n, E = 52, 2, 9
    dt, mt = (torch.bfloat16, B.MOE_BF16) if dtype == "bf16" else (torch.float32, B.MOE_F32)
    cfg = B.make_config(T, M, 8, E, k, 0.7, n, mt, 0)
    Cp = B.moe_capacity(cfg)
    ref, _ = _slots(_choices(T, E, k, k), n, E, Cp)
    assert (ref < 0).any()
    g = torch.Generator(D).manual_seed(M)
    src = torch.randn((T, M), generator=g, device=D).to(dt)
    saved = torch.randn((E * Cp, M), generator=g, device=D).to(dt)
    slot = torch.from_numpy(ref).to(D)
    dw = torch.full((T, k), float("nan"), device=D)
    for p in range(n):
        held = torch.zeros((E * Cp,), dtype=torch.bool, device=D)
        q = slice(p * T // n, (p + 1) * T // n)
        s = slot[q].long()
        held[s[s >= 0]] = True
        kept = saved.clone()
        kept[~held] = float("nan")
        for with_dw in (False, True):
            out = torch.full((E * Cp, M), float("nan"), device=D).to(dt)
            B.moe_dispatch(cfg, p, src, slot, out, kept if with_dw else None, dw if with_dw else None)
            want = torch.full_like(out, float("nan"))
            t, j = torch.nonzero(s >= 0, as_tuple=True)
            want[s[t, j]] = src[q][t]
            assert torch.equal(out.isnan(), want.isnan()) and torch.equal(out[held], want[held])
        rows = torch.where((s >= 0)[..., None], saved[s.clamp(min=0)].double(), 0.0)
        prod = src[q].double()[:, None] * rows
        err = (dw[q].double() - prod.sum(2)).abs()
        assert bool((err <= prod.abs().sum(2) * M * 2.0 ** -24).all())


@pytest.mark.parametrize("T,M,k,dtype", [
    (2047, 8, 3, "bf16"), (2049, 520, 1, "bf16"), (2049, 2040, 2, "bf16"), (2048, 1032, 4, "f32"), (2049, 1016, 4, "f32"),
    (2049, 1032, 2, "f32"), (2049, 1032, 3, "f32"), (2100, 512, 5, "bf16"), (2100, 504, 8, "bf16"), (2100, 776, 7, "bf16"), (2100, 392, 6, "f32"),
])
def test_dispatch_of_many_tokens(T, M, k, dtype):
    """Around the numbers of tokens, row lengths and choices by which dispatch changes the form of its stores: rows land bit
    for bit and nowhere else."""
    E, dt, mt = 9, *((torch.bfloat16, B.MOE_BF16) if dtype == "bf16" else (torch.float32, B.MOE_F32))
    cfg = B.make_config(T, M, 8, E, k, 0.7, 1, mt, 0)
    Cp = B.moe_capacity(cfg)
    ref, _ = _slots(_choices(T, E, k, k), 1, E, Cp)
    assert (ref < 0).any()
    src = torch.randn((T, M), generator=torch.Generator(D).manual_seed(M), device=D).to(dt)
    slot = torch.from_numpy(ref).to(D)
    out = torch.full((E * Cp + 8, M), float("nan"), device=D).to(dt)
    B.moe_dispatch(cfg, 0, src, slot, out[:E * Cp])
    want = torch.full_like(out, float("nan"))
    t, j = torch.nonzero(slot >= 0, as_tuple=True)
    want[slot[t, j].long()] = src[t]
    assert torch.equal(out.isnan(), want.isnan()) and torch.equal(out.nan_to_num(), want.nan_to_num())


@pytest.mark.parametrize("T,M,H,E,k,n,dtype,mode,fuse", [
    (120, 72, 136, 5, 3, 5, "bf16", 0, 0), (96, 520, 264, 9, 8, 1, "bf16", 0, 1), (90, 264, 136, 3, 1, 3, "f32", 0, 0),
    (128, 2056, 72, 4, 2, 2, "bf16", 0, 0), (128, 2056, 72, 4, 2, 2, "bf16", 2, 0), (96, 520, 264, 9, 8, 1, "bf16", 1, 1),
    (90, 264, 136, 3, 3, 2, "f32", 2, 1), (90, 264, 136, 7, 5, 1, "f32", 1, 0), (120, 72, 136, 5, 3, 5, "bf16", 2, 0),
])
def test_step_equals_its_two_halves(T, M, H, E, k, n, dtype, mode, fuse):
    """In a whole step with a T_DO buffer for every partition the combine shares backward's dispatch of dy, which may take
    the rows' place: the same bits as by itself."""
    from paper_2506_22175_amd import runner, synth
    s = synth.custom_shape(T, M, H, E, k, 0.75, dtype=dtype, x_std=1.0, w_std=0.05, name="halves")
    st = runner.LayerState(T, M, H, E, k, 0.75, n, dtype, mode, grad_overwrite=1, fuse_gather=fuse)
    assert B.moe_layer_streams(st.cfg) == 1
    st.upload(synth.make_inputs(s, seed=5))
    out = []
    for halves in (False, True):
        st.poison()
        if halves:
            st.forward()
            st.backward()
        else:
            st.step()
        out.append(st.results())
    assert (out[0]["slot"] < 0).any()
    for name in ("y", "dx", "dWg", "dW1", "dW2"):
        assert np.isfinite(out[0][name]).all() and np.array_equal(out[0][name], out[1][name]), name


@pytest.mark.parametrize("T,M,H,E,k,n,dtype,mode,opts", [
    (1024, 72, 136, 32, 2, 4, "bf16", 0, {}),                                 # two partitions fill the 64 expert numbers
    (1023, 72, 136, 21, 2, 3, "bf16", 2, dict(wgrad_group=3)),                # three in forward
    (1056, 72, 264, 33, 2, 4, "bf16", 1, dict(wgrad_group=2)),                # one at a time
    (512, 136, 72, 5, 1, 8, "bf16", 2, dict(fuse_gather=1, fuse_combine=1, wgrad_group=4)),
    (512, 136, 72, 5, 1, 8, "f32", 0, dict(fuse_gather=1, fuse_combine=1, wgrad_group=2)),
    (2048, 512, 1024, 4, 2, 2, "bf16", 0, {}),                                # 128 x 128 instead of one partition's 64 x 128
    (1600, 1032, 2056, 4, 2, 2, "bf16", 1, {}),
    (4096, 24, 40, 3, 2, 2, "bf16", 2, {}),                                   # the weight gradients' tiles before the input gradient's
    (4096, 24, 40, 3, 2, 2, "f32", 1, {}),
    (600, 72, 1032, 3, 2, 3, "f32", 0, {}),                                   # no room for a second activation buffer
], ids=["two", "three", "one", "gathered_combined", "gathered_combined_f32", "other_tiles", "other_tiles_shared", "long_rows", "long_rows_f32", "no_room"])
def test_gemms_of_several_partitions_in_one_launch(T, M, H, E, k, n, dtype, mode, opts):
    """One stream runs the GEMMs of several partitions at once where their buffers allow it, two streams one by one: the
    same bits."""
    from paper_2506_22175_amd import runner, synth
    s = synth.custom_shape(T, M, H, E, k, 0.8, dtype=dtype, x_std=1.0, w_std=0.05, zipf_s=1.2, zipf_tau=0.3, name="batch")
    d = synth.make_inputs(s, seed=6)
    one = runner.run_layer_step(s, d, n, mode, second_stream=False, grad_overwrite=1, **opts)
    two = runner.run_layer_step(s, d, n, mode, grad_overwrite=1, gemm_free_cus=8, **opts)
    assert (one["slot"] < 0).any()
    for name in ("y", "dx", "dWg", "dW1", "dW2", "slot", "counts"):
        assert np.isfinite(one[name]).all() and np.array_equal(one[name], two[name]), name


@pytest.mark.parametrize("T,M,H,E,n,tile", [
    (404, 136, 1288, 4, 2, (64, 64)), (130, 72, 2056, 3, 1, (64, 64)), (3000, 1544, 1544, 2, 1, (256, 128)),
])
def test_scattered_rows_in_other_tiles(T, M, H, E, n, tile):
    """The fused combine from 64 x 64 and 256 x 128 tiles: what the combine kernel gives up to one rounding, zeros for
    dropped tokens."""
    from paper_2506_22175_amd import runner, synth
    s = synth.custom_shape(T, M, H, E, 1, 0.9, dtype="bf16", x_std=1.0, w_std=0.05, zipf_s=1.2, zipf_tau=0.5, name="k1")
    d = synth.make_inputs(s, seed=17)
    cfg = B.make_config(T, M, H, E, 1, 0.9, n, B.MOE_BF16, 0, 1, fuse_combine=1)
    assert B.moe_gemm_tile(cfg, 0, "second") == tile
    plain = runner.run_layer_step(s, d, n, 0, grad_overwrite=1)
    fused = runner.run_layer_step(s, d, n, 0, grad_overwrite=1, fuse_combine=1)
    dropped = (fused["slot"] < 0).all(axis=1)
    assert dropped.any() and np.all(fused["y"][dropped] == 0.0)
    # row by row: both round w * row to bfloat16 (2^-8 of it), the plain combine after a rounding of the row
    scale = np.abs(plain["y"]).max(axis=1, keepdims=True)
    assert np.all(np.abs(fused["y"] - plain["y"]) <= 2.0 ** -6 * scale)
    assert np.array_equal(fused["dW1"], plain["dW1"])
