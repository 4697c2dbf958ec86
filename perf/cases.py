"""What the MoE layer is used for, as cases that can be timed and compared.

A case is one of four kinds of call, all through the package's public entry points:

  step     one training step of the layer (forward and backward, LayerState.step)
  forward  the forward half alone, as an evaluation pass runs it (LayerState.forward)
  ffn      the expert FFN of one partition, forward then backward (moe_expert_ffn_fwd / _bwd)
  rows     everything around the experts: gate, slots, dispatch and combine, then dispatch of the
           upstream gradient, gate backward and dispatch backward, for every partition

Sizes are those of the workloads in paper_2506_22175_amd/synth.py, the layers of the paper's Table III
(model / hidden dimension 768/3072 with 64 experts, 1024/4096, 2048/8192), the shapes of the tests, and
generic odd sizes between them.
"""
import math

import torch

from paper_2506_22175_amd import binding as B
from paper_2506_22175_amd import runner

DEVICE = "cuda:0"
TORCH_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
MOE_DT = {"f32": B.MOE_F32, "bf16": B.MOE_BF16}

DEFAULTS = dict(kind="step", T=4096, M=512, H=2048, E=8, k=2, cf=1.25, n=1, dtype="bf16", reuse=0, renorm=0,
                fuse_gather=0, fuse_combine=0, wgrad_group=0, x_std=1.0, w_std=0.02, zipf_s=0.0, zipf_tau=0.0)


def _case(name=None, **kw):
    c = dict(DEFAULTS, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest layer of the workloads: launches and their latency are all there is; float32
        _case("tiny_step", T=256, M=64, H=128, E=4, k=1, dtype="f32", x_std=0.02),
        # a few sequences' last tokens through a mid-size layer, forward only: the weights are read for
        # a handful of rows each
        _case("few_forward", kind="forward", T=64, M=1024, H=4096, E=8),
        # a small layer's training step, two micro-batches, activations recomputed
        _case("small_step", T=4096, M=512, H=2048, E=8, n=2, reuse=2),
        # the mid-size layer in four micro-batches with shared buffers and recomputation
        _case("gpt_step", T=16384, M=1024, H=4096, E=8, n=4, reuse=2),
        # the same layer's evaluation pass in one piece
        _case("gpt_forward", kind="forward", T=16384, M=1024, H=4096, E=8),
        # the large layer's training step, the configuration of the headline number
        _case("large_step", T=32768, M=2048, H=8192, E=16, cf=1.0, n=2, reuse=2),
        # a skewed gate: drops, padding and experts of very different sizes; shared buffers
        _case("skewed_step", T=16384, M=1024, H=4096, E=16, cf=2.0, n=4, reuse=1, zipf_s=1.2, zipf_tau=0.390625),
        # odd sizes in every dimension, three choices per token with renormalised weights, three micro-batches
        _case("ragged_step", T=3003, M=776, H=2600, E=6, k=3, cf=1.0, n=3, renorm=1),
        # a small layer in float32
        _case("f32_step", T=2048, M=512, H=2048, E=8, n=2, dtype="f32"),
        # the paper's own gate (one choice) over its 64 experts of 768/3072, with the fused gather and combine
        _case("top1_step", T=8192, M=768, H=3072, E=64, k=1, n=2, reuse=2, fuse_gather=1, fuse_combine=1, wgrad_group=2),
        # the experts of one micro-batch alone, ragged loads
        _case("expert_ffn", kind="ffn", T=6000, M=1024, H=4096, E=8, cf=1.0),
        # the gate and the row permutations of the large layer, without the experts
        _case("gate_and_rows", kind="rows", T=32768, M=2048, H=64, E=16, cf=1.0, n=2),
    ]


def _flops(c):
    return 12.0 * min(c["T"] * c["k"], c["n"] * c["E"] * _capacity(c)) * c["M"] * c["H"]


def _capacity(c):
    return max(1, math.ceil(c["cf"] * c["k"] * (c["T"] // c["n"]) / c["E"]))


def _loads(c):
    """Rows of each expert in an "ffn" case: between 0.6 of the capacity and all of it, spread evenly."""
    Cp = _capacity(c)
    return [max(1, int(Cp * (0.6 + 0.4 * ((e + 1) * 0.6180339887 % 1.0)))) for e in range(c["E"])]


def draw(rng):
    largest, f32_most = 12.0 * 65536 * 2048 * 8192, 4 * 12.0 * 4096 * 512 * 2048
    while True:
        logu = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
        kind = rng.choice(["step", "step", "step", "forward", "ffn", "rows"])
        E = rng.choice([1, 2, 4, 5, 8, 8, 12, 16, 16, 32, 64]) if kind != "ffn" else rng.choice([1, 2, 4, 5, 8, 12, 16])
        k = rng.choice([q for q in (1, 1, 2, 2, 3, 4) if q <= E])
        n = 1 if kind == "ffn" else rng.choice([1, 1, 2, 2, 3, 4, 8])
        M = max(64, logu(64, 2048) // 8 * 8)
        if rng.random() < 0.5:
            M = max(64, M // 64 * 64)
        H = min(8192, int(M * rng.choice([1.5, 2, 3, 4, 4])) // 8 * 8)
        T = max(n, logu(64, 32768) // n * n)
        c = _case(kind=kind, T=T, M=M, H=H if kind != "rows" else 64, E=E, k=k, n=n,
                  cf=rng.choice([0.5, 1.0, 1.0, 1.25, 1.25, 2.0]),
                  dtype=rng.choice(["bf16", "bf16", "bf16", "bf16", "f32"]),
                  reuse=rng.choice([0, 1, 2, 2]) if kind == "step" else 0,
                  renorm=int(rng.random() < 0.25) if k > 1 else 0)
        if kind == "step":
            c["wgrad_group"] = rng.choice([0, 0, 2, 4]) if n > 1 else 0
            c["fuse_gather"] = int(rng.random() < 0.25)
            c["fuse_combine"] = int(k == 1 and rng.random() < 0.5)
        if E > 2 and kind != "ffn" and rng.random() < 0.3:
            c["zipf_s"], c["zipf_tau"] = 1.2, 0.390625
        if E * M * H > 16 * 2048 * 8192:
            continue
        if _flops(c) <= (largest if c["dtype"] == "bf16" else f32_most):
            return c


# ---- inputs -----------------------------------------------------------------------------------

def _normal(g, dims, std, dt):
    return (torch.randn(dims, generator=g, device=DEVICE, dtype=torch.float32) * std).to(dt)


def _inputs(c, seed):
    """Everything random, from the seed alone, on the GPU."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    dt, T, M, H, E = TORCH_DT[c["dtype"]], c["T"], c["M"], c["H"], c["E"]
    i = {"x": _normal(g, (T, M), c["x_std"], dt), "Wg": _normal(g, (M, E), c["w_std"], dt)}
    i["dy"] = _normal(g, (T, M), 1.0, dt)
    if c["kind"] != "rows":
        i["W1"] = _normal(g, (E, M, H), c["w_std"], dt)
        i["W2"] = _normal(g, (E, H, M), c["w_std"], dt)
    i["gate_bias"] = None
    if c["zipf_s"]:
        p = (torch.arange(E, dtype=torch.float64) + 1.0) ** (-c["zipf_s"])
        i["gate_bias"] = (c["zipf_tau"] * torch.log(p / p.sum())).to(torch.float32).to(DEVICE)
    if c["kind"] == "ffn":
        # what a partition's experts are handed: rows of x and of dy in expert order, some experts short of
        # their capacity, and each row's combine weight
        Cp = _capacity(c)
        i["DI"] = _normal(g, (E * Cp, M), c["x_std"], dt)
        i["dDO"] = _normal(g, (E * Cp, M), 1.0, dt)
        i["counts"] = torch.tensor([_loads(c)], dtype=torch.int32, device=DEVICE)
        i["slot_w"] = torch.rand((E * Cp,), generator=g, device=DEVICE, dtype=torch.float32) * 0.5 + 0.05
    return i


def _config(c):
    return B.make_config(c["T"], c["M"], c["H"], c["E"], c["k"], c["cf"], c["n"], MOE_DT[c["dtype"]], c["reuse"], 1,
                         c["renorm"], c["fuse_gather"], c["wgrad_group"], 0, c["fuse_combine"])


def prepare(case, seed):
    c = case
    i = _inputs(c, seed)
    dt, T, M, H, E, k, n = TORCH_DT[c["dtype"]], c["T"], c["M"], c["H"], c["E"], c["k"], c["n"]
    if c["kind"] in ("step", "forward"):
        st = runner.LayerState(T, M, H, E, k, c["cf"], n, c["dtype"], c["reuse"], DEVICE, grad_overwrite=1,
                               gate_renormalize=c["renorm"], fuse_gather=c["fuse_gather"],
                               wgrad_group=c["wgrad_group"], fuse_combine=c["fuse_combine"])
        for name in ("x", "dy", "Wg", "W1", "W2", "gate_bias"):
            st.inputs[name] = i[name]
        out = {"y": st.y, "logits": st.logits, "topk_idx": st.topk_idx, "topk_w": st.topk_w, "slot": st.slot,
               "counts": st.counts}
        if c["kind"] == "step":
            out.update(dx=st.dx, dWg=st.dWg, dW1=st.dW1, dW2=st.dW2)
        return {"kind": c["kind"], "layer": st, "out": out}
    cfg = _config(c)
    Cp = _capacity(c)
    empty = lambda *dims, dtype=dt: torch.empty(dims, device=DEVICE, dtype=dtype)  # noqa: E731
    s = {"kind": c["kind"], "cfg": cfg, "n": n, "in": i}
    if c["kind"] == "ffn":
        s.update(Z=empty(E * Cp, H), A=empty(E * Cp, H), DO=empty(E * Cp, M), dZ=empty(E * Cp, H), dDI=empty(E * Cp, M),
                 dW1=empty(E, M, H, dtype=torch.float32), dW2=empty(E, H, M, dtype=torch.float32))
        # the rows that hold something, expert by expert
        kept = [slice(e * Cp, e * Cp + r) for e, r in enumerate(_loads(c))]
        s["out"] = {"DO": [s["DO"][q] for q in kept], "dDI": [s["dDI"][q] for q in kept], "dW1": s["dW1"], "dW2": s["dW2"]}
        return s
    f32, i32 = torch.float32, torch.int32
    s.update(DI=[empty(E * Cp, M) for _ in range(n)], dDO=[empty(E * Cp, M) for _ in range(n)],
             slot_scratch=empty(max(1, B.moe_slot_scratch_bytes(cfg)), dtype=torch.uint8),
             gate_scratch=empty(max(1, B.moe_gate_scratch_bytes(cfg)), dtype=torch.uint8))
    s["out"] = {"logits": empty(T, E, dtype=f32), "topk_idx": empty(T, k, dtype=i32), "topk_w": empty(T, k, dtype=f32),
                "slot": empty(T, k, dtype=i32), "counts": empty(n, E, dtype=i32), "y": empty(T, M), "dx": empty(T, M),
                "dw": empty(T, k, dtype=f32), "dL": empty(T, E, dtype=f32), "dWg": empty(M, E, dtype=f32)}
    return s


def run(state):
    s = state
    if s["kind"] == "step":
        s["layer"].step()
        return s["out"]
    if s["kind"] == "forward":
        s["layer"].forward()
        return s["out"]
    cfg, i, o = s["cfg"], s["in"], s["out"]
    if s["kind"] == "ffn":
        B.moe_expert_ffn_fwd(cfg, 0, i["DI"], i["counts"], i["W1"], i["W2"], s["Z"], s["A"], s["DO"])
        B.moe_expert_ffn_bwd(cfg, 0, 0, i["DI"], s["Z"], i["dDO"], i["counts"], i["slot_w"], i["W1"], i["W2"], s["dZ"],
                             s["dDI"], s["dW1"], s["dW2"], None)
        return o
    B.moe_route(cfg, i["x"], i["Wg"], i["gate_bias"], o["logits"], o["topk_idx"], o["topk_w"])
    B.moe_assign_slots(cfg, o["topk_idx"], o["topk_w"], o["slot"], o["counts"], None, s["slot_scratch"])
    for p in range(s["n"]):
        B.moe_dispatch(cfg, p, i["x"], o["slot"], s["DI"][p])
        B.moe_combine(cfg, p, s["DI"][p], o["slot"], o["topk_w"], o["y"])
    for p in range(s["n"]):
        B.moe_dispatch(cfg, p, i["dy"], o["slot"], s["dDO"][p], s["DI"][p], o["dw"])
        B.moe_gate_bwd(cfg, p, i["x"], o["logits"], o["topk_idx"], o["slot"], o["dw"], None, o["dL"], o["dWg"],
                       s["gate_scratch"])
        B.moe_dispatch_bwd(cfg, p, s["dDO"][p], o["slot"], o["dL"], i["Wg"], o["dx"])
    return o


# ---- what a pass cannot do without ----------------------------------------------------------------

def work(case):
    """Model floating-point operations (no recomputation, kept rows only, none of the padding) and bytes of
    every input read once and every output written once."""
    c = case
    T, M, H, E, k = c["T"], c["M"], c["H"], c["E"], c["k"]
    es = 2 if c["dtype"] == "bf16" else 4
    R = min(T * k, c["n"] * E * _capacity(c))
    gate = 2.0 * T * M * E
    routing = T * E * 4 + T * k * 12
    if c["kind"] == "ffn":
        R = sum(_loads(c))
        return {"flops": 12.0 * R * M * H, "bytes": 4 * R * M * es + 2 * E * M * H * (es + 4)}
    if c["kind"] == "rows":
        return {"flops": 3 * gate + 6.0 * R * M, "bytes": 4 * T * M * es + 4 * R * M * es + M * E * (es + 4) + routing}
    if c["kind"] == "forward":
        return {"flops": 4.0 * R * M * H + gate, "bytes": 2 * T * M * es + min(E, R) * 2 * M * H * es + M * E * es + routing}
    return {"flops": 12.0 * R * M * H + 3 * gate, "bytes": 4 * T * M * es + 2 * E * M * H * (es + 4) + M * E * (es + 4) + routing}


def tolerance(case):
    # bfloat16: every stored activation is rounded to 8 bits of mantissa, and a row passes four such
    # roundings (2.6e-3 to 3.6e-3 against 64 bits on every listed case); float32: sums of up to 8192
    # products in another order (up to 1e-6 against 64 bits at 2048 products)
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    return {"rel": 1.2e-2, "max": 0.1}


# ---- the same in 64 bits ----------------------------------------------------------------------------

def _gelu(z):
    cdf = 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0)))
    return z * cdf, cdf + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)


def exact(case, seed):
    c = case
    i = {name: (v.double() if v is not None and v.is_floating_point() and name not in ("W1", "W2") else v)
         for name, v in _inputs(c, seed).items()}
    T, M, H, E, k, n = c["T"], c["M"], c["H"], c["E"], c["k"], c["n"]
    Cp = _capacity(c)
    f64 = torch.float64
    if c["kind"] == "ffn":
        rows = _loads(c)
        out = {"DO": [], "dDI": [], "dW1": torch.zeros((E, M, H), dtype=f64, device=DEVICE),
               "dW2": torch.zeros((E, H, M), dtype=f64, device=DEVICE)}
        for e in range(E):
            q = slice(e * Cp, e * Cp + rows[e])
            W1, W2, x, dy, w = i["W1"][e].double(), i["W2"][e].double(), i["DI"][q], i["dDO"][q], i["slot_w"][q, None]
            z = x @ W1
            a, da = _gelu(z)
            out["DO"].append(a @ W2)
            dz = w * (dy @ W2.t()) * da
            out["dDI"].append(dz @ W1.t())
            out["dW1"][e] = x.t() @ dz
            out["dW2"][e] = (w * a).t() @ dy
        return out

    # gate
    logits = i["x"] @ i["Wg"]
    if i["gate_bias"] is not None:
        logits = logits + i["gate_bias"]
    prob = torch.softmax(logits, 1)
    idx = torch.sort(logits, dim=1, descending=True, stable=True)[1][:, :k]
    chosen = prob.gather(1, idx)
    w = chosen / chosen.sum(1, keepdim=True) if c["renorm"] else chosen
    # which assignments are kept: choice-major order inside each partition, Cp rows per expert
    Tp = T // n
    by_choice = idx.reshape(n, Tp, k).transpose(1, 2).reshape(n, k * Tp)
    one = torch.nn.functional.one_hot(by_choice, E)
    place = (one.cumsum(1) * one).sum(2) - 1
    kept = (place < Cp).reshape(n, k, Tp).transpose(1, 2).reshape(T, k)

    y = torch.zeros((T, M), dtype=f64, device=DEVICE)
    dx = torch.zeros((T, M), dtype=f64, device=DEVICE)
    dw = torch.zeros((T, k), dtype=f64, device=DEVICE)
    backward = c["kind"] in ("step", "rows")
    out = {"logits": logits, "topk_idx": None, "topk_w": w, "slot": None, "counts": None, "y": y}
    if c["kind"] == "rows":
        y += (w * kept).sum(1, keepdim=True) * i["x"]
        dw += kept * (i["dy"] * i["x"]).sum(1, keepdim=True)
        dx += kept.sum(1, keepdim=True) * i["dy"]
    else:
        if backward:
            out["dW1"] = torch.zeros((E, M, H), dtype=f64, device=DEVICE)
            out["dW2"] = torch.zeros((E, H, M), dtype=f64, device=DEVICE)
        for e in range(E):
            t, j = torch.nonzero((idx == e) & kept, as_tuple=True)
            if t.numel() == 0:
                continue
            W1, W2, x = i["W1"][e].double(), i["W2"][e].double(), i["x"][t]
            z = x @ W1
            a, da = _gelu(z)
            rows = a @ W2
            we = w[t, j][:, None]
            y.index_add_(0, t, we * rows)
            if backward:
                dy = i["dy"][t]
                dw[t, j] = (dy * rows).sum(1)
                dz = we * (dy @ W2.t()) * da
                dx.index_add_(0, t, dz @ W1.t())
                out["dW1"][e] = x.t() @ dz
                out["dW2"][e] = (we * a).t() @ dy
                del dy, dz
            del W1, W2, x, z, a, da, rows
    if not backward:
        return out
    # gate backward: the softmax Jacobian, over all experts or over the chosen ones
    dL = torch.zeros((T, E), dtype=f64, device=DEVICE)
    inner = (dw * w).sum(1, keepdim=True)
    if c["renorm"]:
        dL.scatter_(1, idx, w * (dw - inner))
    else:
        dp = torch.zeros_like(dL).scatter_(1, idx, dw)
        dL += prob * (dp - inner)
    out["dWg"] = i["x"].t() @ dL
    dx += dL @ i["Wg"].t()
    out["dx"] = dx
    if c["kind"] == "rows":
        out["dw"], out["dL"] = dw, dL
    return out
