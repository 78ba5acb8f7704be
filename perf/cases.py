"""The work a program has this framework do, as measurable cases.

A case is a dict of plain values; `kind` picks the path:

  stage     one training iteration of a pipeline stage (begin_iteration, every
            F and B in the planned order) through tpstage.Stage: outputs, input
            gradients and the f32 gradient of every parameter
  attn_fwd  causal attention forward, o and lse
  attn_bwd  causal attention backward, dqkv
  mlp       the GPT MLP forward: up-projection with bias and GeLU (the
            pre-activation kept) and down-projection with bias and residual
  norm      LayerNorm forward and backward of one activation
  swiglu    SwiGLU forward and backward of one activation

Sizes are those of the workloads in paper_2503_03182_amd/configs.py (one or two
layers and micro-batches of each, resident weights), of the repository's tests,
or generic ones between them; sequences need not divide by any tile.
"""
from __future__ import annotations

import math

import torch

from paper_2503_03182_amd import configs
from paper_2503_03182_amd import tpstage as T

_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
_CODE = {"bf16": T.TPS_BF16, "f32": T.TPS_F32}
_EPS = 1e-5
_ROPE = 10000.0


def _stage(name, arch, dtype, layers, hidden, heads, kv, mlp, seq, batch, micro, policy):
    return {"name": name, "kind": "stage", "arch": arch, "dtype": dtype, "layers": layers, "hidden": hidden,
            "heads": heads, "kv": kv, "mlp": mlp, "seq": seq, "batch": batch, "micro": micro, "policy": policy}


def _attn(name, kind, dtype, batch, seq, heads, kv, dim):
    return {"name": name, "kind": kind, "dtype": dtype, "batch": batch, "seq": seq, "heads": heads, "kv": kv,
            "dim": dim}


def listed() -> list:
    return [
        # the f32 correctness workload: every kernel is small, launches count
        _stage("stage_tiny_f32", "gpt", "f32", 2, 256, 4, 4, 1024, 128, 2, 4, "recompute"),
        # a small GPT (head dim 64) on sequences that divide by no tile
        _stage("stage_h1024_d64_ragged", "gpt", "bf16", 1, 1024, 16, 16, 4096, 1000, 2, 2, "selective"),
        # two layers of the hidden-2048 workload
        _stage("stage_h2048", "gpt", "bf16", 2, 2048, 16, 16, 8192, 2048, 1, 2, "selective"),
        # one layer of the hidden-5120 workload, every activation kept
        _stage("stage_h5120", "gpt", "bf16", 1, 5120, 40, 40, 20480, 2048, 1, 2, "keep"),
        # one layer of the LLAMA-style workload at hidden 4096
        _stage("stage_llama_h4096", "llama", "bf16", 1, 4096, 32, 8, 14336, 4096, 1, 1, "selective"),
        # one layer of the long-sequence workload, recomputed from its input
        _stage("stage_h4096_s8192", "gpt", "bf16", 1, 4096, 32, 32, 16384, 8192, 1, 1, "inputs"),
        # long-sequence attention on its own
        _attn("attn_fwd_s8192", "attn_fwd", "bf16", 1, 8192, 32, 32, 128),
        # attention backward at the LLAMA2-70B widths (64 query, 8 key/value heads)
        _attn("attn_bwd_gqa_h8192", "attn_bwd", "bf16", 1, 4096, 64, 8, 128),
        # small models' head dim: batched, tile-aligned forward
        _attn("attn_fwd_d64", "attn_fwd", "bf16", 4, 2048, 16, 16, 64),
        # ... and a backward whose sequence divides by no tile
        _attn("attn_bwd_d64_ragged", "attn_bwd", "bf16", 2, 1999, 12, 12, 64),
        # the MLP of the hidden-8192 workload
        {"name": "mlp_h8192", "kind": "mlp", "dtype": "bf16", "tokens": 4096, "hidden": 8192, "mlp": 32768},
        # LayerNorm of the hidden-5120 workload
        {"name": "norm_h5120", "kind": "norm", "dtype": "bf16", "tokens": 2048, "hidden": 5120},
    ]


# --- drawn cases ---------------------------------------------------------------
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _candidate(rng) -> dict:
    kind = rng.choice(["stage_f32", "stage_gpt", "stage_gpt", "stage_llama", "attn_fwd", "attn_bwd", "mlp", "norm",
                       "swiglu"])
    policy = rng.choice(["keep", "selective", "inputs"])
    if kind == "stage_f32":
        heads = rng.randint(2, 8)
        hidden = 64 * heads
        c = _stage("", "gpt", "f32", rng.randint(1, 2), hidden, heads, heads, 4 * hidden, _log(rng, 16, 512),
                   rng.randint(1, 2), rng.randint(1, 4), rng.choice(["keep", "recompute"]))
    elif kind == "stage_gpt":
        dim = rng.choice([64, 128])
        heads = _log(rng, 512, 5120) // dim
        hidden = dim * heads
        c = _stage("", "gpt", "bf16", rng.randint(1, 2), hidden, heads, heads, 4 * hidden, _log(rng, 128, 4096),
                   rng.randint(1, 3), rng.randint(1, 2), policy)
    elif kind == "stage_llama":
        kv = rng.choice([2, 4, 8])
        heads = kv * rng.choice([1, 2, 4])
        hidden = 128 * heads
        c = _stage("", "llama", "bf16", 1, hidden, heads, kv, 64 * int(hidden * rng.uniform(2.6, 3.5) / 64),
                   _log(rng, 128, 4096), rng.randint(1, 2), rng.randint(1, 2), policy)
    elif kind in ("attn_fwd", "attn_bwd"):
        dim = rng.choice([64, 128])
        heads = rng.choice([8, 12, 16, 32, 40, 64])
        kv = heads // rng.choice([1, 4]) if dim == 128 else heads
        c = _attn("", kind, "bf16", rng.randint(1, 4), _log(rng, 64, 8192), heads, kv, dim)
    elif kind == "mlp":
        hidden = 128 * _log(rng, 4, 64)
        c = {"kind": "mlp", "dtype": "bf16", "tokens": _log(rng, 64, 8192), "hidden": hidden, "mlp": 4 * hidden}
    elif kind == "norm":
        c = {"kind": "norm", "dtype": "bf16", "tokens": _log(rng, 64, 8192), "hidden": 64 * _log(rng, 8, 128)}
    else:
        c = {"kind": "swiglu", "dtype": "bf16", "tokens": _log(rng, 64, 8192), "mlp": 64 * _log(rng, 16, 448)}
    c.pop("name", None)
    return c


def draw(rng) -> dict:
    """One more case of the listed cases' ranges, no larger than the largest of them."""
    works = [work(c) for c in listed()]
    flops, nbytes = max(w["flops"] for w in works), max(w["bytes"] for w in works)
    while True:
        c = _candidate(rng)
        w = work(c)
        if w["flops"] <= flops and w["bytes"] <= nbytes:
            return c


# --- work ----------------------------------------------------------------------
def _esize(case) -> int:
    return 2 if case["dtype"] == "bf16" else 4


def work(case) -> dict:
    """What one pass cannot do without: inputs read once, outputs written
    once, and the products of the forward (and the backward's two per linear;
    attention: two forward, five backward, over the causal triangle)."""
    k, e = case["kind"], _esize(case)
    if k == "stage":
        h, f, s, b = case["hidden"], case["mlp"], case["seq"], case["batch"]
        t, units = b * s, case["layers"] * case["micro"]
        n = sum(math.prod(sh) for sh in _shapes(case).values())
        mats = sum(math.prod(sh) for sh in _shapes(case).values() if len(sh) == 2)
        flops = units * (6.0 * t * mats + 7.0 * b * s * (s + 1) * h)
        return {"bytes": float(case["layers"] * n * (e + 4) + 4 * case["micro"] * t * h * e), "flops": flops}
    if k in ("attn_fwd", "attn_bwd"):
        b, s, nh, kv, d = (case[x] for x in ("batch", "seq", "heads", "kv", "dim"))
        qkv, o, lse = b * s * (nh + 2 * kv) * d * e, b * s * nh * d * e, b * s * nh * 4
        tri = b * s * (s + 1.0) * nh * d
        if k == "attn_fwd":
            return {"bytes": float(qkv + o + lse), "flops": 2 * tri}
        return {"bytes": float(2 * qkv + 2 * o + lse), "flops": 5 * tri}
    if k == "mlp":
        t, h, f = case["tokens"], case["hidden"], case["mlp"]
        # in: c, x1, the weights and biases; out: u, g, y
        return {"bytes": float(e * (3 * t * h + 2 * t * f + 2 * h * f + h + f)), "flops": 4.0 * t * h * f}
    if k == "norm":
        t, h = case["tokens"], case["hidden"]
        # in: x, dout, the residual gradient; out: the normalised rows and dx
        return {"bytes": float(5 * t * h * e + 2 * h * (e + 4) + 8 * t), "flops": 20.0 * t * h}
    t, f = case["tokens"], case["mlp"]
    # in: u (2f) and dg; out: g and du (2f)
    return {"bytes": float(6 * t * f * e), "flops": 24.0 * t * f}


# --- inputs --------------------------------------------------------------------
def _gen(seed) -> torch.Generator:
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)


def _normal(g, shape, dtype, scale=1.0, shift=0.0):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * scale + shift).to(dtype)


def _shapes(case) -> dict:
    h, f = case["hidden"], case["mlp"]
    if case["arch"] == "llama":
        d = h // case["heads"]
        return {"w_qkv": ((case["heads"] + 2 * case["kv"]) * d, h), "w_o": (h, h), "w_1": (2 * f, h), "w_2": (h, f),
                "g1": (h,), "g2": (h,)}
    return {"w_qkv": (3 * h, h), "b_qkv": (3 * h,), "w_o": (h, h), "b_o": (h,), "w_1": (f, h), "b_1": (f,),
            "w_2": (h, f), "b_2": (h,), "g1": (h,), "be1": (h,), "g2": (h,), "be2": (h,)}


def _stage_inputs(case, seed):
    """Parameters of every layer, stage inputs and output gradients: matrices,
    biases and shifts N(0, 0.02), gains 1 + N(0, 0.02), x and dy N(0, 1)."""
    g, dt = _gen(seed), _TORCH[case["dtype"]]
    params = [{n: _normal(g, sh, dt, 0.02, 1.0 if n in ("g1", "g2") else 0.0) for n, sh in _shapes(case).items()}
              for _ in range(case["layers"])]
    rows = (case["batch"] * case["seq"], case["hidden"])
    xs = [_normal(g, rows, dt) for _ in range(case["micro"])]
    dys = [_normal(g, rows, dt) for _ in range(case["micro"])]
    return params, xs, dys


def _attn_inputs(case, seed):
    """Packed qkv rows, and for the backward the forward's o and lse (plain
    torch, f32) and an output gradient."""
    g, dt = _gen(seed), _TORCH[case["dtype"]]
    b, s, nh, kv, d = (case[x] for x in ("batch", "seq", "heads", "kv", "dim"))
    qkv = _normal(g, (b * s, (nh + 2 * kv) * d), dt)
    if case["kind"] == "attn_fwd":
        return qkv, None, None, None
    do = _normal(g, (b * s, nh * d), dt)
    o, lse = _attention(qkv.float(), b, s, nh, kv, d)
    return qkv, o.to(dt), lse, do


def _mlp_inputs(case, seed):
    g, dt = _gen(seed), _TORCH[case["dtype"]]
    t, h, f = case["tokens"], case["hidden"], case["mlp"]
    return {"c": _normal(g, (t, h), dt), "x1": _normal(g, (t, h), dt), "w1": _normal(g, (f, h), dt, 0.02),
            "b1": _normal(g, (f,), dt, 0.02), "w2": _normal(g, (h, f), dt, 0.02), "b2": _normal(g, (h,), dt, 0.02)}


def _norm_inputs(case, seed):
    g, dt = _gen(seed), _TORCH[case["dtype"]]
    t, h = case["tokens"], case["hidden"]
    return {"x": _normal(g, (t, h), dt), "dout": _normal(g, (t, h), dt), "resid": _normal(g, (t, h), dt),
            "gamma": _normal(g, (h,), dt, 0.02, 1.0), "beta": _normal(g, (h,), dt, 0.02)}


def _swiglu_inputs(case, seed):
    g, dt = _gen(seed), _TORCH[case["dtype"]]
    return {"u": _normal(g, (case["tokens"], 2 * case["mlp"]), dt),
            "dg": _normal(g, (case["tokens"], case["mlp"]), dt)}


def _config(case) -> T.StageConfig:
    L = case["layers"]
    policy = {"keep": None, "selective": configs.policy_selective(L), "inputs": configs.policy_layer_inputs(L),
              "recompute": configs.policy_all(L, T.RECOMPUTE)}[case["policy"]]
    llama = case["arch"] == "llama"
    return T.StageConfig(n_layers=L, hidden=case["hidden"], n_heads=case["heads"], mlp=case["mlp"], seq=case["seq"],
                         micro_batch=case["batch"], n_micro=case["micro"], dtype=case["dtype"], ln_eps=_EPS,
                         policy=policy, arch=T.ARCH_LLAMA if llama else T.ARCH_GPT,
                         n_kv_heads=case["kv"] if llama else 0, rope_base=_ROPE)


def prepare(case, seed):
    k = case["kind"]
    if k == "stage":
        return _prepare_stage(case, seed)
    if k in ("attn_fwd", "attn_bwd"):
        qkv, o, lse, do = _attn_inputs(case, seed)
        b, s, nh, d = (case[x] for x in ("batch", "seq", "heads", "dim"))
        st = {"case": case, "qkv": qkv, "o": o, "lse": lse, "do": do}
        if k == "attn_fwd":
            st["o"] = torch.empty((b * s, nh * d), dtype=qkv.dtype, device="cuda")
            st["lse"] = torch.empty((b, nh, s), dtype=torch.float32, device="cuda")
        else:
            st["dqkv"] = torch.empty_like(qkv)
            st["ws"] = torch.empty(T.op_workspace_bytes(T.WS_ATTN_BWD, b * s, nh) // 4, dtype=torch.float32,
                                   device="cuda")
            st["kv_ws"] = (torch.empty((b * s, 2 * nh * d), dtype=qkv.dtype, device="cuda")
                           if case["kv"] != nh else None)
        return st
    if k == "mlp":
        st = {"case": case, **_mlp_inputs(case, seed)}
        st["u"] = torch.empty((case["tokens"], case["mlp"]), dtype=st["c"].dtype, device="cuda")
        st["g"], st["y"] = torch.empty_like(st["u"]), torch.empty_like(st["c"])
        return st
    if k == "norm":
        t, h = case["tokens"], case["hidden"]
        st = {"case": case, **_norm_inputs(case, seed)}
        st["out"], st["dx"] = torch.empty_like(st["x"]), torch.empty_like(st["x"])
        st["mean"], st["rstd"] = (torch.empty(t, dtype=torch.float32, device="cuda") for _ in range(2))
        st["dparam"] = torch.empty((2, h), dtype=torch.float32, device="cuda")
        st["ws"] = torch.empty(T.op_workspace_bytes(T.WS_COLSUM, t, 2 * h) // 4, dtype=torch.float32, device="cuda")
        return st
    st = {"case": case, **_swiglu_inputs(case, seed)}
    st["g"], st["du"] = torch.empty_like(st["dg"]), torch.empty_like(st["u"])
    return st


def _prepare_stage(case, seed):
    cfg = _config(case)
    po, pb, go, gb = T.param_layout(cfg)
    dt, shapes = _TORCH[case["dtype"]], _shapes(case)
    params, xs, dys = _stage_inputs(case, seed)
    blocks, grads, views = [], [], []
    for p in params:
        blk = torch.zeros(pb, dtype=torch.uint8, device="cuda")
        grd = torch.zeros(gb, dtype=torch.uint8, device="cuda")
        view = {}
        for n, sh in shapes.items():
            i, numel = T.PARAMS.index(n), math.prod(sh)
            blk[po[i]:po[i] + numel * dt.itemsize].view(dt).copy_(p[n].reshape(-1))
            view[n] = grd[go[i]:go[i] + 4 * numel].view(torch.float32).view(sh)
        blocks.append(blk)
        grads.append(grd)
        views.append(view)
    del params
    return {"case": case, "stage": T.Stage(cfg, blocks, grads), "order": cfg.order(), "xs": xs, "dys": dys,
            "ys": [torch.empty_like(x) for x in xs], "dxs": [torch.empty_like(x) for x in xs], "grads": views}


# --- one pass --------------------------------------------------------------------
def run(state):
    case = state["case"]
    k = case["kind"]
    if k == "stage":
        st, xs, ys, dys, dxs = (state[n] for n in ("stage", "xs", "ys", "dys", "dxs"))
        st.begin_iteration(zero_grads=True)
        for op, mb in state["order"]:
            if op == "F":
                st.forward(mb, xs[mb], ys[mb])
            else:
                st.backward(mb, dys[mb], dxs[mb])
        return {"y": ys, "dx": dxs, "grads": state["grads"]}
    dt = _CODE[case["dtype"]]
    if k in ("attn_fwd", "attn_bwd"):
        b, s, nh, kv, d = (case[x] for x in ("batch", "seq", "heads", "kv", "dim"))
        if k == "attn_fwd":
            if kv != nh:
                T.op_attention_gqa_fwd(b, s, nh, kv, state["qkv"], state["o"], state["lse"])
            else:
                T.op_attention_fwd(dt, b, s, nh, d, state["qkv"], state["o"], state["lse"])
            return {"o": state["o"], "lse": state["lse"]}
        if kv != nh:
            T.op_attention_gqa_bwd(b, s, nh, kv, state["qkv"], state["o"], state["lse"], state["do"], state["dqkv"],
                                   state["ws"], state["kv_ws"])
        else:
            T.op_attention_bwd(dt, b, s, nh, d, state["qkv"], state["o"], state["lse"], state["do"], state["dqkv"],
                               state["ws"])
        return {"dqkv": state["dqkv"]}
    if k == "mlp":
        t, h, f = case["tokens"], case["hidden"], case["mlp"]
        T.op_gemm(dt, T.GEMM_NT, T.EPI_BIAS_GELU, t, f, h, state["c"], h, state["w1"], h, state["g"], f,
                  bias=state["b1"], aux=state["u"], ldaux=f)
        T.op_gemm(dt, T.GEMM_NT, T.EPI_BIAS_RESID, t, h, f, state["g"], f, state["w2"], f, state["y"], h,
                  bias=state["b2"], resid=state["x1"], ldr=h)
        return {"u": state["u"], "g": state["g"], "y": state["y"]}
    if k == "norm":
        t, h = case["tokens"], case["hidden"]
        dgamma, dbeta = state["dparam"].zero_()   # the backward adds to them
        T.op_layernorm_fwd(dt, t, h, state["x"], state["gamma"], state["beta"], _EPS, state["out"], state["mean"],
                           state["rstd"])
        T.op_layernorm_bwd(dt, t, h, state["dout"], state["x"], state["mean"], state["rstd"], state["gamma"],
                           state["resid"], state["dx"], dgamma, dbeta, state["ws"])
        return {"out": state["out"], "dx": state["dx"], "dparam": state["dparam"]}
    t, f = case["tokens"], case["mlp"]
    T.op_swiglu_fwd(t, f, state["u"], state["g"])
    T.op_swiglu_bwd(t, f, state["dg"], state["u"], state["du"])
    return {"g": state["g"], "du": state["du"]}


# --- tolerances ------------------------------------------------------------------
def tolerance(case) -> dict:
    """About four times the distance from the 64-bit result that the path
    shows (one bf16 rounding per stored tensor; through a whole layer's
    forward and backward the roundings of every stored tensor add up)."""
    if case["kind"] == "stage":
        return {"rel": 1e-5 if case["dtype"] == "f32" else 3e-2}
    return {"rel": 1.2e-2 if case["kind"] == "attn_bwd" else 8e-3}


# --- 64-bit results ----------------------------------------------------------------
def _mask(s, dev):
    i = torch.arange(s, device=dev)
    return i[None, :] > i[:, None]


def _attention(qkv, b, s, nh, kv, d):
    """o [b s, nh d] and lse [b, nh, s] in the precision of qkv, head by head."""
    x = qkv.view(b, s, nh + 2 * kv, d)
    o = torch.empty((b, s, nh, d), dtype=qkv.dtype, device=qkv.device)
    lse = torch.empty((b, nh, s), dtype=qkv.dtype, device=qkv.device)
    mask = _mask(s, qkv.device)
    for i in range(b):
        for n in range(nh):
            kvh = n // (nh // kv)
            sc = (x[i, :, n] @ x[i, :, nh + kvh].T / math.sqrt(d)).masked_fill_(mask, -math.inf)
            lse[i, n] = torch.logsumexp(sc, dim=1)
            o[i, :, n] = torch.exp_(sc.sub_(lse[i, n][:, None])) @ x[i, :, nh + kv + kvh]
    return o.view(b * s, nh * d), lse


def _attention_bwd(qkv, o, lse, do, b, s, nh, kv, d):
    x, dx = qkv.view(b, s, nh + 2 * kv, d), torch.zeros_like(qkv).view(b, s, nh + 2 * kv, d)
    o, do = o.view(b, s, nh, d), do.view(b, s, nh, d)
    mask = _mask(s, qkv.device)
    for i in range(b):
        for n in range(nh):
            kk, vv = nh + n // (nh // kv), nh + kv + n // (nh // kv)
            p = (x[i, :, n] @ x[i, :, kk].T / math.sqrt(d)).masked_fill_(mask, -math.inf)
            p = torch.exp_(p.sub_(lse[i, n][:, None]))
            dx[i, :, vv] += p.T @ do[i, :, n]
            ds = p.mul_(do[i, :, n] @ x[i, :, vv].T - (do[i, :, n] * o[i, :, n]).sum(1, keepdim=True))
            dx[i, :, n] = ds @ x[i, :, kk] / math.sqrt(d)
            dx[i, :, kk] += ds.T @ x[i, :, n] / math.sqrt(d)
    return dx.view_as(qkv)


class _Attention(torch.autograd.Function):
    @staticmethod
    def forward(ctx, qkv, dims):
        o, lse = _attention(qkv, *dims)
        ctx.save_for_backward(qkv, o, lse)
        ctx.dims = dims
        return o

    @staticmethod
    def backward(ctx, do):
        return _attention_bwd(*ctx.saved_tensors, do.contiguous(), *ctx.dims), None


def _rope(x, s, d):
    """Rotates pairs (i, i + d/2) of every head of x [rows, heads, d]."""
    pos = torch.arange(x.shape[0], device=x.device, dtype=torch.float64) % s
    ang = pos[:, None] * _ROPE ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    c, sn = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * c - b * sn, b * c + a * sn], dim=-1)


def _layer(case, p, x):
    F = torch.nn.functional
    h, nh, kv, s = case["hidden"], case["heads"], case["kv"], case["seq"]
    d = h // nh
    if case["arch"] == "gpt":
        qkv = F.linear(F.layer_norm(x, (h,), p["g1"], p["be1"], _EPS), p["w_qkv"], p["b_qkv"])
        x1 = x + F.linear(_Attention.apply(qkv, (case["batch"], s, nh, nh, d)), p["w_o"], p["b_o"])
        u = F.linear(F.layer_norm(x1, (h,), p["g2"], p["be2"], _EPS), p["w_1"], p["b_1"])
        return x1 + F.linear(F.gelu(u), p["w_2"], p["b_2"])
    qkv = F.linear(F.rms_norm(x, (h,), p["g1"], _EPS), p["w_qkv"]).view(-1, nh + 2 * kv, d)
    qkv = torch.cat([_rope(qkv[:, :nh + kv], s, d), qkv[:, nh + kv:]], dim=1).reshape(-1, (nh + 2 * kv) * d)
    x1 = x + F.linear(_Attention.apply(qkv, (case["batch"], s, nh, kv, d)), p["w_o"])
    gate, up = F.linear(F.rms_norm(x1, (h,), p["g2"], _EPS), p["w_1"]).chunk(2, dim=-1)
    return x1 + F.linear(F.silu(gate) * up, p["w_2"])


def exact(case, seed):
    k = case["kind"]
    if k == "stage":
        params, xs, dys = _stage_inputs(case, seed)
        params = [{n: t.double().requires_grad_() for n, t in p.items()} for p in params]
        out = {"y": [], "dx": [], "grads": None}
        for x, dy in zip(xs, dys):
            x = x.double().requires_grad_()
            y = x
            for p in params:
                y = _layer(case, p, y)
            y.backward(dy.double())
            out["y"].append(y.detach())
            out["dx"].append(x.grad)
            del y
        out["grads"] = [{n: t.grad for n, t in p.items()} for p in params]
        return out
    if k in ("attn_fwd", "attn_bwd"):
        qkv, o, lse, do = _attn_inputs(case, seed)
        dims = tuple(case[x] for x in ("batch", "seq", "heads", "kv", "dim"))
        if k == "attn_fwd":
            o, lse = _attention(qkv.double(), *dims)
            return {"o": o, "lse": lse}
        return {"dqkv": _attention_bwd(qkv.double(), o.double(), lse.double(), do.double(), *dims)}
    F = torch.nn.functional
    if k == "mlp":
        i = {n: t.double() for n, t in _mlp_inputs(case, seed).items()}
        u = F.linear(i["c"], i["w1"], i["b1"])
        g = F.gelu(u)
        return {"u": u, "g": g, "y": i["x1"] + F.linear(g, i["w2"], i["b2"])}
    if k == "norm":
        i = {n: t.double() for n, t in _norm_inputs(case, seed).items()}
        x, gamma, beta = (i[n].requires_grad_() for n in ("x", "gamma", "beta"))
        y = F.layer_norm(x, (case["hidden"],), gamma, beta, _EPS)
        y.backward(i["dout"])
        return {"out": y.detach(), "dx": x.grad + i["resid"], "dparam": torch.stack([gamma.grad, beta.grad])}
    i = {n: t.double() for n, t in _swiglu_inputs(case, seed).items()}
    gate, up = i["u"].chunk(2, dim=-1)
    sg = torch.sigmoid(gate)
    return {"g": gate * sg * up, "du": torch.cat([i["dg"] * up * sg * (1 + gate * (1 - sg)), i["dg"] * gate * sg], 1)}
