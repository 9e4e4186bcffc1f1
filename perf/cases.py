"""What is timed: the work that a training program has this library do on one GPU.

Every case goes through the public entry points as such a program calls them: layers and stages through the buffer
helpers of ``runner``, single operations of the path and the first / last stage's extras through the binding.  Sizes are
those of the named workloads (``inputs.WORKLOADS``), of ``bench.py`` and of the tests, or generic ones.
"""
import math

import torch

import paper_2201_11990_amd as M
from paper_2201_11990_amd import binding as B
from paper_2201_11990_amd.inputs import PARAM_NAMES, Workload, make_activations, make_layer_params, torch_dtype
from paper_2201_11990_amd.runner import LayerRunner, StageRunner

EPS = 1e-5


# ------------------------------------------------------------------ the cases
def _layer(name, hidden, heads, head_dim, ffn, seq, micro_batch, dtype="bf16", w_std=0.02, gelu="tanh", layers=1,
           micro=1, recompute=False, hook=False, grad_fp32=False):
    return {"name": name, "kind": "stage" if layers > 1 or micro > 1 or recompute or hook else "layer", "hidden": hidden,
            "heads": heads, "head_dim": head_dim, "ffn": ffn, "seq": seq, "micro_batch": micro_batch, "dtype": dtype,
            "w_std": w_std, "gelu": gelu, "layers": layers, "micro": micro, "recompute": recompute, "hook": hook,
            "grad_fp32": grad_fp32}


def listed():
    return [
        # fp32 path, smallest call: the unsliced toy layer (workload tiny_fp32), forward and backward.  Stands for
        # bring-up, unit tests and debugging runs, where launches and latency count.
        _layer("layer_fp32_tiny", 256, 4, 64, 1024, 128, 2, "fp32"),
        # fp32 path at a size that somebody trains or verifies a small model with.
        _layer("layer_fp32_mid", 1024, 16, 64, 4096, 512, 2, "fp32"),
        # bf16 path, small: a narrow slice with few tokens (the shape that smoke() runs), launch- and latency-bound.
        _layer("layer_bf16_small", 512, 2, 160, 1024, 256, 1),
        # ordinary bf16 training: the 1.3B-shaped layer at micro-batch 4.
        _layer("layer_gpt1p3b", 2048, 16, 128, 8192, 2048, 4),
        # the same layer on a sequence of odd length (packed or truncated documents): no size is a multiple of a tile.
        _layer("layer_ragged", 2048, 16, 128, 8192, 1990, 1),
        # the largest: one layer of the MT-NLG slice that the benchmark chains three of.
        _layer("layer_mtnlg_tp8", 20480, 16, 160, 10240, 2048, 1, w_std=0.004),
        # one rank's steady state: two stacked layers, two micro-batches with recomputation, gradients accumulated in
        # fp32, and a tensor-parallel hook (a group of one: nothing to add), i.e. the unfused residual / bias kernels.
        _layer("stage_accumulate", 2048, 16, 128, 8192, 2048, 1, layers=2, micro=2, recompute=True, hook=True, grad_fp32=True),
        # attention alone, forward and backward, MT-NLG's heads at the tests' ragged sequence length.
        {"name": "attention_d160_ragged", "kind": "attention", "batch": 1, "seq": 1990, "heads": 16, "head_dim": 160},
        # attention at a head size between the usual powers of two.
        {"name": "attention_d96", "kind": "attention", "batch": 2, "seq": 1024, "heads": 16, "head_dim": 96},
        # last pipeline stage: final LayerNorm, tied projection on a 6400-row vocabulary slice, cross-entropy, and back.
        {"name": "lm_head", "kind": "lm_head", "hidden": 20480, "vocab": 6400, "seq": 2048, "micro_batch": 1},
        # first pipeline stage: token embedding with positions and its gradients, on the slice with the frequent ids.
        {"name": "embedding", "kind": "embedding", "hidden": 20480, "vocab": 6400, "vocab_total": 51200, "vocab_start": 0,
         "seq": 2048, "micro_batch": 1},
        # optimizer: squared gradient norm and Adam over the twelve tensors of the 1.3B-shaped layer.
        {"name": "optimizer", "kind": "optimizer", "hidden": 2048, "proj": 2048, "ffn": 8192},
    ]


def _log_int(rng, lo, hi, step=1):
    """Spread evenly over the logarithm, a multiple of ``step``."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _draw_layer(rng):
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
    d = rng.choice([64, 128, 160]) if dtype == "bf16" or rng.random() < 0.5 else 8 * rng.randint(4, 16)
    heads = _log_int(rng, 1, 16)
    hidden = rng.choice([heads * d, _log_int(rng, 256, 20480 if dtype == "bf16" else 1536, 64)])
    hidden = max(hidden, 64)
    # FFN widths of a slice: usually four times the slice's share of the hidden size, now and then an odd multiple of 8
    ffn = rng.choice([4 * heads * d, _log_int(rng, 256, 10240 if dtype == "bf16" else 4096, 8)])
    seq = rng.choice([_log_int(rng, 32, 2048), _log_int(rng, 64, 2048, 64)])
    mb = rng.choice([1, 1, 2, 4])
    kw = {}
    if rng.random() < 0.4:
        kw = {"layers": rng.choice([1, 2]), "micro": rng.choice([1, 2]), "recompute": rng.random() < 0.5,
              "hook": rng.random() < 0.5, "grad_fp32": dtype == "bf16" and rng.random() < 0.5}
    c = _layer("drawn", hidden, heads, d, ffn, seq, mb, dtype, gelu=rng.choice(["tanh", "tanh", "erf"]),
               w_std=0.02 if hidden < 8192 else 0.004, **kw)
    return c, 2.0e11 if dtype == "fp32" else 4.0e12


def draw(rng):
    while True:
        kind = rng.choice(["layer"] * 5 + ["attention"] * 2 + ["lm_head", "embedding", "optimizer"])
        limit = 4.0e12
        if kind == "layer":
            c, limit = _draw_layer(rng)
        elif kind == "attention":
            d = rng.choice([64, 128, 160, 8 * rng.randint(4, 20)])
            c = {"kind": kind, "batch": rng.choice([1, 1, 2, 4]), "seq": _log_int(rng, 33, 2048), "heads": _log_int(rng, 1, 16),
                 "head_dim": d}
        elif kind == "lm_head":
            c = {"kind": kind, "hidden": _log_int(rng, 512, 20480, 64), "vocab": _log_int(rng, 512, 6400, 8),
                 "seq": _log_int(rng, 64, 2048), "micro_batch": rng.choice([1, 1, 2])}
        elif kind == "embedding":
            vocab = _log_int(rng, 512, 6400, 8)
            c = {"kind": kind, "hidden": _log_int(rng, 512, 20480, 64), "vocab": vocab, "vocab_total": 8 * vocab,
                 "vocab_start": vocab * rng.randint(0, 7), "seq": _log_int(rng, 64, 2048), "micro_batch": rng.choice([1, 2, 4])}
        else:
            proj = 64 * rng.randint(4, 40)
            c = {"kind": kind, "hidden": _log_int(rng, 256, 6144, 8), "proj": proj, "ffn": 4 * proj}
        c.pop("name", None)
        w = work(c)
        if w["flops"] <= limit and w["bytes"] <= 3.0e9:
            return c


# ------------------------------------------------------------------ what a program has in hand
def _workload(c):
    return Workload("case", c["hidden"], c["heads"], c["head_dim"], c["ffn"], c["seq"], c["micro_batch"], c["layers"],
                    c["dtype"], c["w_std"], recompute=c["recompute"])


def _stage_inputs(c, seed):
    wl = _workload(c)
    ws = [make_layer_params(wl, l, seed=seed, device="cuda", affine="random") for l in range(c["layers"])]
    acts = [make_activations(wl, seed=seed * 64 + m, device="cuda") for m in range(c["micro"])]
    return wl, ws, torch.stack([a[0] for a in acts]), torch.stack([a[1] for a in acts])


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _randn(shape, g, scale=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=g, device="cuda") * scale).to(dtype)


def _attention_inputs(c, seed):
    g = _gen(seed)
    T, p = c["batch"] * c["seq"], c["heads"] * c["head_dim"]
    return _randn((T, 3 * p), g), _randn((T, p), g)


def _lm_head_inputs(c, seed):
    g = _gen(seed)
    T, h, V = c["seq"] * c["micro_batch"], c["hidden"], c["vocab"]
    return {"x": _randn((T, h), g), "ln_g": _randn((h,), g, 0.1) + 1, "ln_b": _randn((h,), g, 0.1),
            "emb": _randn((V, h), g, 0.02 if h < 8192 else 0.004),
            "targets": torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)}


def _embedding_inputs(c, seed):
    g = _gen(seed)
    T, h = c["seq"] * c["micro_batch"], c["hidden"]
    # token ids fall off like 1 / rank, as the ids of a frequency-ordered vocabulary do
    u = torch.rand(T, generator=g, device="cuda", dtype=torch.float64)
    ids = (torch.exp(u * math.log(c["vocab_total"])) - 1).long().clamp(0, c["vocab_total"] - 1).to(torch.int32)
    return {"tokens": ids, "emb": _randn((c["vocab"], h), g, 0.02), "pos": _randn((c["seq"], h), g, 0.02),
            "dx": _randn((T, h), g)}


def _optimizer_shapes(c):
    h, p, f = c["hidden"], c["proj"], c["ffn"]
    return [(h,), (h,), (3 * p, h), (3 * p,), (h, p), (h,), (h,), (h,), (f, h), (f,), (h, f), (h,)]


def _optimizer_inputs(c, seed):
    g = _gen(seed)
    out = []
    for shape in _optimizer_shapes(c):
        grad = _randn(shape, g, 1e-3, torch.float32)
        out.append({"master": _randn(shape, g, 0.02, torch.float32), "m": _randn(shape, g, 1e-4, torch.float32),
                    "v": _randn(shape, g, 1e-3, torch.float32) ** 2, "grad": grad})
    return out


def _no_exchange(ptr, count, dtype, stream):
    """The sum over a tensor-parallel group of one."""


def prepare(case, seed):
    c = case
    if c["kind"] in ("layer", "stage"):
        wl, ws, xs, dys = _stage_inputs(c, seed)
        gelu = B.GELU_ERF if c["gelu"] == "erf" else B.GELU_TANH
        flags = B.WGRAD_FP32 if c["grad_fp32"] else 0
        if c["kind"] == "layer":
            return {"case": c, "run": LayerRunner(wl, ws[0], flags=flags, gelu=gelu), "x": xs[0], "dy": dys[0]}
        return {"case": c, "run": StageRunner(wl, ws, flags=flags, gelu=gelu), "x": xs, "dy": dys,
                "hook": _no_exchange if c["hook"] else None}
    if c["kind"] == "attention":
        qkv, da = _attention_inputs(c, seed)
        b, s, n, d = c["batch"], c["seq"], c["heads"], c["head_dim"]
        return {"case": c, "qkv": qkv, "da": da, "a": torch.empty_like(da), "dqkv": torch.empty_like(qkv),
                "lse": torch.empty((b, n, s), device="cuda"),
                "ws": torch.empty(M.mtnlg_attention_bwd_workspace(b, s, n, d), dtype=torch.uint8, device="cuda")}
    if c["kind"] == "lm_head":
        st = _lm_head_inputs(c, seed)
        desc = B.head_desc(c["hidden"], c["vocab"], 0, c["seq"], c["micro_batch"], "bf16", EPS)
        st.update(case=c, desc=desc, loss=torch.empty(st["x"].shape[0], device="cuda"), dx=torch.empty_like(st["x"]),
                  d_ln_g=torch.empty_like(st["ln_g"]), d_ln_b=torch.empty_like(st["ln_b"]), demb=torch.empty_like(st["emb"]),
                  ws=torch.empty(M.mtnlg_lm_head_workspace(desc), dtype=torch.uint8, device="cuda"))
        return st
    if c["kind"] == "embedding":
        st = _embedding_inputs(c, seed)
        st.update(case=c, desc=B.head_desc(c["hidden"], c["vocab"], c["vocab_start"], c["seq"], c["micro_batch"], "bf16", EPS),
                  x=torch.empty_like(st["dx"]), demb=torch.empty_like(st["emb"]), dpos=torch.empty_like(st["pos"]))
        return st
    tensors = _optimizer_inputs(c, seed)
    for t in tensors:
        t["w16"] = torch.empty_like(t["master"], dtype=torch.bfloat16)
    return {"case": c, "tensors": tensors, "sqnorm": torch.zeros(1, device="cuda"),
            "ws": torch.empty(M.mtnlg_grad_sqnorm_workspace(), dtype=torch.uint8, device="cuda")}


# ------------------------------------------------------------------ one pass
def run(state):
    s = state
    kind = s["case"]["kind"]
    if kind == "layer":
        y = s["run"].forward(s["x"])
        dx, grads = s["run"].backward(s["x"], s["dy"])
        return {"y": y, "dx": dx, **grads}
    if kind == "stage":
        ys, dxs, grads = s["run"].step_accumulate(s["x"], s["dy"], reduce=s["hook"])
        return {"y": ys, "dx": dxs, "grads": grads}
    if kind == "attention":
        c = s["case"]
        dims = (c["batch"], c["seq"], c["heads"], c["head_dim"], 1.0 / math.sqrt(c["head_dim"]))
        M.mtnlg_attention_fwd(*dims, s["qkv"], s["a"], s["lse"])
        M.mtnlg_attention_bwd(*dims, s["qkv"], s["a"], s["lse"], s["da"], s["dqkv"], s["ws"])
        return {"a": s["a"], "lse": s["lse"], "dqkv": s["dqkv"]}
    if kind == "lm_head":
        M.mtnlg_lm_head_step(s["desc"], s["x"], s["ln_g"], s["ln_b"], s["emb"], s["targets"], None, s["loss"], s["dx"],
                             s["d_ln_g"], s["d_ln_b"], s["demb"], s["ws"])
        return {k: s[k] for k in ("loss", "dx", "d_ln_g", "d_ln_b", "demb")}
    if kind == "embedding":
        M.mtnlg_embedding_fwd(s["desc"], s["tokens"], s["emb"], s["pos"], s["x"])
        M.mtnlg_embedding_bwd(s["desc"], s["tokens"], s["dx"], s["demb"], s["dpos"])
        return {k: s[k] for k in ("x", "demb", "dpos")}
    for i, t in enumerate(s["tensors"]):
        M.mtnlg_grad_sqnorm(t["grad"], s["ws"], s["sqnorm"], accumulate=i > 0)
    for t in s["tensors"]:
        M.mtnlg_adam_step(t["master"], t["m"], t["v"], t["grad"], t["w16"], s["sqnorm"], lr=5e-5, step=3,
                          weight_decay=0.1 if t["master"].dim() > 1 else 0.0)
    return {"sqnorm": s["sqnorm"], "tensors": [{k: t[k] for k in ("master", "m", "v", "w16")} for t in s["tensors"]]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    if c["kind"] in ("layer", "stage"):
        wl = _workload(c)
        es = 2 if c["dtype"] == "bf16" else 4
        params = sum(math.prod(s) for s in wl.param_shapes().values())
        fwd = M.flops.layer_forward_flops(wl.hidden, wl.heads, wl.head_dim, wl.ffn, wl.seq, wl.micro_batch)
        gs = 4 if c["grad_fp32"] else es
        return {"bytes": c["layers"] * params * (es + gs) + c["micro"] * 4 * wl.tokens * wl.hidden * es,
                "flops": 3.0 * fwd * c["layers"] * c["micro"]}
    if c["kind"] == "attention":
        T, p = c["batch"] * c["seq"], c["heads"] * c["head_dim"]
        # forward: qkv in, a and lse out; backward: qkv, a, lse, da in, dqkv out
        # two products forward and five backward on the causal half
        return {"bytes": 2 * T * p * (3 + 1 + 3 + 1 + 1 + 3) + 8 * T * c["heads"], "flops": 7.0 * T * p * (c["seq"] + 1)}
    if c["kind"] == "lm_head":
        T, h, V = c["seq"] * c["micro_batch"], c["hidden"], c["vocab"]
        return {"bytes": 2 * (2 * T * h + 2 * V * h), "flops": 6.0 * T * V * h}
    if c["kind"] == "embedding":
        T, h, V, s = c["seq"] * c["micro_batch"], c["hidden"], c["vocab"], c["seq"]
        # rows of the embedding that the tokens name, positions and dx in; x, demb and dpos out
        return {"bytes": 2 * h * (3 * T + V + 2 * s), "flops": 3.0 * T * h}
    n = sum(math.prod(s) for s in _optimizer_shapes(c))
    return {"bytes": 34 * n, "flops": 16.0 * n}


def tolerance(case):
    """About four times the largest relative error against ``exact`` that any output of the kind shows."""
    c = case
    if c["kind"] in ("layer", "stage"):   # 1.4e-6 in fp32, 4e-3 to 8e-3 in bf16 (gradients of gains behind a whole layer)
        return {"rel": 1e-5 if c["dtype"] == "fp32" else 2e-2}
    if c["kind"] == "optimizer":          # 3e-6: a bf16 weight next to a tie may round the other way
        return {"rel": 1e-5, "max": 1e-2}
    return {"rel": 1e-2}                  # single operations in bf16: 1.7e-3 to 2.7e-3


# ------------------------------------------------------------------ the same in 64 bits
def _layer_norm64(x, g, b):
    mu = x.mean(-1, keepdim=True)
    xc = x - mu
    return xc / torch.sqrt((xc * xc).mean(-1, keepdim=True) + EPS) * g + b


def _attention64(qkv, b, s, n, d):
    """[b*s, n*3*d] -> a [b*s, n*d], lse [b, n, s]; plain torch operations."""
    q, k, v = (t.transpose(1, 2) for t in qkv.view(b, s, n, 3, d).unbind(3))
    mask = torch.ones(s, s, dtype=torch.bool, device=qkv.device).triu(1)
    outs, lses = [], []
    for i in range(b):
        sc = (q[i].contiguous() @ k[i].transpose(1, 2).contiguous() / math.sqrt(d)).masked_fill(mask, -math.inf)
        lses.append(torch.logsumexp(sc, -1))
        outs.append((torch.softmax(sc, -1) @ v[i].contiguous()).transpose(0, 1).reshape(s, n * d))
    return torch.cat(outs), torch.stack(lses)


def _layer64(c, w, x):
    b, s = c["micro_batch"], c["seq"]
    gelu = "none" if c["gelu"] == "erf" else "tanh"
    x = x.reshape(b * s, -1)
    qkv = _layer_norm64(x, w["ln1_g"], w["ln1_b"]) @ w["w_qkv"].T + w["b_qkv"]
    a, _ = _attention64(qkv, b, s, c["heads"], c["head_dim"])
    x1 = x + a @ w["w_o"].T + w["b_o"]
    z = _layer_norm64(x1, w["ln2_g"], w["ln2_b"]) @ w["w_fc1"].T + w["b_fc1"]
    return x1 + torch.nn.functional.gelu(z, approximate=gelu) @ w["w_fc2"].T + w["b_fc2"]


def exact(case, seed):
    c = case
    if c["kind"] in ("layer", "stage"):
        wl, ws, xs, dys = _stage_inputs(c, seed)
        ws = [{k: t.double().requires_grad_() for k, t in w.items()} for w in ws]
        ys, dxs = [], []
        for x, dy in zip(xs, dys):
            x = x.double().requires_grad_()
            y = x
            for w in ws:
                y = _layer64(c, w, y)
            y.backward(dy.double().reshape(y.shape))
            ys.append(y.detach().view(x.shape))
            dxs.append(x.grad)
        grads = [{k: w[k].grad for k in PARAM_NAMES} for w in ws]
        if c["kind"] == "layer":
            return {"y": ys[0], "dx": dxs[0], **grads[0]}
        return {"y": torch.stack(ys), "dx": torch.stack(dxs), "grads": grads}
    if c["kind"] == "attention":
        qkv, da = _attention_inputs(c, seed)
        qkv = qkv.double().requires_grad_()
        a, lse = _attention64(qkv, c["batch"], c["seq"], c["heads"], c["head_dim"])
        a.backward(da.double())
        return {"a": a.detach(), "lse": lse.detach(), "dqkv": qkv.grad}
    if c["kind"] == "lm_head":
        st = _lm_head_inputs(c, seed)
        x, g, b, e = (st[k].double().requires_grad_() for k in ("x", "ln_g", "ln_b", "emb"))
        loss = torch.nn.functional.cross_entropy(_layer_norm64(x, g, b) @ e.T, st["targets"].long(), reduction="none")
        loss.mean().backward()
        return {"loss": loss.detach(), "dx": x.grad, "d_ln_g": g.grad, "d_ln_b": b.grad, "demb": e.grad}
    if c["kind"] == "embedding":
        st = _embedding_inputs(c, seed)
        ids = st["tokens"].long() - c["vocab_start"]
        mine = ((ids >= 0) & (ids < c["vocab"])).double()[:, None]
        ids = ids.clamp(0, c["vocab"] - 1)
        dx = st["dx"].double()
        x = st["emb"].double()[ids] * mine + st["pos"].double().repeat(c["micro_batch"], 1)
        demb = torch.zeros((c["vocab"], c["hidden"]), dtype=torch.float64, device="cuda").index_add_(0, ids, dx * mine)
        return {"x": x, "demb": demb, "dpos": dx.view(c["micro_batch"], c["seq"], -1).sum(0)}
    tensors = _optimizer_inputs(c, seed)
    sq = sum((t["grad"].double() ** 2).sum() for t in tensors)
    coef = torch.clamp(1.0 / (sq.sqrt() + 1e-6), max=1.0)
    out = []
    for t in tensors:
        p, m, v, g = (t[k].double() for k in ("master", "m", "v", "grad"))
        g = g * coef
        m = 0.9 * m + 0.1 * g
        v = 0.95 * v + 0.05 * g * g
        wd = 0.1 if p.dim() > 1 else 0.0
        p = p - 5e-5 * (m / (1 - 0.9 ** 3) / ((v / (1 - 0.95 ** 3)).sqrt() + 1e-8) + wd * p)
        out.append({"master": p, "m": m, "v": v, "w16": p.to(torch.bfloat16).double()})
    return {"sqnorm": sq.reshape(1), "tensors": out}
