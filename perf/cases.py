"""The work that users of this library have it do, as timed cases.

Six kinds of work, each through the public entry points of ``paper_2104_05343_amd``:

``layer``   one training step (forward and backward) of a transformer layer for ONE device of the q x q grid, the other
            devices' blocks resident: what each rank of the 2D scheme does per layer.  bf16, both attention forms.
``stack``   forward and backward of a checkpointed stack of layers, whole grid on one GPU.
``ends``    both ends of the model for one device: embedding, lm-head, cross entropy, and their gradients.
``mlp``     the feed-forward half of a layer in fp32 (the layer entry points are bf16 only), forward and backward, composed
            from LayerNorm, the products with their epilogues and the bias gradients.
``linear``  a linear layer's three products (forward, input gradient, weight gradient) of one device, bf16.
``attention``  the attention that keeps no [s x s] tensor, forward and backward, one device: long sequences.

A case is a dict of plain values; ``listed()`` names twelve, ``draw()`` gives more of the same ranges.
"""
from __future__ import annotations

import math

import torch

import paper_2104_05343_amd as opt

DEV = "cuda:0"


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # fp32 feed-forward of the smallest benchmark configuration, all four devices' blocks: launches and latency only
        {"name": "mlp_fp32_smallest", "kind": "mlp", "b": 2, "s": 16, "h": 64, "q": 2, "i": -1, "j": -1},
        # a two-layer model of the size of a unit test or a debugging run: launches and latency again, the bf16 path
        {"name": "stack_small", "kind": "stack", "b": 4, "s": 64, "h": 256, "n": 4, "q": 2, "layers": 2, "fused": False, "causal": True},
        # one device of a BERT-Large-sized layer on a 4 x 4 grid: about forty short kernels per step
        {"name": "layer_h1024", "kind": "layer", "b": 8, "s": 512, "h": 1024, "n": 16, "q": 4, "i": 1, "j": 2, "fused": False, "causal": True},
        # one device of a 4096-wide causal layer: the flagship step of the benchmark, with either attention
        {"name": "layer_h4096", "kind": "layer", "b": 8, "s": 1024, "h": 4096, "n": 32, "q": 4, "i": 1, "j": 2, "fused": False, "causal": True},
        {"name": "layer_h4096_fused", "kind": "layer", "b": 8, "s": 1024, "h": 4096, "n": 32, "q": 4, "i": 1, "j": 2, "fused": True, "causal": True},
        # large batch on an 8 x 8 grid: tall blocks, thin panels
        {"name": "layer_q8_large_batch", "kind": "layer", "b": 64, "s": 512, "h": 4096, "n": 32, "q": 8, "i": 5, "j": 3, "fused": True, "causal": True},
        # a sequence length and a width that are multiples of no tile
        {"name": "layer_ragged", "kind": "layer", "b": 8, "s": 1000, "h": 1280, "n": 20, "q": 4, "i": 2, "j": 1, "fused": True, "causal": True},
        # a checkpointed four-layer model, every device's share on one GPU: the largest launches
        {"name": "stack_h1024", "kind": "stack", "b": 8, "s": 512, "h": 1024, "n": 16, "q": 4, "layers": 4, "fused": False, "causal": True},
        # embedding, lm-head and loss of the 1024-wide model over a sub-word vocabulary, on a device that owns the most
        # frequent words (the others wait for it)
        {"name": "ends_v32768", "kind": "ends", "b": 8, "s": 512, "h": 1024, "v": 32768, "q": 4, "i": 0, "j": 1, "dtype": "bf16"},
        # fp32 feed-forward of one device at the 1024-wide layer's size
        {"name": "mlp_fp32_h1024", "kind": "mlp", "b": 8, "s": 512, "h": 1024, "q": 4, "i": 1, "j": 2},
        # 3072 -> 12288 linear layer on an 8 x 8 grid: skinny blocks, long contractions
        {"name": "linear_h3072_q8", "kind": "linear", "b": 32, "s": 512, "k": 3072, "n": 12288, "q": 8, "i": 2, "j": 5},
        # a sequence too long for score matrices in memory
        {"name": "attention_s4096", "kind": "attention", "b": 8, "s": 4096, "h": 4096, "n": 32, "q": 4, "i": 1, "j": 2, "causal": True},
    ]


def _log_int(rng, lo, hi, multiple=1):
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(multiple, int(round(x / multiple)) * multiple)


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    most_flops = max(work(c)["flops"] for c in listed() if c["kind"] == "layer")
    while True:
        kind = rng.choice(["layer", "layer", "layer", "stack", "ends", "mlp", "linear", "linear", "attention"])
        q = rng.choice([1, 2, 2, 4, 4, 8])
        i, j = rng.randrange(q), rng.randrange(q)
        if kind in ("layer", "stack"):
            fused = rng.random() < 0.5
            d = rng.choice([64, 128]) if fused else rng.choice([64, 64, 128, 80, 96])
            nh = rng.choice([1, 2, 3, 4, 5, 8])
            s = _log_int(rng, 64, 2048, rng.choice([1, 2, 64]) if fused else rng.choice([8, 8, 64]))
            case = {"kind": kind, "b": q * _log_int(rng, 1, 8), "s": s, "h": q * nh * d, "n": q * nh, "q": q, "fused": fused,
                    "causal": rng.random() < 0.8}
            if kind == "layer":
                case.update(i=i, j=j)
            else:
                case.update(layers=rng.randint(1, 4))
        elif kind == "ends":
            case = {"kind": kind, "b": q * _log_int(rng, 1, 4), "s": _log_int(rng, 64, 1024), "h": q * _log_int(rng, 64, 1024, 8),
                    "v": q * _log_int(rng, 500, 16384), "q": q, "i": i, "j": j, "dtype": rng.choice(["bf16", "bf16", "bf16", "fp32"])}
        elif kind == "mlp":
            case = {"kind": kind, "b": q * _log_int(rng, 1, 4), "s": _log_int(rng, 16, 512), "h": q * _log_int(rng, 32, 256, rng.choice([1, 4, 32])),
                    "q": q, "i": i, "j": j}
        elif kind == "linear":
            case = {"kind": kind, "b": q * _log_int(rng, 1, 8), "s": _log_int(rng, 64, 1024, rng.choice([1, 8, 64])),
                    "k": q * _log_int(rng, 64, 1024, rng.choice([8, 64])), "n": q * _log_int(rng, 64, 4096, rng.choice([8, 64])), "q": q, "i": i, "j": j}
        else:
            nh, d = rng.choice([1, 2, 4, 8]), rng.choice([64, 128])
            case = {"kind": kind, "b": q * _log_int(rng, 1, 4), "s": _log_int(rng, 256, 4096), "h": q * nh * d, "n": q * nh, "q": q,
                    "i": i, "j": j, "causal": rng.random() < 0.8}
        rows, width = case["b"] * case["s"], case.get("h", case.get("n"))
        fits = rows * width <= 32768 * 4096
        if kind in ("layer", "stack") and not case["fused"]:
            fits = fits and case["b"] * case["n"] * case["s"] ** 2 <= 1 << 29
        if fits and work(case)["flops"] <= most_flops:
            return case


# ------------------------------------------------------------------------------------------------ what a pass needs
def _attention_flops(case):
    nmat = (case["b"] // case["q"]) * (case["n"] // case["q"])
    one = 2 * nmat * case["s"] ** 2 * (case["h"] // case["n"]) * (0.5 if case["causal"] else 1.0)
    return 2 * one, 4 * one   # forward: Q K^T, P V; backward: dV, dP, dQ, dK


def work(case):
    """Bytes and flops of one pass that no implementation avoids: every input read once, every output written once
    (saved activations are outputs of the forward and inputs of the backward), the products' multiply-adds."""
    kind, q = case["kind"], case["q"]
    if kind == "attention":
        rows, cols = case["b"] * case["s"] // q, case["h"] // q
        fwd, bwd = _attention_flops(case)
        nbytes = rows * cols * 2 * (3 + 1 + 3 + 1 + 1 + 3)   # qkv, O; qkv, O, dO, d_qkv
        return {"bytes": nbytes, "flops": fwd + bwd}
    M = case["b"] * case["s"]
    if kind == "linear":
        K, N = case["k"], case["n"]
        Mb, Kb, Nb = M // q, K // q, N // q
        elems = (Mb * K + K * Nb + Mb * Nb) + (Mb * N + N * Kb + Mb * Kb) + (M * Kb + M * Nb)
        return {"bytes": 2 * elems + 4 * Kb * Nb, "flops": 3 * 2 * Mb * K * Nb}
    h = case["h"]
    Mb, hb = M // q, h // q
    if kind == "ends":
        v, e = case["v"], 2 if case["dtype"] == "bf16" else 4
        vb = v // q
        # embedding rows; logits = hidden table^T; loss; d_logits; d_hidden = d_logits table; table gradient; d_x rows in, gradient out
        elems = 2 * Mb * hb + (Mb * h + vb * h + Mb * vb) + Mb * vb + 2 * Mb * vb + (Mb * v + v * hb + Mb * hb) + (M * vb + M * hb) + M * hb
        return {"bytes": e * elems + 2 * 4 * vb * hb, "flops": 3 * 2 * Mb * h * vb}
    if kind == "mlp":
        devices = q * q if case["i"] < 0 else 1
        wide = 4 * h // q
        panels = (Mb * h + h * wide) + (Mb * 4 * h + 4 * h * hb)
        back = (Mb * h + wide * h) + (M * wide + M * hb) + (Mb * 4 * h + hb * 4 * h) + (M * hb + M * wide)
        blocks = 4 * Mb * hb + 3 * Mb * wide + Mb * hb + 2 * Mb * wide + 2 * h * wide + 4 * Mb * hb
        return {"bytes": 4 * devices * (panels + back + blocks), "flops": devices * 6 * 2 * Mb * h * wide}
    att_f, att_b = _attention_flops(case)
    linear = 2 * 12 * Mb * h * hb
    panels = Mb * h * 3 + Mb * 4 * h + 12 * h * hb                                  # forward: row panels and weight columns
    back = Mb * (h + 4 * h + h + 3 * h) + 12 * h * hb + M * hb * (4 + 1 + 1 + 4 + 1 + 1 + 1 + 3)   # input-gradient and weight-gradient operands
    blocks = Mb * hb * (1 + 2 + 3 + 1 + 1 + 2 + 4 + 4 + 1 + 4 + 1 + 1 + 1 + 3 + 1 + 1)   # saved tensors and gradients written
    scores = 0 if case["fused"] else (case["b"] // q) * (case["n"] // q) * case["s"] ** 2 * 2   # P written, P read
    one = {"bytes": 2 * (panels + back + blocks + scores) + 4 * 12 * hb * hb, "flops": 3 * linear + att_f + att_b}
    if kind == "layer":
        return one
    again = linear * 2 // 3 + att_f   # the recomputation, without the last product
    return {"bytes": one["bytes"] * q * q * case["layers"], "flops": (one["flops"] + again) * q * q * case["layers"]}


def tolerance(case):
    """Largest relative error between two correct implementations, each about four times (whole layers: twice) what was
    measured.  fp32: 1.4e-6 against fp64 for the feed-forward, 4.3e-6 for sums over a vocabulary.  bf16: 1.7e-3 against
    fp64 for single products (one rounding); layers and stacks differ by 5.8e-3 and 6.8e-3 between the two attention
    forms (other roundings, other order of the sums), and layers by 7.6e-3 from fp64."""
    if case["kind"] == "mlp":
        return {"rel": 6e-6}
    if case.get("dtype") == "fp32":
        return {"rel": 1.5e-5}
    return {"rel": {"layer": 1.5e-2, "stack": 2e-2, "attention": 1e-2}.get(case["kind"], 7e-3)}


# ------------------------------------------------------------------------------------------------ inputs and passes
class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, n, scale=1.0, dtype=torch.bfloat16, shift=0.0):
        out = torch.empty(n, dtype=dtype, device=DEV)
        for a in range(0, n, 1 << 26):   # in pieces: the fp32 draws of the largest tensors would not be needed at once
            m = min(1 << 26, n - a)
            out[a:a + m] = torch.randn(m, generator=self.g, device=DEV) * scale + shift
        return out

    def zipf(self, n, v):
        """Token indices with the rank-frequency shape of text."""
        p = 1.0 / torch.arange(1, v + 1, dtype=torch.float64, device=DEV)
        return torch.multinomial(p, n, replacement=True, generator=self.g).to(torch.int32)


def _block(t, q, i, j):
    """Device (i, j)'s part of a block-major tensor, or of a [q][q][...] one."""
    return t.view(q * q, -1)[i * q + j]


_WIDTHS = {  # [M x k*h] tensors of a layer beside its input
    "ln1_out": 1, "xhat1": 1, "qkv": 3, "attn": 1, "h_mid": 1, "ln2_out": 1, "xhat2": 1, "pre_gelu": 4, "gelu": 4, "out": 1,
    "d_pre_gelu": 4, "d_ln2_out": 1, "d_h_mid": 1, "d_attn": 1, "d_qkv": 3, "d_ln1_out": 1, "d_x": 1,
}
_WEIGHTS = {"w_qkv": 3, "w_o": 1, "w1": 4, "w2": 4}
_VECTORS = {"b_qkv": 3, "b_o": 1, "b1": 4, "b2": 1, "ln1_g": 1, "ln1_b": 1, "ln2_g": 1, "ln2_b": 1}


def _layer_params(r, h):
    p = {name: r.normal(k * h * h, 0.02) for name, k in _WEIGHTS.items()}
    for name, k in _VECTORS.items():
        p[name] = r.normal(k * h, 0.1, torch.float32, 1.0 if name.endswith("_g") else 0.0)
    return p


def _cfg(case):
    return opt.LayerCfg(case["b"], case["s"], case["h"], case["n"], case["q"], 1e-5, int(case["causal"]), opt.BF16, int(case["fused"]))


def _prepare_layer(case, r):
    b, s, h, n, q = (case[k] for k in "bshnq")
    M, nmat = b * s, b * n
    t = _layer_params(r, h)
    t["x"], t["d_out"] = r.normal(M * h), r.normal(M * h)
    for name, k in _WIDTHS.items():
        t[name] = torch.empty(k * M * h, dtype=torch.bfloat16, device=DEV)
    for name, k in _WEIGHTS.items():
        t["d_" + name] = torch.empty(k * h * h, dtype=torch.float32, device=DEV)
    for name, k in _VECTORS.items():
        t["d_" + name] = torch.empty(q * k * h, dtype=torch.float32, device=DEV)
    for name in ("rstd1", "rstd2"):
        t[name] = torch.empty(q * M, dtype=torch.float32, device=DEV)
    for name in ("stats1", "stats2", "bstats1", "bstats2"):
        t[name] = torch.empty(2 * q * M, dtype=torch.float32, device=DEV)
    if case["fused"]:
        t["lse"] = torch.empty(nmat * s, dtype=torch.float32, device=DEV)
    else:
        t["probs"] = torch.empty(nmat * s * s, dtype=torch.bfloat16, device=DEV)
    cfg = _cfg(case)
    ws = torch.empty(opt.layer_workspace_bytes(cfg), dtype=torch.uint8, device=DEV)
    lt = opt.make_layer_tensors(t)
    opt.layer_fwd(cfg, lt, -1, -1, ws)   # the peers' blocks of every stage: what a broadcast would have delivered
    opt.layer_bwd(cfg, lt, -1, -1, ws)
    names = list(_WIDTHS) + ["d_" + k for k in list(_WEIGHTS) + list(_VECTORS)]
    return {"cfg": cfg, "lt": lt, "ws": ws, "tensors": t, "out": {k: _block(t[k], q, case["i"], case["j"]) for k in names}}


def _run_layer(case, st):
    opt.layer_fwd(st["cfg"], st["lt"], case["i"], case["j"], st["ws"])
    opt.layer_bwd(st["cfg"], st["lt"], case["i"], case["j"], st["ws"])
    return st["out"]


def _prepare_stack(case, r):
    b, s, h, L = case["b"], case["s"], case["h"], case["layers"]
    M, cfg = b * s, _cfg(case)
    params = [_layer_params(r, h) for _ in range(L)]
    sizes = opt.stack_sizes(cfg, L)

    def buf(n):
        return torch.empty(n, dtype=torch.uint8, device=DEV)
    raw = [buf(getattr(sizes, k)) for k in ("workspace", "forward", "backward", "conjunction", "checkpoint")]
    grads = [buf(sizes.param_grad).zero_() for _ in range(L)]
    st = {"cfg": cfg, "keep": (params, raw), "params": [opt.make_layer_params(p) for p in params], "buf": opt.make_stack_buffers(*raw),
          "grads": [opt.layer_grads_in(cfg, g) for g in grads], "x": r.normal(M * h), "d_out": r.normal(M * h),
          "out": torch.empty(M * h, dtype=torch.bfloat16, device=DEV), "d_x": torch.empty(M * h, dtype=torch.bfloat16, device=DEV)}
    outputs = {"out": st["out"], "d_x": st["d_x"]}
    fields = {**{"d_" + k: w * h * h for k, w in _WEIGHTS.items()}, **{"d_" + k: case["q"] * w * h for k, w in _VECTORS.items()}}
    for layer, (g, at) in enumerate(zip(grads, st["grads"])):
        for name, n in fields.items():
            first = getattr(at, name) - g.data_ptr()
            outputs[f"{name}.{layer}"] = g[first:first + 4 * n].view(torch.float32)
    st["outputs"] = outputs
    return st


def _run_stack(case, st):
    opt.stack_fwd(st["cfg"], st["params"], st["x"], st["buf"], st["out"])
    opt.stack_bwd(st["cfg"], st["params"], st["grads"], st["d_out"], st["buf"], st["d_x"])
    return st["outputs"]


def _prepare_ends(case, r):
    b, s, h, v, q = (case[k] for k in "bshvq")
    M = b * s
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    st = {"dt": opt.BF16 if case["dtype"] == "bf16" else opt.FP32, "tokens": r.zipf(M, v), "labels": r.zipf(M, v),
          "table": r.normal(v * h, 0.02, dt), "hidden": r.normal(M * h, 1.0, dt), "d_x": r.normal(M * h, 1e-3, dt)}
    for name, n in (("x", M * h), ("logits", M * v), ("d_logits", M * v), ("d_hidden", M * h)):
        st[name] = torch.empty(n, dtype=dt, device=DEV)
    for name, n in (("stats", 2 * q * M), ("loss", q * M), ("lse", q * M), ("d_table_head", v * h), ("d_table", v * h)):
        st[name] = torch.empty(n, dtype=torch.float32, device=DEV)
    shapes = (("abt", M, h, v), ("ab", M, v, h), ("atb", v, M, h))
    st["ws"] = torch.empty(max(256, *(opt.summa_workspace_bytes(*x, q, case["i"], case["j"], st["dt"]) for x in shapes)),
                           dtype=torch.uint8, device=DEV)
    _ends_pass(case, st, -1, -1)   # the peers' blocks
    names = ("x", "logits", "loss", "lse", "d_logits", "d_hidden", "d_table_head", "d_table")
    st["out"] = {k: _block(st[k], q, case["i"], case["j"]) for k in names}
    return st


def _ends_pass(case, st, i, j):
    b, s, h, v, q = (case[k] for k in "bshvq")
    M, dt, ws = b * s, st["dt"], st["ws"]
    opt.embedding_fwd(st["tokens"], st["table"], st["x"], M, v, h, q, i, j, dt)
    opt.summa_abt(st["hidden"], st["table"], st["logits"], M, h, v, q, i, j, dt, ws=ws)
    opt.cross_entropy2d(st["logits"], st["labels"], st["loss"], st["lse"], st["stats"], M, v, q, i, j, dt)
    opt.cross_entropy2d_bwd(st["logits"], st["labels"], st["lse"], st["d_logits"], 1.0 / M, M, v, q, i, j, dt)
    opt.summa_ab(st["d_logits"], st["table"], st["d_hidden"], M, v, h, q, i, j, dt, ws=ws)
    opt.summa_ex("atb", st["d_logits"], st["hidden"], st["d_table_head"], v, M, h, q, i, j, dt, out_fp32=True, ws=ws)
    opt.embedding_bwd(st["tokens"], st["d_x"], st["d_table"], M, v, h, q, i, j, dt)


def _run_ends(case, st):
    _ends_pass(case, st, case["i"], case["j"])
    return st["out"]


def _prepare_mlp(case, r):
    b, s, h, q = case["b"], case["s"], case["h"], case["q"]
    M, f32 = b * s, torch.float32
    st = {"x": r.normal(M * h, 1.0, f32), "d_out": r.normal(M * h, 1.0, f32), "w1": r.normal(4 * h * h, 0.02, f32),
          "w2": r.normal(4 * h * h, 0.02, f32), "b1": r.normal(4 * h, 0.1, f32), "b2": r.normal(h, 0.1, f32),
          "g": r.normal(h, 0.1, f32, 1.0), "be": r.normal(h, 0.1, f32)}
    sizes = {"y": M * h, "xhat": M * h, "pre": 4 * M * h, "gelu": 4 * M * h, "out": M * h, "d_pre": 4 * M * h, "d_y": M * h, "d_x": M * h,
             "d_w1": 4 * h * h, "d_w2": 4 * h * h, "rstd": q * M, "stats": 2 * q * M, "bstats": 2 * q * M, "d_b1": 4 * q * h, "d_b2": q * h,
             "d_g": q * h, "d_be": q * h}
    for name, n in sizes.items():
        st[name] = torch.empty(n, dtype=f32, device=DEV)
    _mlp_pass(case, st, -1, -1)
    names = ("y", "pre", "gelu", "out", "d_pre", "d_y", "d_x", "d_w1", "d_w2", "d_b1", "d_b2", "d_g", "d_be")
    st["outputs"] = {k: st[k] if case["i"] < 0 else _block(st[k], q, case["i"], case["j"]) for k in names}
    return st


def _mlp_pass(case, st, i, j):
    h, q = case["h"], case["q"]
    M, f = case["b"] * case["s"], opt.FP32
    opt.layernorm2d(st["x"], st["g"], st["be"], st["y"], st["xhat"], st["rstd"], st["stats"], M, h, q, i, j, 1e-5, f)
    opt.summa_ex("ab", st["y"], st["w1"], st["gelu"], M, h, 4 * h, q, i, j, f, bias=st["b1"], pre_act=st["pre"], act=1)
    opt.summa_ex("ab", st["gelu"], st["w2"], st["out"], M, 4 * h, h, q, i, j, f, bias=st["b2"], residual=st["x"])
    opt.summa_ex("abt", st["d_out"], st["w2"], st["d_pre"], M, h, 4 * h, q, i, j, f, gelu_grad_of=st["pre"])
    opt.summa_atb(st["gelu"], st["d_out"], st["d_w2"], 4 * h, M, h, q, i, j, f)
    opt.bias_grad(st["d_out"], st["d_b2"], M, h, q, i, j, f)
    opt.summa_abt(st["d_pre"], st["w1"], st["d_y"], M, 4 * h, h, q, i, j, f)
    opt.summa_atb(st["y"], st["d_pre"], st["d_w1"], h, M, 4 * h, q, i, j, f)
    opt.bias_grad(st["d_pre"], st["d_b1"], M, 4 * h, q, i, j, f)
    opt.layernorm2d_bwd(st["d_y"], st["xhat"], st["rstd"], st["g"], st["d_out"], st["d_x"], st["d_g"], st["d_be"], st["bstats"], M, h, q, i, j, f)


def _run_mlp(case, st):
    _mlp_pass(case, st, case["i"], case["j"])
    return st["outputs"]


def _prepare_linear(case, r):
    K, N, q, i, j = case["k"], case["n"], case["q"], case["i"], case["j"]
    M = case["b"] * case["s"]
    st = {"x": r.normal(M * K), "w": r.normal(K * N, 0.02), "d_y": r.normal(M * N), "bias": r.normal(N, 0.1, torch.float32),
          "y": torch.empty(M * N, dtype=torch.bfloat16, device=DEV), "d_x": torch.empty(M * K, dtype=torch.bfloat16, device=DEV),
          "d_w": torch.empty(K * N, dtype=torch.float32, device=DEV)}
    shapes = (("ab", M, K, N), ("abt", M, N, K), ("atb", K, M, N))
    st["ws"] = torch.empty(max(256, *(opt.summa_workspace_bytes(*x, q, i, j, opt.BF16) for x in shapes)), dtype=torch.uint8, device=DEV)
    st["out"] = {k: _block(st[k], q, i, j) for k in ("y", "d_x", "d_w")}
    return st


def _run_linear(case, st):
    K, N, q, i, j = case["k"], case["n"], case["q"], case["i"], case["j"]
    M = case["b"] * case["s"]
    opt.summa_ex("ab", st["x"], st["w"], st["y"], M, K, N, q, i, j, opt.BF16, bias=st["bias"], ws=st["ws"])
    opt.summa_abt(st["d_y"], st["w"], st["d_x"], M, N, K, q, i, j, opt.BF16, ws=st["ws"])
    opt.summa_ex("atb", st["x"], st["d_y"], st["d_w"], K, M, N, q, i, j, opt.BF16, out_fp32=True, ws=st["ws"])
    return st["out"]


def _prepare_attention(case, r):
    b, s, h, n, q = (case[k] for k in "bshnq")
    M = b * s
    bf = torch.bfloat16
    st = {"qkv": r.normal(3 * M * h), "d_attn": r.normal(M * h), "attn": torch.empty(M * h, dtype=bf, device=DEV),
          "d_qkv": torch.empty(3 * M * h, dtype=bf, device=DEV), "lse": torch.empty(b * n * s, dtype=torch.float32, device=DEV),
          "ws": torch.empty(opt.attention_fused_workspace_bytes(b, s, h, n, q), dtype=torch.uint8, device=DEV)}
    st["out"] = {k: _block(st[k], q, case["i"], case["j"]) for k in ("attn", "lse", "d_qkv")}
    return st


def _run_attention(case, st):
    b, s, h, n, q = (case[k] for k in "bshnq")
    where = (b, s, h, n, q, case["i"], case["j"], case["causal"], opt.BF16)
    opt.attention_fused_fwd(st["qkv"], st["attn"], st["lse"], *where)
    opt.attention_fused_bwd(st["qkv"], st["attn"], st["lse"], st["d_attn"], st["d_qkv"], *where, st["ws"])
    return st["out"]


_KINDS = {
    "layer": (_prepare_layer, _run_layer), "stack": (_prepare_stack, _run_stack), "ends": (_prepare_ends, _run_ends),
    "mlp": (_prepare_mlp, _run_mlp), "linear": (_prepare_linear, _run_linear), "attention": (_prepare_attention, _run_attention),
}


def prepare(case, seed):
    """Inputs, weights, resident peers and buffers of a case, on the GPU, from the seed alone."""
    state = _KINDS[case["kind"]][0](case, _Rand(seed))
    return {"case": case, "state": state}


def run(st):
    """One pass through the public entry points; the outputs are the state's own buffers."""
    case = st["case"]
    return _KINDS[case["kind"]][1](case, st["state"])


# ------------------------------------------------------------------------------------------------ the same in 64 bits
def _logical(t, rows, cols, q):
    """Block-major [q][q][rows/q][cols/q] -> [rows, cols] in 64 bits."""
    return t.view(q, q, rows // q, cols // q).permute(0, 2, 1, 3).reshape(rows, cols).double()


def _part(T, q, i, j):
    """What device (i, j) holds of a matrix, or the whole of it block-major (i < 0), flat."""
    r, c = T.shape[0] // q, T.shape[1] // q
    blocks = T.view(q, r, q, c).permute(0, 2, 1, 3)
    return (blocks if i < 0 else blocks[i, j]).reshape(-1)


def _column_sums(T, q, i, j):
    """Sums over each device's own rows: the partial vector gradients, [q][q][cols/q] flat or device (i, j)'s."""
    sums = T.view(q, T.shape[0] // q, q, T.shape[1] // q).sum(dim=1)
    return (sums if i < 0 else sums[i, j]).reshape(-1)


def _norm64(x, gamma, beta, eps=1e-5):
    rstd = torch.rsqrt(x.var(dim=1, unbiased=False, keepdim=True) + eps)
    xhat = (x - x.mean(dim=1, keepdim=True)) * rstd
    return xhat * gamma + beta, xhat, rstd


def _norm_bwd64(dy, xhat, rstd, gamma):
    g = dy * gamma
    return rstd * (g - xhat * (xhat * g).mean(dim=1, keepdim=True) - g.mean(dim=1, keepdim=True))


def _gelu64(z):
    return 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))


def _gelu_grad64(z):
    return 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)


def _attention64(qkv, b, s, heads, causal, d_attn=None):
    """[b*s, 3*heads*d] with columns (head, {Q, K, V}, d): attention output and log-sum-exp, or the gradient for qkv."""
    d = qkv.shape[1] // (3 * heads)
    mask = torch.ones(s, s, dtype=torch.bool, device=DEV).triu(1) if causal else None
    outs, lses = [], []
    for seq in range(b):
        Q, K, V = qkv[seq * s:(seq + 1) * s].view(s, heads, 3, d).permute(2, 1, 0, 3)
        S = torch.matmul(Q, K.transpose(1, 2)) / math.sqrt(d)
        if causal:
            S.masked_fill_(mask, -math.inf)
        lse = torch.logsumexp(S, dim=2)
        P = S.sub_(lse[:, :, None]).exp_()
        if d_attn is None:
            outs.append(torch.matmul(P, V).permute(1, 0, 2).reshape(s, heads * d))
            lses.append(lse)
            continue
        dO = d_attn[seq * s:(seq + 1) * s].view(s, heads, d).permute(1, 0, 2)
        dV = torch.matmul(P.transpose(1, 2), dO)
        dP = torch.matmul(dO, V.transpose(1, 2))
        dS = P * (dP - (dP * P).sum(dim=2, keepdim=True))
        dQ, dK = torch.matmul(dS, K) / math.sqrt(d), torch.matmul(dS.transpose(1, 2), Q) / math.sqrt(d)
        outs.append(torch.stack((dQ, dK, dV)).permute(2, 1, 0, 3).reshape(s, 3 * heads * d))
    return (torch.cat(outs), torch.stack(lses)) if d_attn is None else torch.cat(outs)


def _params64(p, h, q):
    out = {name: p[name].double() for name in _VECTORS}
    for name, (rows, cols) in {"w_qkv": (h, 3 * h), "w_o": (h, h), "w1": (h, 4 * h), "w2": (4 * h, h)}.items():
        out[name] = _logical(p[name], rows, cols, q)
    return out


def _layer_fwd64(x, p, b, s, n, causal):
    t = {}
    t["ln1_out"], t["xhat1"], rstd1 = _norm64(x, p["ln1_g"], p["ln1_b"])
    t["qkv"] = t["ln1_out"] @ p["w_qkv"] + p["b_qkv"]
    t["attn"] = _attention64(t["qkv"], b, s, n, causal)[0]
    t["h_mid"] = x + t["attn"] @ p["w_o"] + p["b_o"]
    t["ln2_out"], t["xhat2"], rstd2 = _norm64(t["h_mid"], p["ln2_g"], p["ln2_b"])
    t["pre_gelu"] = t["ln2_out"] @ p["w1"] + p["b1"]
    t["gelu"] = _gelu64(t["pre_gelu"])
    t["out"] = t["h_mid"] + t["gelu"] @ p["w2"] + p["b2"]
    return t, rstd1, rstd2


def _layer_bwd64(d_out, f, rstd1, rstd2, p, b, s, n, causal):
    """Activation gradients, weight gradients, and the matrices whose column sums are the vector gradients."""
    t, w, v = {}, {}, {}
    w["d_w2"], v["d_b2"] = f["gelu"].T @ d_out, d_out
    t["d_pre_gelu"] = (d_out @ p["w2"].T) * _gelu_grad64(f["pre_gelu"])
    t["d_ln2_out"] = t["d_pre_gelu"] @ p["w1"].T
    w["d_w1"], v["d_b1"] = f["ln2_out"].T @ t["d_pre_gelu"], t["d_pre_gelu"]
    v["d_ln2_g"], v["d_ln2_b"] = t["d_ln2_out"] * f["xhat2"], t["d_ln2_out"]
    t["d_h_mid"] = d_out + _norm_bwd64(t["d_ln2_out"], f["xhat2"], rstd2, p["ln2_g"])
    t["d_attn"] = t["d_h_mid"] @ p["w_o"].T
    w["d_w_o"], v["d_b_o"] = f["attn"].T @ t["d_h_mid"], t["d_h_mid"]
    t["d_qkv"] = _attention64(f["qkv"], b, s, n, causal, t["d_attn"])
    t["d_ln1_out"] = t["d_qkv"] @ p["w_qkv"].T
    w["d_w_qkv"], v["d_b_qkv"] = f["ln1_out"].T @ t["d_qkv"], t["d_qkv"]
    v["d_ln1_g"], v["d_ln1_b"] = t["d_ln1_out"] * f["xhat1"], t["d_ln1_out"]
    t["d_x"] = t["d_h_mid"] + _norm_bwd64(t["d_ln1_out"], f["xhat1"], rstd1, p["ln1_g"])
    return t, w, v


def _exact_layer(case, r):
    b, s, h, n, q, i, j = (case[k] for k in "bshnqij")
    p = _params64(_layer_params(r, h), h, q)
    x, d_out = _logical(r.normal(b * s * h), b * s, h, q), _logical(r.normal(b * s * h), b * s, h, q)
    f, rstd1, rstd2 = _layer_fwd64(x, p, b, s, n, case["causal"])
    t, w, v = _layer_bwd64(d_out, f, rstd1, rstd2, p, b, s, n, case["causal"])
    return {**{k: _part(T, q, i, j) for k, T in {**f, **t, **w}.items()}, **{k: _column_sums(T, q, i, j) for k, T in v.items()}}


def _exact_stack(case, r):
    b, s, h, n, q, causal = (case[k] for k in ("b", "s", "h", "n", "q", "causal"))
    params = [_params64(_layer_params(r, h), h, q) for _ in range(case["layers"])]
    x, d = _logical(r.normal(b * s * h), b * s, h, q), _logical(r.normal(b * s * h), b * s, h, q)
    kept, out = [], {}
    for p in params:
        kept.append(_layer_fwd64(x, p, b, s, n, causal))
        x = kept[-1][0]["out"]
    out["out"] = _part(x, q, -1, -1)
    for layer in reversed(range(len(params))):
        t, w, v = _layer_bwd64(d, *kept.pop(), params[layer], b, s, n, causal)
        d = t["d_x"]
        out.update({f"{k}.{layer}": _part(T, q, -1, -1) for k, T in w.items()})
        out.update({f"{k}.{layer}": _column_sums(T, q, -1, -1) for k, T in v.items()})
    out["d_x"] = _part(d, q, -1, -1)
    return out


def _exact_ends(case, r):
    b, s, h, v, q, i, j = (case[k] for k in "bshvqij")
    M, dt = b * s, torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    tokens, labels = r.zipf(M, v).long(), r.zipf(M, v).long()
    table, hidden = _logical(r.normal(v * h, 0.02, dt), v, h, q), _logical(r.normal(M * h, 1.0, dt), M, h, q)
    d_x = _logical(r.normal(M * h, 1e-3, dt), M, h, q)
    logits = hidden @ table.T
    lse = torch.logsumexp(logits, dim=1)
    at = torch.arange(M, device=DEV)
    loss = lse - logits[at, labels]
    d_logits = torch.exp(logits - lse[:, None])
    d_logits[at, labels] -= 1.0
    d_logits /= M
    rows = slice(i * (M // q), (i + 1) * (M // q))   # every device of a grid row holds its rows' losses
    mats = {"x": table[tokens], "logits": logits, "d_logits": d_logits, "d_hidden": d_logits @ table, "d_table_head": d_logits.T @ hidden,
            "d_table": torch.zeros(v, h, dtype=torch.float64, device=DEV).index_add_(0, tokens, d_x)}
    return {**{k: _part(T, q, i, j) for k, T in mats.items()}, "loss": loss[rows], "lse": lse[rows]}


def _exact_mlp(case, r):
    b, s, h, q, i, j = (case[k] for k in "bshqij")
    M, f32 = b * s, torch.float32
    x, d_out = _logical(r.normal(M * h, 1.0, f32), M, h, q), _logical(r.normal(M * h, 1.0, f32), M, h, q)
    w1, w2 = _logical(r.normal(4 * h * h, 0.02, f32), h, 4 * h, q), _logical(r.normal(4 * h * h, 0.02, f32), 4 * h, h, q)
    b1, b2 = r.normal(4 * h, 0.1, f32).double(), r.normal(h, 0.1, f32).double()
    g, be = r.normal(h, 0.1, f32, 1.0).double(), r.normal(h, 0.1, f32).double()
    y, xhat, rstd = _norm64(x, g, be)
    pre = y @ w1 + b1
    gelu = _gelu64(pre)
    d_pre = (d_out @ w2.T) * _gelu_grad64(pre)
    d_y = d_pre @ w1.T
    mats = {"y": y, "pre": pre, "gelu": gelu, "out": x + gelu @ w2 + b2, "d_pre": d_pre, "d_y": d_y,
            "d_x": d_out + _norm_bwd64(d_y, xhat, rstd, g), "d_w1": y.T @ d_pre, "d_w2": gelu.T @ d_out}
    sums = {"d_b1": d_pre, "d_b2": d_out, "d_g": d_y * xhat, "d_be": d_y}
    return {**{k: _part(T, q, i, j) for k, T in mats.items()}, **{k: _column_sums(T, q, i, j) for k, T in sums.items()}}


def _exact_linear(case, r):
    M, K, N, q, i, j = case["b"] * case["s"], case["k"], case["n"], case["q"], case["i"], case["j"]
    x, w, d_y = _logical(r.normal(M * K), M, K, q), _logical(r.normal(K * N, 0.02), K, N, q), _logical(r.normal(M * N), M, N, q)
    bias = r.normal(N, 0.1, torch.float32).double()
    return {"y": _part(x @ w + bias, q, i, j), "d_x": _part(d_y @ w.T, q, i, j), "d_w": _part(x.T @ d_y, q, i, j)}


def _exact_attention(case, r):
    b, s, h, n, q, i, j = (case[k] for k in "bshnqij")
    M = b * s
    qkv, d_attn = _block(r.normal(3 * M * h), q, i, j), _block(r.normal(M * h), q, i, j)   # attention is local to the device
    qkv, d_attn = qkv.view(M // q, 3 * h // q).double(), d_attn.view(M // q, h // q).double()
    attn, lse = _attention64(qkv, b // q, s, n // q, case["causal"])
    return {"attn": attn.reshape(-1), "lse": lse.reshape(-1), "d_qkv": _attention64(qkv, b // q, s, n // q, case["causal"], d_attn).reshape(-1)}


def exact(case, seed):
    """What ``run`` returns for these inputs, from the definitions in 64 bits."""
    one = {"layer": _exact_layer, "stack": _exact_stack, "ends": _exact_ends, "mlp": _exact_mlp, "linear": _exact_linear,
           "attention": _exact_attention}[case["kind"]]
    return one(case, _Rand(seed))
