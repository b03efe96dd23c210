"""The work that is timed on one MI355X: what a program that trains one pipeline stage has this library do,
through its public entry points (`binding.Stage`, `binding.op_*`), over the sizes, types and options it takes.

Kinds of a case:
  step       one mini-batch on a stage: reset, M forwards, M recompute+backward calls, flush (last=True: the last
             stage's keeping forward and stored backward); returns outputs, input gradients, parameter gradients
  forward    the M forwards alone (what the next stage waits for)
  attention  attention forward, and with backward=True the backward on its result
  gemm       one of the three products of a linear layer with its fused epilogue
  layernorm  LayerNorm forward, and with backward=True the backward with gamma / beta gradients
  tail       gradient statistics and the Adam update at the end of a mini-batch
"""
import math

import torch

from paper_2111_04007_amd import binding as B
from paper_2111_04007_amd.synth import StageConfig

DT = {"f32": torch.float32, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "bf16": 2}


def _step(name, L, h, heads, s, b, M, dtype, causal=True, f=0, dropout=0.0, group=1, last=False, side=True, kind="step"):
    return {"name": name, "kind": kind, "layers": L, "hidden": h, "heads": heads, "seq": s, "batch": b, "micro_batches": M,
            "mlp": f or 4 * h, "causal": causal, "dtype": dtype, "dropout": dropout, "group": group, "last": last, "side": side}


def listed():
    return [
        # the smallest configuration, fp32: every kernel is tiny, launches and latency count
        _step("tiny-fp32-step", 2, 128, 2, 64, 2, 4, "f32", side=False),
        # one fp32 layer of ordinary size whose sequence length is no multiple of a tile: the 1e-5 path used to check
        # a bf16 run against
        _step("fp32-layer-odd-seq", 1, 768, 12, 500, 2, 1, "f32"),
        # one bf16 layer whose width (25 heads of 64) and sequence length fit no 128-wide tile
        _step("bf16-layer-ragged", 1, 1600, 25, 1000, 2, 1, "bf16"),
        # one BERT-large-shaped layer on the last stage, trained with dropout: keeping forward, stored backward
        _step("bert-large-layer-last-dropout", 1, 1024, 16, 512, 8, 1, "bf16", causal=False, dropout=0.1, last=True),
        # one 2.5B-shaped layer (head dim 96), forward and recompute+backward
        _step("gpt2-2.5b-layer", 1, 1920, 20, 1024, 4, 1, "bf16"),
        # the forwards of the 8.3B-shaped stage: what the next stage waits for
        _step("gpt-8.3b-stage-forward", 3, 3072, 32, 1024, 2, 2, "bf16", kind="forward"),
        # the largest configuration's whole step, weight gradients grouped over its two micro-batches
        _step("gpt-200b-class-stage-step", 2, 8192, 64, 2048, 1, 2, "bf16", group=2),
        # attention alone: short bidirectional forward (head dim 64), long causal backward (head dim 128)
        {"name": "attention-bert-large-forward", "kind": "attention", "dtype": "bf16", "batch": 8, "seq": 512, "heads": 16,
         "dim": 64, "causal": False, "backward": False},
        {"name": "attention-200b-class-backward", "kind": "attention", "dtype": "bf16", "batch": 1, "seq": 2048, "heads": 64,
         "dim": 128, "causal": True, "backward": True},
        # the weight gradient of an 8.3B-shaped MLP matrix, accumulated in fp32
        {"name": "gemm-8.3b-weight-gradient", "kind": "gemm", "dtype": "bf16", "op": 2, "epi": 0, "M": 12288, "N": 3072, "K": 2048},
        # LayerNorm forward and backward over a 2.5B-shaped micro-batch
        {"name": "layernorm-2.5b", "kind": "layernorm", "dtype": "bf16", "rows": 4096, "width": 1920, "backward": True},
        # gradient statistics and optimizer update of one 2.5B-shaped layer (44 M parameters)
        dict(_step("tail-2.5b-layer", 1, 1920, 20, 1024, 1, 1, "bf16", side=False, kind="tail")),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _some(rng, lo, hi, mult):
    """A size in [lo, hi], spread over its logarithm: two in three are multiples of `mult`, the others anything."""
    v = _log(rng, lo, hi)
    return max(mult, v // mult * mult) if rng.random() < 2 / 3 else v


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "forward", "attention", "attention", "gemm", "gemm", "layernorm", "tail"])
    if kind in ("step", "forward", "tail"):
        dtype = "f32" if rng.random() < 0.3 else "bf16"
        even = rng.random() < 0.6
        d = rng.choice((64, 96, 128)) if even else rng.choice((32, 40, 64, 72, 80, 96, 112, 128))
        heads = max(1, min(_log(rng, 2, 40), (1024 if dtype == "f32" else 5120 if even else 1600) // d))
        s = max(1, _log(rng, 128, 2048) // 128) * 128 if even else _log(rng, 30, 1500)
        tokens = _log(rng, 256, 1024 if dtype == "f32" else 6144 if even else 2048)
        c = _step("", rng.randint(1, 2), heads * d, heads, s, max(1, tokens // s), rng.randint(1, 3), dtype, causal=rng.random() < 0.7,
                  dropout=rng.choice((0.0, 0.0, 0.1)) if kind != "tail" else 0.0, group=rng.choice((1, 1, 2)) if kind == "step" else 1,
                  last=kind == "step" and rng.random() < 0.25, side=rng.random() < 0.7, kind=kind)
        del c["name"]
        return c
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    if kind == "attention":
        even = rng.random() < 0.6
        return {"kind": kind, "dtype": dtype, "batch": _log(rng, 1, 8), "seq": _log(rng, 128, 2048) // 128 * 128 if even else _log(rng, 20, 2000),
                "heads": _log(rng, 1, 16 if dtype == "f32" else 32), "dim": rng.choice((64, 96, 128) if even else (32, 40, 64, 72, 80, 96, 112, 128)),
                "causal": rng.random() < 0.6, "backward": rng.random() < 0.5}
    if kind == "gemm":
        hi = 2048 if dtype == "f32" else 12288
        op = rng.randint(0, 2)
        c = {"kind": kind, "dtype": dtype, "op": op, "epi": {0: rng.choice((0, 1, 2)), 1: rng.choice((0, 3)), 2: 0}[op],
             "M": _some(rng, 64, hi, 128), "N": _some(rng, 64, hi, 128), "K": _some(rng, 64, hi, 64)}
        while c["M"] * c["N"] * c["K"] > 4e10:
            c["K"] = c["K"] // 2 // 64 * 64
        return c
    return {"kind": "layernorm", "dtype": dtype, "rows": _log(rng, 64, 16384), "width": _some(rng, 64, 8192, 8), "backward": rng.random() < 0.6}


# ---- inputs -------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)


def _normal(g, shape, dtype, std=1.0, mean=0.0):
    return torch.empty(shape, device="cuda", dtype=torch.float32).normal_(mean, std, generator=g).to(DT[dtype])


PARAMS = ("ln1_g", "ln1_b", "wqkv", "bqkv", "wo", "bo", "ln2_g", "ln2_b", "w1", "b1", "w2", "b2")


def _shapes(c):
    h, f = c["hidden"], c["mlp"]
    return ((h,), (h,), (3 * h, h), (3 * h,), (h, h), (h,), (h,), (h,), (f, h), (f,), (h, f), (h,))


def _stage_inputs(c, seed):
    """Flat parameters, stage inputs and upstream gradients [M, T, h], dropout seed."""
    g = _gen(seed)
    std = 0.02 if c["hidden"] < 8192 else 0.01
    flat = []
    for _ in range(c["layers"]):
        for name, shape in zip(PARAMS, _shapes(c)):
            if len(shape) == 2:
                flat.append(_normal(g, shape, c["dtype"], std).reshape(-1))
            else:
                flat.append(_normal(g, shape, c["dtype"], 0.05, 1.0 if name.endswith("_g") else 0.0))
    act = (c["micro_batches"], c["batch"] * c["seq"], c["hidden"])
    return torch.cat(flat), _normal(g, act, c["dtype"]), _normal(g, act, c["dtype"]), int(seed) * 7919 + 3


def _config(c):
    return StageConfig("case", c["layers"], c["hidden"], c["heads"], c["seq"], c["batch"], c["micro_batches"], c["mlp"], c["causal"],
                       c["dtype"], wgrad_group=c["group"], dropout_p=c["dropout"])


ADAM = {"lr": 1e-4, "beta1": 0.9, "beta2": 0.95, "eps": 1e-8, "weight_decay": 0.01, "grad_scale": 0.125}


def _tail_inputs(c, seed):
    """Master weights, first and second moments, gradients: a mini-batch in the middle of a run."""
    g = _gen(seed)
    n = c["layers"] * sum(math.prod(s) for s in _shapes(c))
    return (_normal(g, n, "f32", 0.02), _normal(g, n, "f32", 1e-3), _normal(g, n, "f32", 1e-3).square_(), _normal(g, n, "f32", 0.05))


def _op_inputs(c, seed):
    g, dt = _gen(seed), c["dtype"]
    if c["kind"] == "attention":
        T, h = c["batch"] * c["seq"], c["heads"] * c["dim"]
        return {"qkv": _normal(g, (T, 3 * h), dt), "dctx": _normal(g, (T, h), dt)}
    if c["kind"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        a, b = {0: ((M, K), (N, K)), 1: ((M, K), (K, N)), 2: ((K, M), (K, N))}[c["op"]]
        return {"a": _normal(g, a, dt), "b": _normal(g, b, dt, 1.0 if c["op"] == 2 else 0.05),
                "bias": _normal(g, (N,), dt, 0.1) if c["op"] == 0 else None,
                "aux_in": _normal(g, (M, N), dt) if c["epi"] >= 2 else None}
    shape = (c["rows"], c["width"])
    return {"x": _normal(g, shape, dt, 1.5, 0.2), "gamma": _normal(g, shape[1:], dt, 0.1, 1.0), "beta": _normal(g, shape[1:], dt, 0.1),
            "dy": _normal(g, shape, dt), "res": _normal(g, shape, dt)}


def prepare(case, seed):
    c = dict(case)
    if c["kind"] in ("step", "forward"):
        params, xs, dys, drop = _stage_inputs(c, seed)
        st = B.Stage(_config(c), "cuda:0", params_flat=params)
        if c["side"]:
            st.set_side_stream(torch.cuda.Stream())
        if c["dropout"] > 0:
            st.set_dropout_seed(drop)
        return {"case": c, "stage": st, "xs": xs, "dys": dys, "ys": torch.empty_like(xs), "dxs": torch.empty_like(xs)}
    if c["kind"] == "tail":
        master, m, v, grads = _tail_inputs(c, seed)
        st = B.Stage(_config(c), "cuda:0", params_flat=master.to(DT[c["dtype"]]))
        st.grads.copy_(grads)
        return {"case": c, "stage": st, "master": master, "m": m, "v": v, "stats": torch.empty(2, device="cuda"), "steps": 100}
    s = {"case": c, **_op_inputs(c, seed)}
    dt = DT[c["dtype"]]
    if c["kind"] == "attention":
        s.update(ctx=torch.empty_like(s["dctx"]), lse=torch.empty(c["batch"] * c["heads"] * c["seq"], device="cuda"),
                 delta=torch.empty(c["batch"] * c["heads"] * c["seq"], device="cuda"), dqkv=torch.empty_like(s["qkv"]))
    elif c["kind"] == "gemm":
        s["out"] = torch.zeros(c["M"], c["N"], device="cuda", dtype=torch.float32 if c["op"] == 2 else dt)
        s["aux_out"] = torch.empty(c["M"], c["N"], device="cuda", dtype=dt) if c["op"] == 0 and c["epi"] == 1 else None
    else:
        s.update(y=torch.empty_like(s["x"]), dx=torch.empty_like(s["x"]), stats=torch.empty(2 * c["rows"], device="cuda"),
                 dgamma=torch.zeros(c["width"], device="cuda"), dbeta=torch.zeros(c["width"], device="cuda"),
                 partial=torch.empty(B.colreduce_scratch_bytes(c["rows"], 2 * c["width"]) // 4, device="cuda"))
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind in ("step", "forward"):
        st, xs, ys, dys, dxs = s["stage"], s["xs"], s["ys"], s["dys"], s["dxs"]
        if kind == "forward":
            for m in range(c["micro_batches"]):
                st.forward(m, xs[m], ys[m])
            return {"y": ys}
        st.grad_accum_reset()
        if c["last"]:
            for m in range(c["micro_batches"]):
                st.forward_keep(m, xs[m], ys[m])
                st.backward_stored(m, dys[m], dxs[m])
        else:
            for m in range(c["micro_batches"]):
                st.forward(m, xs[m], ys[m])
            for m in range(c["micro_batches"]):
                st.backward_recompute(m, dys[m], dxs[m])
        st.grad_flush()
        return {"y": ys, "dx": dxs, "grads": st.grads}
    if kind == "tail":
        s["steps"] += 1
        st = s["stage"]
        st.grad_stats(s["stats"])
        st.adam_step(s["master"], s["m"], s["v"], s["steps"], **ADAM)
        return {"stats": s["stats"], "master": s["master"], "m": s["m"], "v": s["v"], "params": st.params}
    if kind == "attention":
        a = (c["batch"], c["seq"], c["heads"], c["dim"], c["causal"])
        B.op_attention_fwd(s["qkv"], s["ctx"], s["lse"], *a)
        if not c["backward"]:
            return {"ctx": s["ctx"], "lse": s["lse"]}
        B.op_attention_bwd(s["qkv"], s["ctx"], s["lse"], s["dctx"], s["dqkv"], s["delta"], *a)
        return {"ctx": s["ctx"], "lse": s["lse"], "dqkv": s["dqkv"]}
    if kind == "gemm":
        B.op_gemm(c["op"], c["epi"], s["a"], s["b"], s["out"], bias=s["bias"], aux_in=s["aux_in"], aux_out=s["aux_out"],
                  M=c["M"], N=c["N"], K=c["K"])
        return {"out": s["out"], "aux_out": s["aux_out"]}
    B.op_layernorm_fwd(s["x"], s["gamma"], s["beta"], s["y"], s["stats"])
    if not c["backward"]:
        return {"y": s["y"], "stats": s["stats"]}
    B.op_layernorm_bwd(s["dy"], s["x"], s["stats"], s["gamma"], s["res"], s["dx"], s["dgamma"], s["dbeta"], s["partial"])
    return {"y": s["y"], "stats": s["stats"], "dx": s["dx"], "dgamma": s["dgamma"], "dbeta": s["dbeta"]}


# ---- what a pass cannot do without --------------------------------------------------------------------------

def work(case):
    c, z = case, SIZE[case["dtype"]]
    if c["kind"] in ("step", "forward", "tail"):
        h, f, L, M, T = c["hidden"], c["mlp"], c["layers"], c["micro_batches"], c["batch"] * c["seq"]
        n = L * sum(math.prod(s) for s in _shapes(c))
        if c["kind"] == "tail":   # gradients read once, master and moments read and written, parameters written
            return {"bytes": (4 + 24 + z) * n, "flops": 15 * n}
        act = M * T * h * z
        fwd = L * (2.0 * T * h * (4 * h + 2 * f) + 4.0 * T * c["seq"] * h * (0.5 if c["causal"] else 1.0))
        if c["kind"] == "forward":
            return {"bytes": n * z + 3 * act, "flops": M * fwd}
        # forward, recompute (not on the last stage; without the top layer's second MLP product), backward
        units = 3 * fwd if c["last"] else 4 * fwd - 2.0 * T * h * f
        return {"bytes": n * (z + 4) + 5 * act, "flops": M * units}
    if c["kind"] == "attention":
        T, h = c["batch"] * c["seq"], c["heads"] * c["dim"]
        dense = 4.0 * T * c["seq"] * h * (0.5 if c["causal"] else 1.0)
        return {"bytes": T * h * z * (4 + (4 if c["backward"] else 0)) + 4 * c["batch"] * c["heads"] * c["seq"],
                "flops": dense * (3.5 if c["backward"] else 1.0)}
    if c["kind"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        out = 8 if c["op"] == 2 else z * (1 + (c["epi"] > 0))
        return {"bytes": z * (M * K + N * K) + M * N * out, "flops": 2.0 * M * N * K}
    e = c["rows"] * c["width"]
    return {"bytes": e * z * (5 if c["backward"] else 2) + 8 * c["rows"], "flops": e * (24 if c["backward"] else 8)}


def tolerance(case):
    """About four times the distance from the 64-bit result that was measured on listed and drawn cases: fp32 up to
    8e-7 (attention backward and long sums; 1e-6 allowed for), bf16 layers 3e-3 .. 5e-3, bf16 attention 2.4e-3, one
    bf16 rounding 1.7e-3, and the fp32 sums of a bf16 weight gradient 2.7e-7."""
    if case["kind"] == "tail":   # fp32 updates; a bf16 parameter may round to the other neighbour
        return {"rel": 1e-6, "max": 1e-2}
    if case["dtype"] == "f32" or (case["kind"] == "gemm" and case["op"] == 2):
        return {"rel": 5e-6, "max": 5e-4}
    if case["kind"] in ("step", "forward"):
        return {"rel": 2e-2, "max": 0.4}
    if case["kind"] == "attention":
        return {"rel": 1e-2, "max": 0.2}
    return {"rel": 7e-3, "max": 0.1}


# ---- the same results in 64 bits ----------------------------------------------------------------------------

def _words(rows, cols, tag, mb, seed):
    """Random bytes [rows, cols] of the library's documented mask generator (Philox4x32-10, one call per 4x4 patch)."""
    m32 = 0xFFFFFFFF
    c0 = torch.arange((rows + 3) // 4, device="cuda")[:, None]
    c1 = torch.arange((cols + 3) // 4, device="cuda")[None, :]
    c0, c1 = (t.contiguous() for t in torch.broadcast_tensors(c0, c1))
    c2, c3 = torch.full_like(c0, tag), torch.full_like(c0, mb)
    k0, k1 = seed & m32, seed >> 32 & m32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (p1 >> 32 & m32) ^ c1 ^ k0, p1 & m32, (p0 >> 32 & m32) ^ c3 ^ k1, p0 & m32
        k0, k1 = k0 + 0x9E3779B9 & m32, k1 + 0xBB67AE85 & m32
    w = torch.stack([torch.stack([v >> 8 * j & 255 for j in range(4)], -1) for v in (c0, c1, c2, c3)], 1)   # [rows/4, 4, cols/4, 4]
    return w.reshape(w.shape[0] * 4, -1)[:rows, :cols]


def _mask(c, rows, site, layer, mb, seed, cols):
    thr = round(256 * c["dropout"])
    if not thr:
        return None
    return (_words(rows, cols, site + 256 * layer, mb, seed) >= thr).double() * (256 / (256 - thr))


def _norm(x, g, b):
    mu = x.mean(-1, keepdim=True)
    return g * (x - mu) / ((x - mu).square().mean(-1, keepdim=True) + 1e-5).sqrt() + b


def _attend(qkv, batch, seq, heads, causal, mask=None):
    """ctx [T, h] and log-sum-exp [batch, heads, seq] from qkv [T, 3h]."""
    h = qkv.shape[1] // 3
    q, k, v = (t.reshape(batch, seq, heads, h // heads).transpose(1, 2).contiguous() for t in qkv.split(h, 1))
    s = torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(h // heads)
    if causal:
        s = s.masked_fill(torch.ones(seq, seq, dtype=torch.bool, device="cuda").triu(1), -math.inf)
    p = s.softmax(-1)
    if mask is not None:
        p = p * mask.reshape(p.shape)
    return torch.matmul(p, v).transpose(1, 2).reshape(-1, h), s.detach().logsumexp(-1)


def _gelu(u):
    return torch.nn.functional.gelu(u, approximate="tanh")


def _exact_stage(c, seed):
    flat, xs, dys, drop = _stage_inputs(c, seed)
    grad = c["kind"] == "step"
    leaves, at = [], 0
    for _ in range(c["layers"]):
        for shape in _shapes(c):
            n = math.prod(shape)
            leaves.append(flat[at:at + n].double().reshape(shape).requires_grad_(grad))
            at += n
    del flat
    acc, ys, dxs = [None] * len(leaves), [], []
    T, h, rows = c["batch"] * c["seq"], c["hidden"], c["batch"] * c["heads"] * c["seq"]
    for mb in range(c["micro_batches"]):
        x0 = xs[mb].double().requires_grad_(grad)
        x = x0
        for l in range(c["layers"]):
            g1, b1, wqkv, bqkv, wo, bo, g2, b2, w1, bm1, w2, bm2 = leaves[12 * l:12 * l + 12]

            def dropped(v, site):
                k = _mask(c, T, site, l, mb, drop, h)
                return v if k is None else v * k

            ctx, _ = _attend(_norm(x, g1, b1) @ wqkv.t() + bqkv, c["batch"], c["seq"], c["heads"], c["causal"],
                             _mask(c, rows, 0, l, mb, drop, c["seq"]))
            x = x + dropped(ctx @ wo.t() + bo, 1)
            x = x + dropped(_gelu(_norm(x, g2, b2) @ w1.t() + bm1) @ w2.t() + bm2, 2)
        ys.append(x.detach())
        if grad:
            got = torch.autograd.grad(x, [x0] + leaves, dys[mb].double())
            dxs.append(got[0])
            acc = [g if a is None else a + g for a, g in zip(acc, got[1:])]
    if not grad:
        return {"y": torch.stack(ys)}
    return {"y": torch.stack(ys), "dx": torch.stack(dxs), "grads": torch.cat([a.reshape(-1) for a in acc])}


def exact(case, seed):
    c = case
    if c["kind"] in ("step", "forward"):
        return _exact_stage(c, seed)
    if c["kind"] == "tail":
        w, m, v, g = (t.double() for t in _tail_inputs(c, seed))
        stats = torch.stack([g.square().sum(), torch.zeros((), device="cuda").double()])
        lr, b1, b2, eps, wd, gs = (ADAM[k] for k in ("lr", "beta1", "beta2", "eps", "weight_decay", "grad_scale"))
        g = g * gs
        m = b1 * m + (1 - b1) * g
        v = b2 * v + (1 - b2) * g * g
        w = w - lr * ((m / (1 - b1 ** 101)) / ((v / (1 - b2 ** 101)).sqrt() + eps) + wd * w)
        return {"stats": stats, "master": w, "m": m, "v": v, "params": w}
    i = {k: v if v is None else v.double() for k, v in _op_inputs(c, seed).items()}
    if c["kind"] == "attention":
        qkv = i["qkv"].requires_grad_(c["backward"])
        ctx, lse = _attend(qkv, c["batch"], c["seq"], c["heads"], c["causal"])
        out = {"ctx": ctx.detach(), "lse": lse.reshape(-1)}
        if c["backward"]:
            out["dqkv"] = torch.autograd.grad(ctx, qkv, i["dctx"])[0]
        return out
    if c["kind"] == "gemm":
        a, b, aux = i["a"], i["b"], i["aux_in"]
        if c["op"] == 2:
            return {"out": a.t() @ b, "aux_out": None}
        if c["op"] == 1:
            p = a @ b
            if c["epi"] == 3:
                u = aux.requires_grad_(True)
                p = p * torch.autograd.grad(_gelu(u).sum(), u)[0]
            return {"out": p, "aux_out": None}
        u = a @ b.t() + i["bias"]
        return {"out": _gelu(u) if c["epi"] == 1 else u + aux if c["epi"] == 2 else u, "aux_out": u if c["epi"] == 1 else None}
    x, g, b = (i[k].requires_grad_(True) for k in ("x", "gamma", "beta"))
    y = _norm(x, g, b)
    mu = x.detach().mean(-1)
    out = {"y": y.detach(), "stats": torch.cat([mu, 1 / (x.detach().var(-1, unbiased=False) + 1e-5).sqrt()])}
    if c["backward"]:
        dx, dg, db = torch.autograd.grad(y, (x, g, b), i["dy"])
        out.update(dx=dx + i["res"], dgamma=dg, dbeta=db)
    return out
