"""Timed cases of the stage library: whole stage iterations, single layers and single operations, through the public
entry points (paper_2510_05186_amd.stage.Stage and the single-kernel calls of the C ABI), with 64-bit references in
plain torch.

A case is a dict of plain values; "kind" says which entry points it drives:
  stage      one iteration of a stage's event list (F, B, W, with transfers where "offload" is set), as a training loop
             runs it: run, synchronize, reset.  Outputs: every y, every dx, every parameter gradient.
  attention  attention forward and backward of one layer.  Outputs: o, lse, dqkv.
  linear     one linear layer over a batch of tokens: y = r + x W^T, dx = dy W, dW = dy^T x.
  pointwise  norm forward / backward, MLP activation forward / backward, rotary forward / backward of one layer.
  slabs      a layer's weights into the operand layouts the GEMM kernels read, after a weight update.
"""
import math
from types import SimpleNamespace

import torch

from paper_2510_05186_amd import binding as B
from paper_2510_05186_amd.stage import Stage

GPT, LLAMA = 0, 1
FP32, BF16 = 0, 1
EPS, ROPE_BASE = 1e-5, 10000.0
TORCH = {FP32: torch.float32, BF16: torch.bfloat16}


# ---------------------------------------------------------------------------------------------- the cases
def _stage(name, family, dtype, layers, hidden, n_q, n_kv, head_dim, ffn, seq, batch, m, cap, offload=False, recompute=False):
    case = {"kind": "stage", "family": family, "dtype": dtype, "layers": layers, "hidden": hidden, "n_q": n_q, "n_kv": n_kv,
            "head_dim": head_dim, "ffn": ffn, "seq": seq, "batch": batch, "m": m, "cap": cap, "offload": offload,
            "recompute": recompute}
    return dict(case, name=name) if name else case


def _attention(name, dtype, seq, batch, n_q, n_kv, head_dim):
    case = {"kind": "attention", "dtype": dtype, "seq": seq, "batch": batch, "n_q": n_q, "n_kv": n_kv, "head_dim": head_dim}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest iteration a user runs: a two-layer fp32 stage, plain 1F1B with four micro-batches of 128 tokens.
        # Hundreds of launches of a few microseconds each.
        _stage("tiny_fp32_1f1b", GPT, FP32, 2, 256, 4, 4, 64, 1024, 128, 1, 4, 4),
        # a small grouped-query stage under a budget, as a schedule is tried out before the real model runs: ragged 320
        # tokens, every micro-batch's X_IN, QKV and X_MID offloaded to pinned host memory and reloaded
        _stage("small_gqa_offload", LLAMA, BF16, 2, 1024, 8, 2, 128, 1792, 320, 1, 5, 3, offload=True),
        # one layer of the Llama-style stage (hidden 4096), F, B and W of two micro-batches: the ordinary training layer
        _stage("llama_layer", LLAMA, BF16, 1, 4096, 32, 32, 128, 11008, 4096, 1, 2, 2),
        # one layer of the grouped-query stage (hidden 8192, ffn 28672): the largest layer, the headline workload's
        _stage("gqa_layer", LLAMA, BF16, 1, 8192, 64, 8, 128, 28672, 4096, 1, 2, 2),
        # one layer of the GPT-style stage: LayerNorm, GELU, eight sequences of 1024 tokens per micro-batch
        _stage("gpt_layer", GPT, BF16, 1, 2048, 16, 8, 128, 4096, 1024, 8, 2, 2),
        # a layer in 32 bits: a run that checks a bf16 one, or a debugging session
        _stage("fp32_layer", GPT, FP32, 1, 1024, 16, 16, 64, 4096, 512, 1, 2, 2),
        # attention of the long-sequence stage: forward and backward at 16384 tokens
        _attention("attention_16k", BF16, 16384, 1, 40, 40, 128),
        # attention of a ragged batch with grouped heads: a few sequences whose length is a multiple of nothing
        _attention("attention_ragged", BF16, 1237, 3, 16, 4, 128),
        # heads of 64 columns, the other head size the library serves, at a GPT model's ordinary size
        _attention("attention_d64", BF16, 1024, 4, 16, 16, 64),
        # one linear layer over a ragged batch of tokens: forward with the residual, both gradients
        {"name": "linear_ragged", "kind": "linear", "dtype": BF16, "tokens": 1000, "n_in": 1024, "n_out": 3072},
        # everything of a long-sequence layer that is not a matrix product, on a ragged slice of its tokens
        {"name": "pointwise_ragged", "kind": "pointwise", "family": LLAMA, "dtype": BF16, "tokens": 4999, "hidden": 5120, "n_q": 40,
         "n_kv": 40, "head_dim": 128, "ffn": 13824},
        # after the optimizer's step: the Llama-style layer's four weights into the layouts the kernels read
        {"name": "weight_slabs", "kind": "slabs", "hidden": 4096, "qkv": 12288, "ffn": 11008},
    ]


def _log_int(rng, lo, hi, step=1):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step) * step))


def draw(rng):
    kind = rng.choice(["stage", "stage", "stage", "attention", "attention", "linear", "linear", "pointwise", "slabs"])
    dtype = BF16 if rng.random() < 0.8 else FP32
    if kind == "stage":
        family, head_dim = rng.choice([GPT, LLAMA]), rng.choice([128, 128, 64] if dtype == BF16 else [64, 128])
        n_kv = rng.choice([1, 2, 4, 8])
        n_q = n_kv * rng.choice([2, 2, 4]) if head_dim == 128 else n_kv * 2
        most = 4096 if dtype == BF16 and head_dim == 128 else 512
        hidden = _log_int(rng, 256, 4096 if most == 4096 else 1024, 8)
        seq, batch = _log_int(rng, 100, most), rng.choice([1, 1, 2])
        offload = rng.random() < 0.3
        return _stage(None, family, dtype, rng.choice([1, 1, 2]), hidden, n_q, n_kv, head_dim, _log_int(rng, hidden, 4 * hidden, 8),
                      max(100, seq // batch), batch, rng.choice([2, 3]), 2, offload, not offload and rng.random() < 0.3)
    if kind == "attention":
        head_dim = rng.choice([128, 128, 64])
        fast = dtype == BF16 and head_dim == 128
        n_kv = rng.choice([1, 2, 4, 8])
        return _attention(None, dtype, _log_int(rng, 65, 8192 if fast else 1024), rng.choice([1, 2, 3]), n_kv * rng.choice([1, 2, 4]), n_kv, head_dim)
    if kind == "linear":
        most = 8192 if dtype == BF16 else 2048
        return {"kind": kind, "dtype": dtype, "tokens": _log_int(rng, 100, most), "n_in": _log_int(rng, 256, most, 8), "n_out": _log_int(rng, 256, most, 8)}
    if kind == "pointwise":
        n_kv = rng.choice([1, 2, 4, 8, 10])
        hidden = _log_int(rng, 256, 8192 if dtype == BF16 else 4096, 8)
        return {"kind": kind, "family": rng.choice([GPT, LLAMA]), "dtype": dtype, "tokens": _log_int(rng, 100, 8192), "hidden": hidden, "n_q": n_kv * rng.choice([1, 2, 4]),
                "n_kv": n_kv, "head_dim": rng.choice([64, 128]), "ffn": _log_int(rng, hidden, 4 * hidden, 8)}
    hidden = _log_int(rng, 256, 8192, 64)
    return {"kind": kind, "hidden": hidden, "qkv": _log_int(rng, 2 * 128, 3 * hidden, 128), "ffn": _log_int(rng, hidden, 3 * hidden, 128)}


# ---------------------------------------------------------------------------------------------- inputs
def _cfg(case):
    return SimpleNamespace(name="case", family=case["family"], dtype=case["dtype"], n_layers=case["layers"], hidden=case["hidden"],
                           n_q_heads=case["n_q"], n_kv_heads=case["n_kv"], head_dim=case["head_dim"], ffn=case["ffn"],
                           seq=case["seq"], micro_batch=case["batch"], stage_index=0, n_stages=4, n_microbatches=case["m"],
                           norm_eps=EPS, rope_base=ROPE_BASE)


class _Draw:
    """Seeded normal tensors on the device, each with a generator state of its own order."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(0x5EED + 7919 * int(seed))

    def __call__(self, shape, dtype, std=1.0, mean=0.0):
        return (torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32) * std + mean).to(TORCH[dtype])


def _up_width(case):
    return 2 * case["ffn"] if case["family"] == LLAMA else case["ffn"]


def _qkv_width(case):
    return (case["n_q"] + 2 * case["n_kv"]) * case["head_dim"]


def _stage_inputs(case, seed):
    """Weights N(0, 0.02), gains 1 + N(0, 0.02), inputs N(0, 1), output gradients N(0, 1e-3)."""
    d, dt, h = _Draw(seed), case["dtype"], case["hidden"]
    weights = []
    for _ in range(case["layers"]):
        w = {"g1": d((h,), dt, 0.02, 1.0), "wqkv": d((_qkv_width(case), h), dt, 0.02), "wo": d((h, case["n_q"] * case["head_dim"]), dt, 0.02),
             "g2": d((h,), dt, 0.02, 1.0), "wgu": d((_up_width(case), h), dt, 0.02), "wd": d((h, case["ffn"]), dt, 0.02)}
        if case["family"] == GPT:
            w["b1"], w["b2"] = d((h,), dt, 0.02), d((h,), dt, 0.02)
        weights.append(w)
    tokens = case["seq"] * case["batch"]
    io = [(d((tokens, h), dt), d((tokens, h), dt, 1e-3)) for _ in range(case["m"])]
    return weights, io


def _events(case):
    """1F1B with `cap` micro-batches in flight, B and W split.  With transfers: every micro-batch's X_IN, QKV and X_MID
    leave after its F, their bytes count as free one F later, and they come back one op ahead of its B."""
    m, cap, layers, kinds = case["m"], min(case["cap"], case["m"]), range(case["layers"]), ("X_IN", "QKV", "X_MID")
    moves = lambda op, j: [(op, j, l, kinds) for l in layers] if case["offload"] else []  # noqa: E731
    ev, waited, back = [], -1, -1

    def finish(j):
        nonlocal waited, back
        for op, last in (("OWAIT", waited), ("R", back)):
            for k in range(last + 1, j + 1):
                ev.extend(moves(op, k))
        waited, back = max(waited, j), max(back, j)
        ev.extend([("B", j), ("W", j)])

    for j in range(m):
        ev.append(("F", j))
        ev.extend(moves("O", j))
        if j >= 1 and waited < j - 1:
            ev.extend(moves("OWAIT", j - 1))
            waited = j - 1
        if j + 1 >= cap:
            finish(j + 1 - cap)
    for j in range(m + 1 - cap, m):
        finish(j)
    return ev


def prepare(case, seed):
    kind = case["kind"]
    s = SimpleNamespace(case=case, kind=kind, lib=B.lib())
    if kind == "stage":
        weights, io = _stage_inputs(case, seed)
        pool = 0
        if case["offload"]:
            sizes = B.query_sizes(_cfg(case))[2]
            pool = case["m"] * case["layers"] * sum(sizes[k] for k in ("X_IN", "QKV", "X_MID"))
        s.stage = Stage(_cfg(case), host_pool_bytes=pool, recompute=case["recompute"], grad_overwrite=True)
        s.stage.set_weights_device(weights)
        for j, (x, dy) in enumerate(io):
            s.stage.bind(j, x, dy)
        s.events = B.make_events(_events(case))
        return s
    s.stream = torch.cuda.current_stream().cuda_stream
    d = _Draw(seed)
    if kind == "attention":
        dt, rows = case["dtype"], case["seq"] * case["batch"]
        s.qkv = d((rows, _qkv_width(case)), dt)
        s.dout = d((rows, case["n_q"] * case["head_dim"]), dt)
        s.o, s.dqkv = torch.empty_like(s.dout), torch.empty_like(s.qkv)
        s.lse = torch.empty((case["batch"], case["n_q"], case["seq"]), dtype=torch.float32, device="cuda")
        n = s.lib.optstage_op_attn_bwd_ws_floats(case["seq"], case["batch"], case["n_q"], case["n_kv"], case["head_dim"])
        s.ws = torch.empty(max(1, n), dtype=torch.float32, device="cuda")
    elif kind == "linear":
        dt, t, k, n = case["dtype"], case["tokens"], case["n_in"], case["n_out"]
        s.x, s.w, s.r, s.dy = d((t, k), dt), d((n, k), dt, 0.02), d((t, n), dt), d((t, n), dt, 1e-3)
        s.wt = s.w.t().contiguous()                      # the program keeps the transposed copy that dx reads
        s.y, s.dx, s.dw = torch.empty_like(s.r), torch.empty_like(s.x), torch.empty((n, k), dtype=torch.float32, device="cuda")
    elif kind == "pointwise":
        dt, t, h = case["dtype"], case["tokens"], case["hidden"]
        s.x, s.gamma, s.beta = d((t, h), dt, 1.5, 0.2), d((h,), dt, 0.02, 1.0), d((h,), dt, 0.02)
        s.dn, s.dres = d((t, h), dt, 1e-3), d((t, h), dt, 1e-3)
        s.gu, s.da = d((t, _up_width(case)), dt, 1.3), d((t, case["ffn"]), dt, 1e-3)
        s.qkv, s.dqkv = d((t, _qkv_width(case)), dt), d((t, _qkv_width(case)), dt, 1e-3)
        s.n, s.dx, s.a, s.dgu = torch.empty_like(s.x), torch.empty_like(s.x), torch.empty_like(s.da), torch.empty_like(s.gu)
        s.rot, s.drot = torch.empty_like(s.qkv), torch.empty_like(s.qkv)
        s.stats = torch.empty(2 * t, dtype=torch.float32, device="cuda")
        s.partial = torch.empty(2 * min(t, 512) * h, dtype=torch.float32, device="cuda")
        s.dgamma, s.dbeta = (torch.empty(h, dtype=torch.float32, device="cuda") for _ in range(2))
        s.table = torch.empty(t * case["head_dim"], dtype=torch.float32, device="cuda")
        B.check(s.lib.optstage_op_rope_table(s.table.data_ptr(), t, case["head_dim"], ROPE_BASE, s.stream))
    else:
        s.jobs = []
        for w, n, k, code in _slab_jobs(case, d):
            s.jobs.append((w, torch.empty((n + 255) // 256 * 256 * k, dtype=torch.bfloat16, device="cuda"), n, k, code))
    return s


def _slab_jobs(case, d):
    """(weight, N, K, code) of every copy a layer's four weights need: plain or paired forward, transposed backward."""
    h, qkv, f = case["hidden"], case["qkv"], case["ffn"]
    jobs = []
    for rows, cols, fwd in ((qkv, h, 0), (h, h, 0), (2 * f, h, 2), (h, f, 0)):
        w = d((rows, cols), BF16, 0.02)
        jobs += [(w, rows, cols, fwd), (w, cols, rows, 1)]
    return jobs


# ---------------------------------------------------------------------------------------------- one pass
def run(s):
    c, lib, kind = s.case, s.lib, s.kind
    if kind == "stage":
        st = s.stage
        st.run(s.events)
        st.synchronize()
        st.reset()
        return {"y": [st.y[j] for j in range(c["m"])], "dx": [st.dx[j] for j in range(c["m"])], "grads": st.grads}
    p = lambda t: t.data_ptr()  # noqa: E731
    if kind == "attention":
        dims = (c["seq"], c["batch"], c["n_q"], c["n_kv"], c["head_dim"], s.stream)
        B.check(lib.optstage_op_attn_fwd(c["dtype"], p(s.qkv), p(s.o), p(s.lse), *dims))
        B.check(lib.optstage_op_attn_bwd(c["dtype"], p(s.qkv), p(s.o), p(s.dout), p(s.lse), p(s.dqkv), p(s.ws), *dims))
        return {"o": s.o, "lse": s.lse, "dqkv": s.dqkv}
    if kind == "linear":
        dt, t, k, n = c["dtype"], c["tokens"], c["n_in"], c["n_out"]
        B.check(lib.optstage_op_gemm(dt, B.GEMM_NT, B.EPI_RESID, p(s.x), p(s.w), p(s.y), p(s.r), t, n, k, k, k, n, s.stream))
        B.check(lib.optstage_op_gemm(dt, B.GEMM_NT, B.EPI_STORE, p(s.dy), p(s.wt), p(s.dx), 0, t, k, n, n, n, k, s.stream))
        B.check(lib.optstage_op_gemm(dt, B.GEMM_TN, 3, p(s.dy), p(s.x), p(s.dw), 0, n, k, t, n, k, k, s.stream))
        return {"y": s.y, "dx": s.dx, "dw": s.dw}
    if kind == "pointwise":
        dt, fam, t, h, f = c["dtype"], c["family"], c["tokens"], c["hidden"], c["ffn"]
        s.dgamma.zero_()
        s.dbeta.zero_()
        B.check(lib.optstage_op_norm_fwd(dt, fam, p(s.x), p(s.gamma), p(s.beta), p(s.n), p(s.stats), t, h, EPS, s.stream))
        B.check(lib.optstage_op_norm_bwd(dt, fam, p(s.dn), p(s.x), p(s.stats), p(s.gamma), p(s.dres), p(s.dx), p(s.partial),
                                         p(s.dgamma), p(s.dbeta), t, h, s.stream))
        B.check(lib.optstage_op_act_fwd(dt, fam, p(s.gu), p(s.a), t, f, s.stream))
        B.check(lib.optstage_op_act_bwd(dt, fam, p(s.da), p(s.gu), p(s.dgu), t, f, s.stream))
        heads = (t, t, c["n_q"], c["n_kv"], c["head_dim"])
        B.check(lib.optstage_op_rope(dt, p(s.qkv), p(s.rot), p(s.table), *heads, 0, s.stream))
        B.check(lib.optstage_op_rope(dt, p(s.dqkv), p(s.drot), p(s.table), *heads, 1, s.stream))
        out = {"n": s.n, "dx": s.dx, "dgamma": s.dgamma, "a": s.a, "dgu": s.dgu, "rot": s.rot, "drot": s.drot}
        if fam == GPT:
            out["dbeta"] = s.dbeta
        return out
    for w, dst, n, k, code in s.jobs:
        B.check(lib.optstage_op_weight_slabs(p(w), p(dst), n, k, code, s.stream))
    return [dst for _, dst, _, _, _ in s.jobs]


# ---------------------------------------------------------------------------------------------- work
def work(case):
    """Bytes: each input read once, each output written once.  Flops: 2 M N K per product, causal attention 2 s^2 n_q d
    forward and 5 s^2 n_q d backward; the pointwise work has none worth counting."""
    kind = case["kind"]
    if kind == "stage":
        e, tokens, h = (2 if case["dtype"] == BF16 else 4), case["seq"] * case["batch"], case["hidden"]
        params = h * (_qkv_width(case) + case["n_q"] * case["head_dim"] + _up_width(case) + case["ffn"])
        attn = 7.0 * case["batch"] * case["seq"] ** 2 * case["n_q"] * case["head_dim"]
        flops = case["m"] * case["layers"] * (6.0 * tokens * params + attn)
        moved = 0
        if case["offload"]:
            moved = 2.0 * case["m"] * case["layers"] * e * tokens * (2 * h + _qkv_width(case))
        return {"bytes": case["layers"] * params * (e + 4.0) + case["m"] * 4.0 * tokens * h * e + moved, "flops": flops}
    e = 2 if case.get("dtype", BF16) == BF16 else 4
    if kind == "attention":
        rows, q = case["seq"] * case["batch"], case["n_q"] * case["head_dim"]
        return {"bytes": e * rows * (2.0 * _qkv_width(case) + 2.0 * q) + 4.0 * case["batch"] * case["n_q"] * case["seq"],
                "flops": 7.0 * case["batch"] * case["seq"] ** 2 * q}
    if kind == "linear":
        t, k, n = case["tokens"], case["n_in"], case["n_out"]
        return {"bytes": e * (2.0 * t * k + 3.0 * t * n + n * k) + 4.0 * n * k, "flops": 6.0 * t * n * k}
    if kind == "pointwise":
        t = case["tokens"]
        return {"bytes": e * t * (5.0 * case["hidden"] + 2.0 * case["ffn"] + 2.0 * _up_width(case) + 4.0 * _qkv_width(case)), "flops": 0}
    h, qkv, f = case["hidden"], case["qkv"], case["ffn"]
    return {"bytes": 2.0 * 3.0 * h * (qkv + h + 3.0 * f), "flops": 0}


def tolerance(case):
    """Largest relative error (2-norm) against another correct implementation at the same precision: about four times the
    largest distance to the 64-bit reference that any output showed (32 bits 1.3e-6; a bf16 stage 5.5e-3 up to hidden 2048
    and 1.3e-2 at 8192, where more roundings meet in each sum; a single bf16 operation 2.4e-3)."""
    kind = case["kind"]
    if kind == "slabs":
        return "exact"
    if case["dtype"] == FP32:
        return {"rel": 6e-6}
    if kind == "stage":
        return {"rel": 2.2e-2 if case["hidden"] <= 2048 else 5e-2}
    return {"rel": 1e-2}


# ---------------------------------------------------------------------------------------------- 64-bit references
def _norm64(family, x, g, b):
    if family == LLAMA:
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * g
    return torch.nn.functional.layer_norm(x, (x.shape[-1],), g, b, EPS)


def _act64(family, gu):
    if family == GPT:
        return torch.nn.functional.gelu(gu)
    f = gu.shape[-1] // 2
    return torch.nn.functional.silu(gu[:, :f]) * gu[:, f:]


def _rotate64(qkv, seq, n_rot, d, sign):
    rows = qkv.shape[0]
    pos = (torch.arange(rows, device=qkv.device) % seq).double()
    theta = ROPE_BASE ** (-2.0 * torch.arange(d // 2, device=qkv.device).double() / d)
    cos, sin = (f(pos[:, None] * theta[None, :])[:, None, :] for f in (torch.cos, torch.sin))
    heads = qkv.reshape(rows, -1, d)
    lo, hi, sin = heads[:, :n_rot, : d // 2], heads[:, :n_rot, d // 2:], sign * sin
    turned = torch.cat((lo * cos - hi * sin, hi * cos + lo * sin), dim=-1)
    return torch.cat((turned, heads[:, n_rot:]), dim=1).reshape(rows, -1)


def _attend64(qkv, seq, batch, n_q, n_kv, d, want_lse=False):
    """Causal attention over packed rows, a sequence and a head at a time."""
    mask = torch.ones((seq, seq), dtype=torch.bool, device=qkv.device).triu(1)
    out, lses = [], []
    for b in range(batch):
        x = qkv[b * seq:(b + 1) * seq]
        cols = []
        for a in range(n_q):
            g = a * n_kv // n_q
            q, k, v = (x[:, i * d:(i + 1) * d] for i in (a, n_q + g, n_q + n_kv + g))
            scores = ((q @ k.t()) / math.sqrt(d)).masked_fill(mask, float("-inf"))
            if want_lse:
                lses.append(torch.logsumexp(scores, -1))
            cols.append(torch.softmax(scores, -1) @ v)
        out.append(torch.cat(cols, dim=1))
    o = torch.cat(out, dim=0)
    return (o, torch.stack(lses).reshape(batch, n_q, seq)) if want_lse else o


def _layer64(case, w, x):
    fam, nq, nkv, d = case["family"], case["n_q"], case["n_kv"], case["head_dim"]
    qkv = _norm64(fam, x, w["g1"], w.get("b1")) @ w["wqkv"].t()
    if fam == LLAMA:
        qkv = _rotate64(qkv, case["seq"], nq + nkv, d, 1.0)
    mid = x + _attend64(qkv, case["seq"], case["batch"], nq, nkv, d) @ w["wo"].t()
    return mid + _act64(fam, _norm64(fam, mid, w["g2"], w.get("b2")) @ w["wgu"].t()) @ w["wd"].t()


def exact(case, seed):
    kind = case["kind"]
    if kind == "stage":
        weights, io = _stage_inputs(case, seed)
        weights = [{k: t.double().requires_grad_() for k, t in w.items()} for w in weights]
        ys, dxs = [], []
        for x, dy in io:
            x = x.double().requires_grad_()
            y = x
            for w in weights:
                y = _layer64(case, w, y)
            y.backward(dy.double())
            ys.append(y.detach())
            dxs.append(x.grad)
        return {"y": ys, "dx": dxs, "grads": [{k: t.grad for k, t in w.items()} for w in weights]}
    d = _Draw(seed)
    if kind == "attention":
        seq, nq, nkv, hd, rows = case["seq"], case["n_q"], case["n_kv"], case["head_dim"], case["seq"] * case["batch"]
        qkv, dout = d((rows, _qkv_width(case)), case["dtype"]).double(), d((rows, nq * hd), case["dtype"]).double()
        o, lse, dqkv = torch.empty_like(dout), torch.empty((case["batch"], nq, seq), dtype=torch.float64, device="cuda"), torch.zeros_like(qkv)
        for b in range(case["batch"]):                   # one head at a time, so that only its scores are held
            for a in range(nq):
                g, r = a * nkv // nq, slice(b * seq, (b + 1) * seq)
                at = torch.cat([torch.arange(i * hd, (i + 1) * hd, device="cuda") for i in (a, nq + g, nq + nkv + g)])
                x = qkv[r][:, at].requires_grad_()
                oh, lh = _attend64(x, seq, 1, 1, 1, hd, want_lse=True)
                oh.backward(dout[r, a * hd:(a + 1) * hd])
                o[r, a * hd:(a + 1) * hd], lse[b, a] = oh.detach(), lh.detach()[0, 0]
                dqkv[r] = dqkv[r].index_add(1, at, x.grad)
        return {"o": o, "lse": lse, "dqkv": dqkv}
    if kind == "linear":
        dt, t, k, n = case["dtype"], case["tokens"], case["n_in"], case["n_out"]
        x, w, r, dy = (v.double() for v in (d((t, k), dt), d((n, k), dt, 0.02), d((t, n), dt), d((t, n), dt, 1e-3)))
        return {"y": r + x @ w.t(), "dx": dy @ w, "dw": dy.t() @ x}
    if kind == "pointwise":
        s, fam = prepare(case, seed), case["family"]
        x, g, b, gu = (v.double().requires_grad_() for v in (s.x, s.gamma, s.beta, s.gu))
        n, a = _norm64(fam, x, g, b), _act64(fam, gu)
        n.backward(s.dn.double())
        a.backward(s.da.double())
        heads = (case["tokens"], case["n_q"] + case["n_kv"], case["head_dim"])
        out = {"n": n.detach(), "dx": s.dres.double() + x.grad, "dgamma": g.grad, "a": a.detach(), "dgu": gu.grad,
               "rot": _rotate64(s.qkv.double(), *heads, 1.0), "drot": _rotate64(s.dqkv.double(), *heads, -1.0)}
        if fam == GPT:
            out["dbeta"] = b.grad
        return out
    out = []
    for w, n, k, code in _slab_jobs(case, d):
        w = w.double()
        if code == 1:
            w = w.t()
        elif code == 2:                                  # 64 gate rows beside the 64 matching up rows
            w = w.reshape(2, n // 256, 2, 64, k).permute(1, 2, 0, 3, 4).reshape(n, k)
        w = torch.nn.functional.pad(w, (0, 0, 0, -n % 256))
        out.append(w.reshape(-1, 256, k // 64, 64).permute(0, 2, 1, 3).reshape(-1).contiguous())
    return out
