"""The work that a user of this package has it do, as cases that can be timed
and compared: one LoRA linear's training step (forward, then backward) and
forward alone over the layer shapes and token counts of a fine-tuning run, the
same with a quantized frozen base, the frozen LM head's input gradient, the
reduced-vocabulary loss with its gradient, the similarity table behind it, and
the checkpointed step over a chain of linears.

A case is a dict of plain values; `prepare` makes its inputs on the GPU from a
seed, `run` is one pass through the public entry points, `exact` what the pass
returns in 64-bit arithmetic.
"""
from __future__ import annotations

import math

import torch

import paper_2606_19528_amd as lm

BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64
VOCAB = 128256  # the 3B decoder's vocabulary


def _step(name, T, d_in, d_out, r, bits=16, group=0, remat=False, forward_only=False):
    return {"name": name, "kind": "linear", "T": T, "d_in": d_in, "d_out": d_out, "r": r, "bits": bits,
            "group": group, "remat": remat, "forward_only": forward_only}


def listed():
    return [
        # The smallest linear of the workloads: launches and host work count.
        _step("small_linear", 128, 256, 256, 8),
        # Evaluating a short prompt with the adapter in place: forward alone, a
        # handful of tokens against a full square weight.
        _step("eval_prompt", 24, 3072, 3072, 16, forward_only=True),
        # A training step on one short text: an odd number of tokens through an
        # up-projection.
        _step("short_text_up", 203, 3072, 8192, 16),
        # The attention projection of a 3B decoder at an ordinary length.
        _step("q_proj", 1024, 3072, 3072, 16),
        # The narrow key / value projection at the longest context.
        _step("kv_proj", 4096, 3072, 1024, 32),
        # The down-projection at the longest context: the largest layer of the stack.
        _step("down_proj", 4096, 8192, 3072, 32),
        # A wide up-projection of the other model family with a ragged token
        # count, u recomputed in the backward instead of stored.
        _step("up_proj_remat", 1891, 2048, 11008, 8, remat=True),
        # The quantized base the method trains over: INT4 codes, groups of 128.
        _step("gate_proj_int4", 2048, 3072, 8192, 16, bits=4, group=128),
        # The frozen LM head's input gradient over the full vocabulary.
        {"name": "head_dx", "kind": "head_dx", "T": 1024, "d_in": 3072, "d_out": VOCAB, "bits": 16, "group": 0},
        # Reduced-vocabulary loss and gradient: 30 % trainable positions, top 1000.
        {"name": "head_loss", "kind": "head_loss", "T": 4096, "V": VOCAB, "D": 3072, "k": 1000, "trainable": 0.3},
        # The similarity table of the full output embedding (once per model).
        {"name": "similarity_table", "kind": "table", "V": VOCAB, "D": 3072, "k": 1000},
        # The checkpointed step: four MLP pairs, inputs offloaded to the host.
        {"name": "checkpointed_chain", "kind": "chain", "T": 2048, "d": 3072, "hidden": 8192, "pairs": 4, "r": 16},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_DIMS = [256, 1024, 2048, 3072, 8192, 11008]


def _linear_dims(rng, multiple):
    """(d_in, d_out): a layer's, or now and then any that the entry points take."""
    if rng.random() < 0.65:
        d_in, d_out = rng.choice([(256, 256), (3072, 3072), (3072, 1024), (3072, 8192), (8192, 3072), (2048, 2048),
                                  (2048, 256), (2048, 11008), (11008, 2048)])
    else:
        d_in, d_out = (max(8, _log_int(rng, 256, 8192) // 8 * 8) for _ in range(2))
    return -(-d_in // multiple) * multiple, d_out


def draw(rng):
    u = rng.random()
    if u < 0.72:
        quant = u >= 0.52
        bits = rng.choice([4, 4, 8]) if quant else 16
        group = rng.choice([64, 128, 128, 256]) if quant else 0
        d_in, d_out = _linear_dims(rng, group or 8)
        return {"kind": "linear", "T": _log_int(rng, 16, 4096), "d_in": d_in, "d_out": d_out,
                "r": rng.choice([4, 8, 16, 16, 32, 64]), "bits": bits, "group": group,
                "remat": rng.random() < 0.25, "forward_only": rng.random() < 0.2}
    if u < 0.80:
        bits = rng.choice([8, 16])
        return {"kind": "head_dx", "T": _log_int(rng, 64, 1024), "d_in": rng.choice([2048, 3072]),
                "d_out": _log_int(rng, 8192, VOCAB) // 8 * 8, "bits": bits, "group": 128 if bits == 8 else 0}
    if u < 0.88:
        return {"kind": "head_loss", "T": _log_int(rng, 256, 4096), "V": _log_int(rng, 8192, VOCAB),
                "D": rng.choice([2048, 3072]), "k": _log_int(rng, 50, 1000), "trainable": rng.uniform(0.1, 0.6)}
    if u < 0.94:
        return {"kind": "table", "V": _log_int(rng, 3000, 65536), "D": rng.choice([256, 2048, 3072]),
                "k": _log_int(rng, 16, 1000)}
    return {"kind": "chain", "T": _log_int(rng, 128, 2048), "d": rng.choice([1024, 2048, 3072]),
            "hidden": rng.choice([3072, 8192]), "pairs": rng.choice([1, 2, 4]), "r": rng.choice([8, 16, 32])}


# ---- inputs ------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape, std=1.0):
    return (torch.randn(*shape, generator=g, device="cuda", dtype=F32) * std).to(BF16)


def _adapter(g, d_in, d_out, r):
    A = ((torch.rand(r, d_in, generator=g, device="cuda") * 2.0 - 1.0) / math.sqrt(d_in)).to(BF16)
    return A, _randn(g, d_out, r, std=0.02)


def _quantized(g, d_out, d_in, bits, group):
    """Codes, scales and offsets whose weights spread like N(0, 0.02)."""
    levels = 1 << bits
    q = torch.randint(0, levels, (d_out, d_in), generator=g, device="cuda", dtype=torch.uint8)
    codes = q[:, 0::2] | (q[:, 1::2] << 4) if bits == 4 else q
    scale = 0.02 * math.sqrt(12.0) / levels * (0.5 + torch.rand(d_in // group, d_out, generator=g, device="cuda"))
    jitter = 0.25 * (torch.rand(d_in // group, d_out, generator=g, device="cuda") - 0.5)
    offset = -scale * ((levels - 1) / 2.0 + jitter)
    return {"codes": codes.contiguous(), "scale": scale, "offset": offset, "bits": bits}


def _weight(g, c):
    if c["bits"] == 16:
        return _randn(g, c["d_out"], c["d_in"], std=0.02)
    return _quantized(g, c["d_out"], c["d_in"], c["bits"], c["group"])


def _linear_inputs(c, seed):
    g = _gen(seed)
    x = _randn(g, c["T"], c["d_in"])
    W = _weight(g, c)
    A, B = _adapter(g, c["d_in"], c["d_out"], c["r"])
    return {"x": x, "W": W, "A": A, "B": B, "dy": _randn(g, c["T"], c["d_out"])}


def _head_inputs(c, seed):
    """Hidden states, embedding, targets that share neighbourhoods as the
    tokens of one text do, a table of index neighbours, the last positions
    trainable."""
    g = _gen(seed)
    T, V, D, k = c["T"], c["V"], c["D"], c["k"]
    h = _randn(g, T, D)
    W = _randn(g, V, D, std=0.02)
    centres = torch.randint(0, V, (64,), generator=g, device="cuda")
    pick = torch.randint(0, 64, (T,), generator=g, device="cuda")
    off = torch.randint(-32, 33, (T,), generator=g, device="cuda")
    y = ((centres[pick] + off) % V).to(torch.int32)
    n = torch.arange(k, device="cuda", dtype=torch.int32)
    step = (n + 1) // 2 * torch.where(n % 2 == 1, 1, -1).to(torch.int32)
    table = (torch.arange(V, device="cuda", dtype=torch.int32)[:, None] + step[None, :]) % V
    rows = torch.arange(T - _trainable(c), T, device="cuda", dtype=torch.int32)
    return {"h": h, "W": W, "targets": y, "table": table.to(torch.int32).contiguous(), "rows": rows}


def _trainable(c):
    return max(1, int(round(c["T"] * c["trainable"])))


def _chain_dims(c):
    return [c["d"], c["hidden"]] * c["pairs"] + [c["d"]]


def _chain_inputs(c, seed):
    g = _gen(seed)
    dims = _chain_dims(c)
    nodes = []
    for d_in, d_out in zip(dims, dims[1:]):
        W = _randn(g, d_out, d_in, std=0.02)
        A, B = _adapter(g, d_in, d_out, c["r"])
        nodes.append({"W": W, "A": A, "B": B, "scale": 2.0})
    return {"nodes": nodes, "x0": _randn(g, c["T"], dims[0]), "g": _randn(g, c["T"], dims[-1])}


_STREAMS = []


def _copy_stream():
    """The one stream that a program keeps for its host copies."""
    if not _STREAMS:
        _STREAMS.append(torch.cuda.Stream())
    return _STREAMS[0]


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    dev = "cuda"
    if kind == "linear":
        s = _linear_inputs(c, seed)
        T, K, N, r = c["T"], c["d_in"], c["d_out"], c["r"]
        s["y"] = torch.empty(T, N, dtype=BF16, device=dev)
        s["u"] = None if c["remat"] else torch.empty(T, r, dtype=F32, device=dev)
        if not c["forward_only"]:
            s["dx"] = torch.empty(T, K, dtype=BF16, device=dev)
            s["dA"] = torch.empty(r, K, dtype=F32, device=dev)
            s["dB"] = torch.empty(N, r, dtype=F32, device=dev)
        need = max(lm.lora_linear_workspace_bytes(op, T, K, N, r, lm.LORA_BF16)
                   for op in (lm.LORA_OP_FWD, lm.LORA_OP_BWD))
        s["ws"] = torch.empty(max(need, 1), dtype=torch.uint8, device=dev)
    elif kind == "head_dx":
        g = _gen(seed)
        s = {"W": _weight(g, c), "dy": _randn(g, c["T"], c["d_out"])}
        s["dx"] = torch.empty(c["T"], c["d_in"], dtype=BF16, device=dev)
    elif kind == "head_loss":
        s = _head_inputs(c, seed)
        n = s["rows"].numel()
        s["loss"] = torch.empty(n, dtype=F32, device=dev)
        s["total"] = torch.empty(1, dtype=F32, device=dev)
        s["dh"] = torch.empty(c["T"], c["D"], dtype=BF16, device=dev)
    elif kind == "table":
        s = {"W": _randn(_gen(seed), c["V"], c["D"], std=0.02)}
        s["table"] = torch.empty(c["V"], c["k"], dtype=torch.int32, device=dev)
        s["values"] = torch.empty(c["V"], c["k"], dtype=F32, device=dev)
    else:
        s = _chain_inputs(c, seed)
        for nd in s["nodes"]:
            nd["dA"] = torch.empty(nd["A"].shape, dtype=F32, device=dev)
            nd["dB"] = torch.empty(nd["B"].shape, dtype=F32, device=dev)
        ws, stash = lm.lora_ckpt_sizes(s["nodes"], c["T"])
        s["ws"] = torch.empty(ws, dtype=torch.uint8, device=dev)
        s["stash"] = torch.empty(stash, dtype=torch.uint8, pin_memory=True)
        s["out"] = torch.empty_like(s["x0"])
        s["dx0"] = torch.empty_like(s["x0"])
        s["copy"] = _copy_stream()
    s["case"] = c
    return s


# ---- one pass ------------------------------------------------------------------
def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "linear":
        scale = 32.0 / c["r"]
        quant = c["bits"] != 16
        (lm.lora_linear_fwd_q if quant else lm.lora_linear_fwd)(
            s["x"], s["W"], s["A"], s["B"], s["y"], s["u"], scale, ws=s["ws"])
        out = {"y": s["y"]}
        if s["u"] is not None:
            out["u"] = s["u"]
        if not c["forward_only"]:
            (lm.lora_linear_bwd_q if quant else lm.lora_linear_bwd)(
                s["x"], s["W"], s["A"], s["B"], s["u"], s["dy"], s["dx"], s["dA"], s["dB"], scale, ws=s["ws"])
            out.update(dx=s["dx"], dA=s["dA"], dB=s["dB"])
        return out
    if kind == "head_dx":
        (lm.frozen_linear_bwd_dx_q if c["bits"] != 16 else lm.frozen_linear_bwd_dx)(s["dy"], s["W"], s["dx"])
        return s["dx"]
    if kind == "head_loss":
        J, tpos = lm.lm_head_build_vocab(s["table"], c["k"], s["targets"], s["rows"])
        lm.lm_head_reduced_ce(s["h"], s["W"], s["rows"], J, tpos, s["loss"], s["total"], s["dh"],
                              1.0 / s["rows"].numel())
        # (J itself has another length for other inputs; tpos holds each target's place in it.)
        return {"tpos": tpos, "loss": s["loss"], "total": s["total"], "dh": s["dh"]}
    if kind == "table":
        lm.topk_table_build(s["W"], c["k"], s["table"], s["values"])
        return {"table": s["table"], "values": s["values"]}
    main = torch.cuda.current_stream()
    lm.lora_ckpt_forward(s["nodes"], s["x0"], s["out"], s["stash"], s["ws"], main, s["copy"])
    lm.lora_ckpt_backward(s["nodes"], s["g"], s["dx0"], s["stash"], s["ws"], main, s["copy"])
    return {"out": s["out"], "dx0": s["dx0"],
            "grads": [t for nd in s["nodes"] for t in (nd["dA"], nd["dB"])]}


# ---- what a pass cannot do without ------------------------------------------------
def _linear_work(T, K, N, r, bits, group, forward_only=False):
    w = N * K * bits / 8 + (2 * N * (K // group) * 4 if group else 0)
    ad = 2 * r * (K + N)
    nbytes = 2 * T * K + w + ad + 2 * T * N + 4 * T * r
    flops = 2.0 * T * K * N + 2.0 * T * r * (K + N)
    if not forward_only:
        nbytes += 2 * T * N + 2 * T * K + w + ad + 4 * T * r + 2 * T * K + 4 * r * (K + N)
        flops += 2.0 * T * K * N + 4.0 * T * r * (K + N)
    return nbytes, flops


def work(case):
    c = case
    kind = c["kind"]
    if kind == "linear":
        nbytes, flops = _linear_work(c["T"], c["d_in"], c["d_out"], c["r"], c["bits"], c["group"], c["forward_only"])
    elif kind == "head_dx":
        T, K, N = c["T"], c["d_in"], c["d_out"]
        w = N * K * c["bits"] / 8 + (2 * N * (K // c["group"]) * 4 if c["group"] else 0)
        nbytes, flops = 2 * T * N + w + 2 * T * K, 2.0 * T * K * N
    elif kind == "head_loss":
        n, V, D = _trainable(c), c["V"], c["D"]
        J = V * (1.0 - (1.0 - min(1.0, (c["k"] + 64) / V)) ** min(64, n))  # expected size of the union
        nbytes = 2 * n * D + 2 * J * D + 2 * c["T"] * D + 4 * min(n, 64 * 65) * c["k"]
        flops = 4.0 * n * J * D
    elif kind == "table":
        V, D, k = c["V"], c["D"], c["k"]
        nbytes, flops = 2 * V * D + 8 * V * k, float(V) * (V + 1) * D  # each pair of tokens once
    else:
        nbytes = flops = 0
        dims = _chain_dims(c)
        for K, N in zip(dims, dims[1:]):
            b, f = _linear_work(c["T"], K, N, c["r"], 16, 0)
            nbytes += b + 4 * c["T"] * K  # the input to the host and back
            flops += f
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    kind = case["kind"]
    if kind == "table":
        # fp32 sums of bf16 products: neighbours closer than a few 1e-7 may swap
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if kind == "chain":
        return {"rel": 0.02, "max": 0.5}  # bf16 activations and gradients through up to 8 linears
    if kind == "head_loss":
        return {"rel": 8e-3, "max": 0.1}  # dh: a bf16 softmax gradient times bf16 rows, rounded to bf16
    return {"rel": 8e-3, "max": 0.1}      # outputs rounded to bf16; du rounded to bf16 as an operand


# ---- the same in 64 bits -----------------------------------------------------------
def _dense(W, c):
    if c["bits"] == 16:
        return W.to(F64)
    q = W["codes"]
    if c["bits"] == 4:
        q = torch.stack([q & 15, q >> 4], dim=-1).reshape(q.shape[0], -1)
    s = W["scale"].t().to(F64).repeat_interleave(c["group"], dim=1)
    o = W["offset"].t().to(F64).repeat_interleave(c["group"], dim=1)
    return q.to(F64) * s + o


def _linear_exact(x, W, A, B, dy, scale):
    """y, u, dx, dA, dB of one linear; all operands in 64 bits (dy None: forward)."""
    u = x @ A.t()
    y = x @ W.t() + scale * (u @ B.t())
    if dy is None:
        return {"y": y, "u": u}
    du = scale * (dy @ B)
    return {"y": y, "u": u, "dx": dy @ W + du @ A, "dA": du.t() @ x, "dB": scale * (dy.t() @ u)}


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "linear":
        i = _linear_inputs(c, seed)
        v = {k: i[k].to(F64) for k in ("x", "A", "B", "dy")}
        e = _linear_exact(v["x"], _dense(i["W"], c), v["A"], v["B"], None if c["forward_only"] else v["dy"],
                          32.0 / c["r"])
        if c["remat"]:
            del e["u"]
        return e
    if kind == "head_dx":
        g = _gen(seed)
        W = _weight(g, c)
        return _randn(g, c["T"], c["d_out"]).to(F64) @ _dense(W, c)
    if kind == "head_loss":
        i = _head_inputs(c, seed)
        rows = i["rows"].long()
        y = i["targets"].long()[rows]
        J = torch.unique(i["table"].long()[y][:, : c["k"]])
        tpos = torch.searchsorted(J, y)
        h, WJ = i["h"].to(F64)[rows], i["W"][J].to(F64)
        z = h @ WJ.t()
        lse = torch.logsumexp(z, dim=1)
        loss = lse - z.gather(1, tpos[:, None])[:, 0]
        p = torch.exp(z - lse[:, None])
        p[torch.arange(len(rows), device=p.device), tpos] -= 1.0
        dh = torch.zeros(c["T"], c["D"], dtype=F64, device=p.device)
        dh[rows] = (p @ WJ) / len(rows)
        return {"tpos": None, "loss": loss, "total": loss.sum().reshape(1), "dh": dh}
    if kind == "table":
        W = _randn(_gen(seed), c["V"], c["D"], std=0.02).to(F64)
        W = W / W.norm(dim=1, keepdim=True)
        vals = torch.empty(c["V"], c["k"], dtype=F64, device="cuda")
        for r0 in range(0, c["V"], 8192):
            vals[r0 : r0 + 8192] = torch.topk(W[r0 : r0 + 8192] @ W.t(), c["k"], dim=1).values
        return {"table": None, "values": vals}
    i = _chain_inputs(c, seed)
    nodes = [{k: nd[k].to(F64) for k in ("W", "A", "B")} for nd in i["nodes"]]
    xs = [i["x0"].to(F64)]
    for nd in nodes:
        xs.append(xs[-1] @ nd["W"].t() + 2.0 * (xs[-1] @ nd["A"].t()) @ nd["B"].t())
    g, grads = i["g"].to(F64), []
    for x, nd in zip(reversed(xs[:-1]), reversed(nodes)):
        du = 2.0 * (g @ nd["B"])
        grads = [du.t() @ x, 2.0 * (g.t() @ (x @ nd["A"].t()))] + grads
        g = g @ nd["W"] + du @ nd["A"]
    return {"out": xs[-1], "dx0": g, "grads": grads}
