"""The work that programs have this library do, as cases that can be timed and compared.

A case is a dict of plain values; ``prepare`` makes what a program has in hand before the call (weights on the device,
activations, output buffers, marshalled calls), ``run`` is one pass through the library's entry points, ``exact`` the
same outputs in 64 bits from plain torch.  Kinds of case:

  small    two small linears and the rotary embedding on the second one's heads: what a call costs when there is almost
           no work
  layer    the linears (and the rotation) of decoder layers: one token, a decode batch or a prompt
  mamba    the two projections of Mamba-2 blocks: one token, a batch or a prompt
  bits     the gated MLP's linears with codes of 8, 6 or 3 bits
  head     4-bit embedding rows of a prompt and the 4-bit output head for the tokens that are sampled
  settle   a deployment settles on a rate: compact copies of the MLP's matrices, one of them dequantised

Weights, scales, zero points, activations, positions and index tables have the distributions of ``workloads``: uniform
codes and zero points, scales ~ U(0.005, 0.02) on the 4-bit grid, activations ~ N(0, 1), random kept-pair tables.
"""
import math

import torch

import paper_2512_03383_amd as uq

GROUP = 128
# hidden, intermediate, query heads, key/value heads, rotary base, longest context
MODELS = {"llama3_8b": (4096, 14336, 32, 8, 5.0e5, 8192), "qwen25_7b": (3584, 18944, 28, 4, 1.0e6, 32768)}
HEAD_DIM = 128
VOCAB = {"llama3_8b": 128256}
MAMBA = {"hidden": 2560, "heads": 80, "head_dim": 64, "state": 128}
DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}


def listed():
    return [
        # the smallest calls a program makes: a 1024 x 1024 linear, 8 query heads of 64 channels and their rotation
        {"name": "small_linear_rope", "kind": "small", "N": 1024, "K": 1024, "rate": 15, "M": 1, "heads": 8, "head_dim": 64,
         "dtype": "fp16", "zeros": True},
        # token generation, one request: four decoder layers at 15 %, every fused launch, o_proj on head-interleaved words
        {"name": "llama_decode", "kind": "layer", "model": "llama3_8b", "rate": 15, "M": 1, "dtype": "fp16", "zeros": True,
         "layers": 4, "part": "both", "interleave": True},
        # the same in the paper's own compute type and quantisation scheme (no zero points), the MLP as one call
        {"name": "qwen_decode_bf16", "kind": "layer", "model": "qwen25_7b", "rate": 25, "M": 1, "dtype": "bf16", "zeros": False,
         "layers": 3, "part": "both", "interleave": False},
        # a server that decodes eight requests together
        {"name": "qwen_batch8", "kind": "layer", "model": "qwen25_7b", "rate": 25, "M": 8, "dtype": "fp16", "zeros": True,
         "layers": 3, "part": "both", "interleave": False},
        # a larger decode batch, more pruning, bfloat16
        {"name": "llama_batch48_bf16", "kind": "layer", "model": "llama3_8b", "rate": 35, "M": 48, "dtype": "bf16", "zeros": True,
         "layers": 2, "part": "both", "interleave": False},
        # a state-space model reads a short prompt, heads and state pruned
        {"name": "mamba_prompt", "kind": "mamba", "rate": 15, "M": 333, "dtype": "fp16", "zeros": True, "layers": 2,
         "by_head": True},
        # a prompt of ragged length through an attention block: q, k, v, rotation, o_proj
        {"name": "llama_prompt_attention", "kind": "layer", "model": "llama3_8b", "rate": 15, "M": 1000, "dtype": "bf16",
         "zeros": True, "layers": 1, "part": "attention", "interleave": False},
        # a long prompt through the MLP, where the arithmetic of a prompt is
        {"name": "llama_prompt_mlp", "kind": "layer", "model": "llama3_8b", "rate": 15, "M": 4096, "dtype": "fp16", "zeros": True,
         "layers": 1, "part": "mlp", "interleave": False},
        # an 8-bit model reads a prompt
        {"name": "int8_prompt_mlp", "kind": "bits", "model": "llama3_8b", "bits": 8, "rate": 15, "M": 512, "dtype": "fp16",
         "zeros": True, "layers": 1},
        # a 3-bit model generates a token
        {"name": "int3_decode_mlp", "kind": "bits", "model": "llama3_8b", "bits": 3, "rate": 0, "M": 1, "dtype": "fp16",
         "zeros": True, "layers": 3},
        # both ends of a model: 512 prompt tokens looked up, eight requests sampled
        {"name": "embedding_and_head", "kind": "head", "model": "llama3_8b", "n": 512, "M": 8, "dtype": "fp16", "zeros": True},
        # the bytes of pruned channels given back, and a dequantised copy for a program that wants plain weights
        {"name": "settle_on_a_rate", "kind": "settle", "model": "llama3_8b", "rate": 25, "dtype": "fp16", "zeros": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "layer", "layer", "layer", "layer", "layer", "mamba", "bits", "bits", "head", "settle"])
    c = {"kind": kind, "dtype": rng.choice(["fp16", "fp16", "bf16"]), "zeros": rng.random() < 0.7}
    if kind == "small":
        c.update(N=_log_int(rng, 100, 3000), K=GROUP * rng.randint(1, 24), rate=rng.randint(0, 50), M=_log_int(rng, 1, 16),
                 heads=rng.choice([4, 8, 16]), head_dim=rng.choice([64, 128]))
    elif kind == "layer":
        M = _log_int(rng, 1, 4096)
        model = rng.choice(sorted(MODELS))
        part = rng.choice(["both", "attention", "mlp"]) if M <= 2048 else rng.choice(["attention", "mlp"])
        if model == "qwen25_7b":
            M = min(M, 3000)   # (its MLP is wider: no more work than the largest listed case)
        c.update(model=model, rate=rng.randint(0, 50) if M <= 2048 else rng.randint(15, 50), M=M, layers=2 if M <= 64 else 1,
                 part=part, interleave=model == "llama3_8b" and M <= 2 and rng.random() < 0.7)
    elif kind == "mamba":
        M = _log_int(rng, 1, 2048)
        c.update(rate=rng.randint(0, 50), M=M, layers=3 if M <= 64 else 1, by_head=rng.random() < 0.5)
    elif kind == "bits":
        M = _log_int(rng, 1, 512)
        c.update(model=rng.choice(sorted(MODELS)), bits=rng.choice([8, 6, 3]), rate=rng.randint(0, 50), M=M, layers=2 if M <= 16 else 1)
    elif kind == "head":
        c.update(model="llama3_8b", n=_log_int(rng, 1, 4096), M=_log_int(rng, 1, 64))
    else:
        c.update(model=rng.choice(sorted(MODELS)), rate=rng.randint(5, 50))
    return c


# ---- shapes -------------------------------------------------------------------------------------------------------
def _head_keep(d, rate):
    return 2 * (d * (100 - rate) // 200)


def _rows(n, stride=0, keep=0, limit=0, stride2=0, keep2=0, limit2=0):
    return {"n": n, "rs": (stride, keep, limit), "rs2": (stride2, keep2, limit2)}


def _linears(c):
    """(name, stored rows, stored columns, bits, row rule, column rule) of one layer of the case, in call order."""
    rate, bits = c["rate"], c.get("bits", 4)
    whole, all_cols = _rows(0), (0, 0, 0)
    if c["kind"] == "small":
        D = c["head_dim"]
        return [("linear", c["N"], c["K"], 4, _rows(max(1, c["N"] * (100 - rate) // 100)), all_cols),
                ("heads", c["heads"] * D, c["K"], 4, _rows(0, D // 2, _head_keep(D, rate) // 2, c["heads"] * D), all_cols)]
    if c["kind"] == "mamba":
        hid, H, D, S = MAMBA["hidden"], MAMBA["heads"], MAMBA["head_dim"], MAMBA["state"]
        inner = H * D
        N = 2 * inner + 2 * S + H
        if rate == 0:
            return [("in", N, hid, 4, whole, all_cols), ("out", hid, inner, 4, whole, all_cols)]
        if c["by_head"]:
            Dk, Sk = _head_keep(D, rate), S * (100 - rate) // 100
            return [("in", N, hid, 4, _rows(0, D, Dk, 2 * inner, S, Sk, 2 * inner + 2 * S), all_cols),
                    ("out", hid, inner, 4, whole, (0, D, Dk))]
        k = inner * (100 - rate) // 100
        return [("in", N, hid, 4, _rows(0, inner, k, 2 * inner), all_cols), ("out", hid, inner, 4, whole, (k, 0, 0))]
    hid, inter, Hq, Hkv, _, _ = MODELS[c["model"]]
    D, Dk = HEAD_DIM, _head_keep(HEAD_DIM, rate)
    Ik = inter * (100 - rate) // 100
    part = c.get("part", "mlp")
    out = []
    if part in ("both", "attention"):
        qk = (D // 2, Dk // 2) if rate else (0, 0)
        out += [("q", Hq * D, hid, bits, _rows(0, *qk, Hq * D if rate else 0), all_cols),
                ("k", Hkv * D, hid, bits, _rows(0, *qk, Hkv * D if rate else 0), all_cols),
                ("v", Hkv * D, hid, bits, _rows(0, D, Dk, Hkv * D) if rate else whole, all_cols),
                ("o", hid, Hq * D, bits, whole, (0, D, Dk) if rate else all_cols)]
    if part in ("both", "mlp"):
        out += [("gate", inter, hid, bits, _rows(Ik), all_cols), ("up", inter, hid, bits, _rows(Ik), all_cols),
                ("down", hid, inter, bits, whole, (Ik, 0, 0))]
    return out


def _keep(rows, cols):
    return uq.KeepDesc(rows["n"], cols[0], *rows["rs"], cols[1], cols[2], *rows["rs2"])


def _kept_rows(N, rows):
    r = torch.arange(N)
    (s, k, lim), (s2, k2, lim2) = rows["rs"], rows["rs2"]
    if s == 0:
        return r[: rows["n"] or N]
    lim2 = lim2 if s2 else lim
    m = ((r < lim) & (r % s < k)) | (r >= lim2)
    if s2:
        m |= (r >= lim) & (r < lim2) & ((r - lim) % s2 < k2)
    return r[m]


def _kept_cols(K, cols):
    k = torch.arange(K)
    return k[k % cols[1] < cols[2]] if cols[1] else k[: cols[0] or K]


# ---- inputs -------------------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _weight(g, N, K, bits, dtype, zeros):
    f = 16.0 / (1 << bits)
    q = torch.randint(-2 ** 31, 2 ** 31, (N, K * bits // 32), generator=g, device="cuda", dtype=torch.int32)
    s = torch.empty((N, K // GROUP), device="cuda").uniform_(0.005 * f, 0.02 * f, generator=g).to(dtype)
    z = torch.randint(0, 1 << bits, (N, K // GROUP), generator=g, device="cuda", dtype=torch.uint8) if zeros else None
    return uq.QuantLinear(q, s, z, bits=bits)


def _acts(g, M, K, dtype):
    return torch.randn((M, K), generator=g, device="cuda").to(dtype)


def _inputs(c, seed):
    """Weights and activations of every layer, and the rotation's positions and tables."""
    g, dt = _gen(seed), DTYPES[c["dtype"]]
    layers = []
    for _ in range(c.get("layers", 1)):
        lay = {"W": {}, "x": {}, "keep": {}, "spec": {}}
        for name, N, K, bits, rows, cols in _linears(c):
            lay["W"][name] = _weight(g, N, K, bits, dt, c["zeros"])
            lay["keep"][name], lay["spec"][name] = _keep(rows, cols), (N, K, rows, cols)
            if name in ("k", "v"):
                lay["x"][name] = lay["x"]["q"]
            elif name in ("up", "heads"):
                lay["x"][name] = lay["x"]["gate" if name == "up" else "linear"]
            else:
                lay["x"][name] = _acts(g, c["M"], int(_kept_cols(K, cols).numel()), dt)
        layers.append(lay)
    s = {"layers": layers, "dtype": dt}
    if c["kind"] == "small":
        dk = _head_keep(c["head_dim"], c["rate"])
        s["positions"] = torch.randint(0, 4096, (c["M"],), generator=g, device="cuda", dtype=torch.int32)
        s["table"] = _table(g, c["heads"], c["head_dim"] // 2, dk // 2)
    elif any(n == "q" for n, *_ in _linears(c)):
        ctx, hkv = MODELS[c["model"]][5], MODELS[c["model"]][3]
        # a prompt's tokens follow each other; the requests of a decode batch are each at a place of their own
        s["positions"] = (torch.arange(c["M"], device="cuda", dtype=torch.int32) if c["M"] > 64 else
                          torch.randint(0, ctx, (c["M"],), generator=g, device="cuda", dtype=torch.int32))
        s["table"] = _table(g, hkv, HEAD_DIM // 2, _head_keep(HEAD_DIM, c["rate"]) // 2)
    return s


def _table(g, rows, half, keep):
    return torch.stack([torch.randperm(half, generator=g, device="cuda")[:keep] for _ in range(rows)]).to(torch.int32).contiguous()


def _head_inputs(c, seed):
    g, dt = _gen(seed), DTYPES[c["dtype"]]
    hid = MODELS[c["model"]][0]
    s = {"dtype": dt, "head": _weight(g, VOCAB[c["model"]], hid, 4, dt, c["zeros"])}
    s["table"] = _weight(g, VOCAB[c["model"]], hid, 4, dt, c["zeros"])
    s["ids"] = torch.randint(0, VOCAB[c["model"]], (c["n"],), generator=g, device="cuda", dtype=torch.int32)
    s["x"] = _acts(g, c["M"], hid, dt)
    return s


def _settle_inputs(c, seed):
    g, dt = _gen(seed), DTYPES[c["dtype"]]
    return {"dtype": dt, "mats": [(_weight(g, N, K, 4, dt, c["zeros"]), _keep(rows, cols), (N, K, rows, cols))
                                  for _, N, K, _, rows, cols in _linears(dict(c, part="mlp"))]}


# ---- what a program has in hand, and one pass ---------------------------------------------------------------------
def prepare(case, seed):
    c = case
    if c["kind"] == "head":
        s = _head_inputs(c, seed)
        s["rows"] = torch.empty((c["n"], s["table"].K), dtype=s["dtype"], device="cuda")
        s["logits"] = torch.empty((c["M"], s["head"].N), dtype=s["dtype"], device="cuda")
        s["steps"] = [lambda: uq.uniql_w4_embedding(s["table"], s["ids"], s["rows"]),
                      lambda: uq.uniql_w4_linear(s["head"], None, s["x"], s["logits"])]
        s["outputs"] = [s["rows"], s["logits"]]
        return s
    if c["kind"] == "settle":
        return dict(_settle_inputs(c, seed), steps=None)
    s = _inputs(c, seed)
    s["steps"], s["outputs"] = [], []
    for lay in s["layers"]:
        y = {n: torch.empty((c["M"], int(_kept_rows(N, rows).numel())), dtype=s["dtype"], device="cuda")
             for n, (N, K, rows, cols) in lay["spec"].items()}
        if c["kind"] == "layer":
            _layer_steps(c, s, lay, y)
        else:
            for n in lay["W"]:
                s["steps"].append(_linear_step(lay["W"][n], lay["keep"][n], lay["x"][n], y[n]))
                s["outputs"].append(y[n])
    if c["kind"] == "small":
        heads = y["heads"].view(c["M"], c["heads"], -1)
        s["steps"].append(lambda: uq.uniql_pruned_rope(heads, None, s["positions"], s["table"], c["head_dim"], 1.0e4))
    return s


def _linear_step(W, keep, x, y):
    return lambda: uq.uniql_w4_linear(W, keep, x, y)


def _layer_steps(c, s, lay, y):
    """The calls of one layer, as a decode loop or a prompt runner makes them; marshalled once where the library has a call object."""
    hid, inter, Hq, Hkv, theta, _ = MODELS[c["model"]]
    W, keep, x, M = lay["W"], lay["keep"], lay["x"], c["M"]
    Dk = _head_keep(HEAD_DIM, c["rate"])
    steps, outs = s["steps"], s["outputs"]
    multi = lambda names: uq.MultiCall([W[n] for n in names], [keep[n] for n in names], [x[n] for n in names], [y[n] for n in names]).run  # noqa: E731
    if "q" in W:
        q, k = y["q"].view(M, Hq, Dk), y["k"].view(M, Hkv, Dk)
        if M == 1:
            steps.append(uq.QkvRopeCall([W[n] for n in "qkv"], [keep[n] for n in "qkv"], x["q"][0], q[0], k[0], y["v"][0],
                                        s["positions"], s["table"], HEAD_DIM, theta).run)
        else:
            steps.append(multi("qkv"))
            steps.append(lambda: uq.uniql_pruned_rope(q, k, s["positions"], s["table"], HEAD_DIM, theta))
        if c["interleave"]:
            # head-interleaved words, converted once when the model is loaded
            W = dict(W, o=uq.uniql_w4_interleave(W["o"], Hq))
        steps.append(uq.MultiCall([W["o"]], [keep["o"]], [x["o"]], [y["o"]]).run)
        outs += [q, k, y["v"], y["o"]]
    if "gate" in W:
        n_hidden = y["gate"].shape[1]
        if M == 1 and not c["zeros"]:
            # the whole MLP as one call through a workspace the program keeps
            ws = uq.mlp_workspace(n_hidden)
            steps.append(uq.MlpCall([W[n] for n in ("gate", "up", "down")], [keep[n] for n in ("gate", "up", "down")],
                                    x["gate"][0], y["down"][0], ws).run)
            outs += [uq.mlp_hidden(ws, n_hidden, s["dtype"]), y["down"]]
            return
        if M == 1:
            steps.append(uq.GateUpCall([W["gate"], W["up"]], [keep["gate"], keep["up"]], x["gate"][0], y["gate"][0]).run)
            outs.append(y["gate"])
        elif _glu_batch(c):
            pair, kp = [W["gate"], W["up"]], [keep["gate"], keep["up"]]
            steps.append(lambda: uq.uniql_w4_gate_up_silu_batch(pair, kp, x["gate"], y["gate"]))
            outs.append(y["gate"])
        else:
            steps.append(multi(["gate", "up"]))
            outs += [y["gate"], y["up"]]
        steps.append(uq.MultiCall([W["down"]], [keep["down"]], [x["down"]], [y["down"]]).run)
        outs.append(y["down"])


def _glu_batch(c):
    """Whether the decode batch's gate and up share the launch that also applies the activation (the library refuses others)."""
    inter = MODELS[c["model"]][1]
    return 2 <= c["M"] <= 16 and inter * (100 - c["rate"]) // 100 >= 10225


def run(state):
    if state["steps"] is None:
        out = []
        for W, keep, _ in state["mats"]:
            R, _ = uq.uniql_w4_repack(W, keep)
            out += [t for t in (R.qweight, R.scales, R.zeros) if t is not None]
        W, keep, _ = state["mats"][0]
        return out + [uq.uniql_w4_dequant(W, keep)]
    for step in state["steps"]:
        step()
    return state["outputs"]


# ---- what a pass cannot do without --------------------------------------------------------------------------------
def _matrix_bytes(N, K, bits, rows, cols, zeros):
    n, kc = int(_kept_rows(N, rows).numel()), _kept_cols(K, cols)
    groups = int(torch.unique(kc // GROUP).numel())
    return n * kc.numel() * bits / 8 + n * groups * (2 + (bits / 8 if zeros else 0)), n, int(kc.numel())


def work(case):
    c = case
    total, flops = 0.0, 0.0
    if c["kind"] == "head":
        hid, V = MODELS[c["model"]][0], VOCAB[c["model"]]
        row = hid / 2 + hid / GROUP * (2.5 if c["zeros"] else 2)
        return {"bytes": c["n"] * (row + 4 + 2 * hid) + V * row + 2 * c["M"] * (hid + V), "flops": 2.0 * c["M"] * hid * V}
    if c["kind"] == "settle":
        for i, (_, N, K, bits, rows, cols) in enumerate(_linears(dict(c, part="mlp"))):
            b, n, k = _matrix_bytes(N, K, bits, rows, cols, c["zeros"])
            kg = -(-k // GROUP) * GROUP
            total += b + n * (kg / 2 + kg / GROUP * (3 if c["zeros"] else 2))
            total += b + 2.0 * n * k if i == 0 else 0.0
        return {"bytes": total, "flops": 0.0}
    M, seen = c["M"], set()
    for name, N, K, bits, rows, cols in _linears(c):
        b, n, k = _matrix_bytes(N, K, bits, rows, cols, c["zeros"])
        total += b
        x = {"k": "q", "v": "q", "up": "gate", "heads": "linear"}.get(name, name)
        glu = c["kind"] == "layer" and (M == 1 or _glu_batch(c))
        total += 0 if x in seen else 2.0 * M * k
        seen.add(x)
        total += 0 if (name == "up" and glu) else 2.0 * M * n   # (gate and up leave one hidden vector where they are fused)
        flops += 2.0 * M * n * k
    return {"bytes": total * c.get("layers", 1), "flops": flops * c.get("layers", 1)}


def tolerance(case):
    if case["kind"] == "settle":
        return "exact"   # codes are moved, weights are rounded once by definition
    # 32-bit sums rounded once to 16 bits: about 2^-11 / sqrt 3 (2^-8 / sqrt 3) of the value from the exact result, and
    # another correct implementation differs by an ulp here and there; where q and k are rounded before the rotation
    # as well, by that much more
    return {"rel": 1.2e-3, "max": 6e-3} if case["dtype"] == "fp16" else {"rel": 9e-3, "max": 4e-2}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------
def _codes(W):
    """The codes of a matrix, one per element, from the row-wise little-endian bit stream of its words."""
    w = W.qweight.to(torch.int64) & 0xFFFFFFFF
    if 32 % W.bits == 0:
        sh = torch.arange(0, 32, W.bits, device=w.device)
        return ((w[:, :, None] >> sh) & ((1 << W.bits) - 1)).reshape(W.N, W.K)
    b = torch.arange(W.K, device=w.device) * W.bits
    lo, off = b // 32, b % 32
    hi = torch.clamp(lo + 1, max=w.shape[1] - 1)
    return ((w[:, lo] | (w[:, hi] << 32)) >> off) & ((1 << W.bits) - 1)


def _dense(W, rows=None):
    """Dequantised rows in 64 bits: the 16-bit number nearest to (q - z) * s, which is what a weight is defined to be."""
    if rows is not None:
        W = uq.QuantLinear(W.qweight[rows], W.scales[rows], W.zeros[rows] if W.zeros is not None else None, bits=W.bits)
    z = W.zeros.to(torch.float32) if W.zeros is not None else torch.full_like(W.scales, 1 << (W.bits - 1), dtype=torch.float32)
    q = _codes(W).to(torch.float32).view(W.N, -1, GROUP)
    return ((q - z[:, :, None]) * W.scales.to(torch.float32)[:, :, None]).to(W.scales.dtype).view(W.N, W.K).double()


def _linear64(W, spec, x):
    N, K, rows, cols = spec
    r, k = _kept_rows(N, rows).cuda(), _kept_cols(K, cols).cuda()
    x = x.double()
    return torch.cat([x @ _dense(W, part)[:, k].T for part in r.split(4096)], dim=1)


def _rotate64(v, positions, table, D, theta):
    T, H, Dk = v.shape
    j = table.long().repeat_interleave(H // table.shape[0], 0).double()
    ang = positions.double()[:, None, None] * torch.pow(torch.tensor(theta, dtype=torch.float64, device=v.device), -2.0 * j / D)[None]
    a, b = v[..., : Dk // 2], v[..., Dk // 2:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], dim=-1)


def exact(case, seed):
    c = case
    if c["kind"] == "head":
        s = _head_inputs(c, seed)
        ids = s["ids"].long()
        return [_dense(s["table"], ids), _linear64(s["head"], (s["head"].N, s["head"].K, _rows(0), (0, 0, 0)), s["x"])]
    if c["kind"] == "settle":
        s = _settle_inputs(c, seed)
        moved = 3 if c["zeros"] else 2
        W, _, (N, K, rows, cols) = s["mats"][0]
        return [None] * (moved * len(s["mats"])) + [_dense(W, _kept_rows(N, rows).cuda())[:, _kept_cols(K, cols).cuda()]]
    s = _inputs(c, seed)
    out = []
    for lay in s["layers"]:
        y = {n: _linear64(lay["W"][n], lay["spec"][n], lay["x"][n]) for n in lay["W"] if c["kind"] != "layer" or n != "down"}
        if c["kind"] != "layer":
            out += list(y.values())
            continue
        hid, inter, Hq, Hkv, theta, _ = MODELS[c["model"]]
        if "q" in y:
            Dk = _head_keep(HEAD_DIM, c["rate"])
            out += [_rotate64(y["q"].view(c["M"], Hq, Dk), s["positions"], s["table"], HEAD_DIM, theta),
                    _rotate64(y["k"].view(c["M"], Hkv, Dk), s["positions"], s["table"], HEAD_DIM, theta), y["v"], y["o"]]
        if "gate" in y:
            x = lay["x"]["down"]
            h = torch.nn.functional.silu(y["gate"]) * y["up"]
            if c["M"] == 1 and not c["zeros"]:
                x = h.to(s["dtype"])   # the hidden vector is rounded once on its way, like every activation
                out.append(h[0])
            elif c["M"] == 1 or _glu_batch(c):
                out.append(h)
            else:
                out += [y["gate"], y["up"]]
            out.append(_linear64(lay["W"]["down"], lay["spec"]["down"], x))
    if c["kind"] == "small":
        heads = out[1].view(c["M"], c["heads"], -1)
        out[1] = _rotate64(heads, s["positions"], s["table"], c["head_dim"], 1.0e4).view(c["M"], -1)
    return out
