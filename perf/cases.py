"""Performance cases of the group-masked linear layer and the rows around it on one MI355X.

Every case is one call (or one dependent pair of calls) that a mask-learning or inference program makes through the
package's public functions, at sizes of the LLaMA-2-7B and LLaMA-2-13B projections (workloads/configs.py), of the
single-linear workload, or at ragged sizes between them:

  select   the selectors of some decoder layers: hard gate, sparsity budget, straight-through backward with the budget
  step     one masked linear of the student: forward, then dX and dgate (the mask-learning hot path)
  infer    the four stacked projections of one decoder layer of the pruned model (q|k|v, o, gate|up, down), in place
           or from the packed export: 1 .. 16 tokens are decode steps, more are prefill
  distill  the self-distillation loss through the LM head and its gradient
  hyper    the hypernetwork: selector logits, then its backward with the AdamW step on the heads
"""
import math

import torch

import paper_2609_33977_amd as gm

# (d_model, d_ff) of the two models whose projections the workloads use.
MODELS = {"7b": (4096, 11008), "13b": (5120, 13824)}
D13, F13 = MODELS["13b"]
VOCAB = 32000


def _linears(model):
    """(d_out, d_in) of one decoder layer's seven projections: q, k, v, o, gate, up, down."""
    d, f = MODELS[model]
    return [(d, d)] * 4 + [(f, d)] * 2 + [(d, f)]


def _stacked(case):
    """A decoder layer with the projections that read one input stacked: q|k|v, o, gate|up, down."""
    d, f = case["d_model"], case["d_ff"]
    return [(3 * d, d), (d, d), (2 * f, d), (d, f)]


def _layer_groups(model, layers, g, g_out):
    """Selectors of each target linear, `layers` decoder layers back to back."""
    return [(o // g_out) * (i // g) for o, i in _linears(model)] * layers


def listed():
    return [
        # One decoder layer's selectors (790,528): the smallest call of a layer-wise learner; launches count.
        {"name": "select_7b_1_layer", "kind": "select", "model": "7b", "layers": 1, "g": 256, "g_out": 1},
        # All 25.3 M selectors of LLaMA-2-7B: the gate part of every mask-learning step.
        {"name": "select_7b", "kind": "select", "model": "7b", "layers": 32, "g": 256, "g_out": 1},
        # The single-linear workload: a few tiles, bound by latency.
        {"name": "step_1024_t128", "kind": "step", "T": 128, "d_in": 1024, "d_out": 1024, "g": 256, "g_out": 1, "soft": False},
        # An attention projection at the paper's batch of 1 x 2048 tokens.
        {"name": "step_attn_t2048", "kind": "step", "T": 2048, "d_in": 4096, "d_out": 4096, "g": 256, "g_out": 1, "soft": False},
        # An MLP projection at 2 x 2048 tokens: most of the headline step's work is in launches of this shape.
        {"name": "step_gate_t4096", "kind": "step", "T": 4096, "d_in": 4096, "d_out": 11008, "g": 256, "g_out": 1, "soft": False},
        # Relaxed (soft) selectors, ragged token and row counts.
        {"name": "step_ragged_soft", "kind": "step", "T": 1000, "d_in": 2816, "d_out": 2056, "g": 128, "g_out": 1, "soft": True},
        # Square groups (App. C) on an attention projection.
        {"name": "step_square32_t2048", "kind": "step", "T": 2048, "d_in": 4096, "d_out": 4096, "g": 32, "g_out": 32, "soft": False},
        # One generated token through a decoder layer of the pruned model, weights in place.
        {"name": "decode_13b_t1", "kind": "infer", "d_model": D13, "d_ff": F13, "T": 1, "packed": False, "g": 256},
        # Eight sequences decoding together, from the packed export.
        {"name": "decode_13b_t8_packed", "kind": "infer", "d_model": D13, "d_ff": F13, "T": 8, "packed": True, "g": 256},
        # A prompt of 512 tokens through the packed export that the decode steps then use.
        {"name": "prefill_13b_t512_packed", "kind": "infer", "d_model": D13, "d_ff": F13, "T": 512, "packed": True, "g": 256},
        # The distillation loss of one 2048-token sequence through the LM head, loss and gradient.
        {"name": "distill_7b_t2048", "kind": "distill", "N": 2048, "d": 4096, "V": VOCAB, "valid": 1.0},
        # The hypernetwork of LLaMA-2-7B with 32 x 32 groups (6.3 M selectors), one training step.
        {"name": "hyper_7b_square32", "kind": "hyper", "model": "7b", "layers": 32, "g": 32, "g_out": 32, "D": 64, "H": 64},
    ]


SHAPES = [(64, 1), (128, 1), (256, 1), (256, 1), (512, 1), (16, 16), (32, 32), (64, 64), (128, 128)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["select", "step", "step", "step", "infer", "infer", "distill", "hyper"])
    if kind == "select":
        g, g_out = rng.choice([(256, 1), (512, 1), (32, 32), (64, 64), (128, 128)])
        return {"kind": kind, "model": "7b", "layers": _log(rng, 1, 32), "g": g, "g_out": g_out}
    if kind == "step":
        g, g_out = rng.choice(SHAPES)
        w = max(g, 64)
        while True:
            T, d_in, d_out = _log(rng, 100, 4096), _log(rng, 1024, 11008) // w * w, _log(rng, 1024, 11008)
            d_out = d_out // max(8, g_out) * max(8, g_out)
            if d_in >= w and d_out * d_in <= 4096 * 11008:
                break
        return {"kind": kind, "T": T, "d_in": d_in, "d_out": d_out, "g": g, "g_out": g_out, "soft": rng.random() < 0.2}
    if kind == "infer":
        T = rng.choice([1, rng.randint(2, 16), rng.randint(2, 16), _log(rng, 17, 512)])
        g = rng.choice([64, 128, 256, 256, 512])
        w = max(g, 256)
        return {"kind": kind, "d_model": rng.randint(2048, D13) // w * w, "d_ff": rng.randint(5120, F13) // w * w, "T": T,
                "packed": rng.random() < 0.5, "g": g}
    if kind == "distill":
        return {"kind": kind, "N": _log(rng, 128, 2048), "d": rng.choice([2048, 4096, 2080]),
                "V": rng.choice([VOCAB, 8 * rng.randint(1000, 4000)]), "valid": rng.choice([1.0, 0.8])}
    g, g_out = rng.choice([(32, 32), (64, 64), (64, 64), (128, 128)])
    H = rng.choice([32, 64, 64, 128])
    layers = rng.randint(4, 16 if H == 128 and g == 32 else 32)
    return {"kind": "hyper", "model": "7b", "layers": layers, "g": g, "g_out": g_out,
            "D": rng.choice([32, 64, 100]), "H": H}


# ---------------------------------------------------------------- inputs

def _gen(seed, dev="cuda"):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    return g


def _normal(gen, shape, std=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * std).to(dtype)


def _uniform(gen, shape, lo=0.0, hi=1.0):
    return torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32) * (hi - lo) + lo


def _bf16(*shape):
    return torch.empty(shape, device="cuda", dtype=torch.bfloat16)


def _f32(*shape):
    return torch.empty(shape, device="cuda", dtype=torch.float32)


def _mask(gen, rows, cols, soft=False):
    """Independent selectors, half of them kept; soft: relaxed values, one in eight of them zero."""
    u = torch.rand((rows, cols), generator=gen, device="cuda", dtype=torch.float32)
    if not soft:
        return (u < 0.5).float()
    return torch.where(u < 0.125, torch.zeros_like(u), torch.sigmoid((u - 0.5) * 6.0))


def _ws(nbytes):
    return torch.empty(nbytes, device="cuda", dtype=torch.uint8) if nbytes else None


def _select_inputs(case, seed):
    gen = _gen(seed)
    groups = _layer_groups(case["model"], case["layers"], case["g"], case["g_out"])
    offsets = [0]
    for n in groups:
        offsets.append(offsets[-1] + n)
    params = [o * i for o, i in _linears(case["model"])] * case["layers"]
    n = offsets[-1]
    return {
        "offsets": torch.tensor(offsets, device="cuda", dtype=torch.int64),
        "params": torch.tensor(params, device="cuda", dtype=torch.int64),
        "logits": _normal(gen, (n,), dtype=torch.float32),
        "noise": _uniform(gen, (n,), 1e-6, 1.0 - 1e-6),
        "dgate": _normal(gen, (n,), 0.1, torch.float32),
    }


def _step_inputs(case, seed):
    gen = _gen(seed)
    T, d_in, d_out, g, go = case["T"], case["d_in"], case["d_out"], case["g"], case["g_out"]
    return {
        "X": _normal(gen, (T, d_in)),
        "W": _normal(gen, (d_out, d_in), 0.02),
        "dY": _normal(gen, (T, d_out)),
        "mask": _mask(gen, d_out // go, d_in // g, case["soft"]),
    }


def _infer_inputs(case, seed):
    gen = _gen(seed)
    out = []
    for d_out, d_in in _stacked(case):
        out.append({"X": _normal(gen, (case["T"], d_in)), "W": _normal(gen, (d_out, d_in), 0.02),
                    "mask": _mask(gen, d_out, d_in // case["g"])})
    return out


def _distill_inputs(case, seed):
    gen = _gen(seed)
    N, d, V = case["N"], case["d"], case["V"]
    ht = torch.randn((N, d), generator=gen, device="cuda")
    hs = ht + 0.3 * torch.randn((N, d), generator=gen, device="cuda")
    valid = None
    if case["valid"] < 1.0:
        valid = (torch.rand(N, generator=gen, device="cuda") < case["valid"]).to(torch.uint8)
    return {"Ht": ht.bfloat16(), "Hs": hs.bfloat16(), "W": _normal(gen, (V, d), 3.0 / math.sqrt(d)), "valid": valid}


def _hyper_inputs(case, seed):
    gen = _gen(seed)
    groups = _layer_groups(case["model"], case["layers"], case["g"], case["g_out"])
    L, D, H, G = len(groups), case["D"], case["H"], sum(groups)
    offsets = [0]
    for n in groups:
        offsets.append(offsets[-1] + n)
    s, a = 1.0 / math.sqrt(H), 1.0 / math.sqrt(2 * H)
    return {
        "offsets": torch.tensor(offsets, device="cuda", dtype=torch.int64),
        "z": _normal(gen, (L, D), dtype=torch.float32),
        "gru": _uniform(gen, (2 * 3 * H * (D + H + 2),), -s, s),
        "A": _uniform(gen, (G, 2 * H), -a, a),
        "c": _uniform(gen, (G,), -a, a),
        "dlogits": _normal(gen, (G,), 0.01, torch.float32),
        "mA": _normal(gen, (G, 2 * H), 1e-3, torch.float32),
        "vA": _uniform(gen, (G, 2 * H), 1e-7, 1e-5),
        "mc": _normal(gen, (G,), 1e-3, torch.float32),
        "vc": _uniform(gen, (G,), 1e-7, 1e-5),
    }


def prepare(case, seed):
    kind = case["kind"]
    if kind == "select":
        s = _select_inputs(case, seed)
        n, L = s["logits"].numel(), s["params"].numel()
        s.update(mask=_f32(n), soft=_f32(n), dlogits=_f32(n), coeff=_f32(L),
                 kept=torch.empty(L, device="cuda", dtype=torch.int64),
                 loss=torch.empty(1, device="cuda", dtype=torch.float64))
    elif kind == "step":
        s = _step_inputs(case, seed)
        T, d_in, d_out, g, go = case["T"], case["d_in"], case["d_out"], case["g"], case["g_out"]
        s.update(Y=_bf16(T, d_out), dX=_bf16(T, d_in), dgate=_f32(d_out // go, d_in // g),
                 ws_f=_ws(gm.gm_workspace_size(gm.GM_OP_FWD, T, d_in, d_out, g, go)),
                 ws_b=_ws(gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g, go)))
    elif kind == "infer":
        s = {"linears": _infer_inputs(case, seed)}
        T, g = case["T"], case["g"]
        for x in s["linears"]:
            d_out, d_in = x["W"].shape
            x["Y"] = _bf16(T, d_out)
            if case["packed"]:
                cap = int(x["mask"].sum().item())
                x["Wp"], x["scale"] = _bf16(cap, g), _f32(cap)
                x["chunk"] = torch.empty(cap, device="cuda", dtype=torch.int32)
                x["rowptr"] = torch.empty(d_out + 1, device="cuda", dtype=torch.int32)
                gm.gm_pack_rows(x.pop("W"), x.pop("mask"), g, cap, x["Wp"], x["chunk"], x["scale"], x["rowptr"])
            else:
                x["ws"] = _ws(gm.gm_workspace_size(gm.GM_OP_FWD, T, d_in, d_out, g))
    elif kind == "distill":
        s = _distill_inputs(case, seed)
        N, d, V = case["N"], case["d"], case["V"]
        s.update(loss=_f32(1), ce=_f32(N), dHs=_bf16(N, d), ws=_ws(gm.gm_distill_workspace_size(N, d, V)))
    else:
        s = _hyper_inputs(case, seed)
        L, D = s["z"].shape
        G = s["A"].shape[0]
        s.update(logits=_f32(G), dgru=_f32(s["gru"].numel()),
                 ws=_ws(gm.gm_hyper_workspace_size(L, D, case["H"], G)))
    s["case"] = case
    return s


# Table 5 of the paper: temperature, budget weight and target, AdamW.
TAU, LAMBDA, TARGET = 0.4, 16.0, 0.5
ADAMW = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.05, step=10)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "select":
        gm.gm_gate(s["logits"], s["noise"], TAU, True, s["mask"], s["soft"])
        gm.gm_budget_loss(s["mask"], s["offsets"], s["params"], TARGET, LAMBDA, False, s["kept"], s["loss"], s["coeff"])
        gm.gm_gate_bwd_budget(s["dgate"], s["soft"], TAU, s["offsets"], s["coeff"], s["dlogits"])
        return {k: s[k] for k in ("mask", "soft", "kept", "loss", "coeff", "dlogits")}
    if kind == "step":
        g, go = case["g"], case["g_out"]
        gm.gm_masked_linear_fwd(s["X"], s["W"], s["mask"], g, s["Y"], ws=s["ws_f"], g_out=go)
        gm.gm_masked_linear_bwd(s["dY"], s["X"], s["W"], s["mask"], g, s["dX"], s["dgate"], s["ws_b"], g_out=go)
        return {k: s[k] for k in ("Y", "dX", "dgate")}
    if kind == "infer":
        for x in s["linears"]:
            if case["packed"]:
                gm.gm_packed_linear_fwd(x["X"], x["Wp"], x["chunk"], x["scale"], x["rowptr"], x["Y"].shape[1],
                                        case["g"], x["Y"])
            else:
                gm.gm_masked_linear_fwd(x["X"], x["W"], x["mask"], case["g"], x["Y"], ws=x["ws"])
        return [x["Y"] for x in s["linears"]]
    if kind == "distill":
        gm.gm_distill_fwd(s["Ht"], s["Hs"], s["W"], s["valid"], s["loss"], s["ce"], s["ws"])
        gm.gm_distill_bwd(s["W"], s["dHs"], s["ws"])
        return {k: s[k] for k in ("loss", "ce", "dHs")}
    H = case["H"]
    gm.gm_hyper_fwd(s["z"], s["gru"], s["A"], s["c"], s["offsets"], H, s["logits"], s["ws"])
    gm.gm_hyper_bwd(s["dlogits"], s["z"], s["gru"], s["A"], s["c"], s["mA"], s["vA"], s["mc"], s["vc"], H,
                    dgru=s["dgru"], ws=s["ws"], **ADAMW)
    return {k: s[k] for k in ("logits", "dgru", "A", "c", "mA", "vA", "mc", "vc")}


# ---------------------------------------------------------------- work and tolerance

def work(case):
    kind = case["kind"]
    if kind == "select":
        groups = _layer_groups(case["model"], case["layers"], case["g"], case["g_out"])
        n, L = sum(groups), len(groups)
        # in: logits, noise, dgate; out: mask, soft, dlogits (the count and the backward can read what is at hand)
        return {"bytes": 24 * n + 40 * L, "flops": 0}
    if kind == "step":
        T, d_in, d_out, g, go = case["T"], case["d_in"], case["d_out"], case["g"], case["g_out"]
        kept = 0.875 if case["soft"] else 0.5
        groups = (d_out // go) * (d_in // g)
        return {"bytes": 2 * (2 * T * d_in + 2 * T * d_out + d_in * d_out) + 8 * groups,
                "flops": 2.0 * T * d_in * d_out * (2 * kept + 1)}  # forward and dX: kept groups; dgate: every group
    if kind == "infer":
        T, g = case["T"], case["g"]
        b = f = 0.0
        for d_out, d_in in _stacked(case):
            groups = d_out * (d_in // g)
            index = 8 * groups / 2 + 4 * d_out if case["packed"] else 4 * groups
            b += d_out * d_in * 2 * 0.5 + index + 2 * T * (d_in + d_out)
            f += 2.0 * T * d_out * d_in * 0.5
        return {"bytes": b, "flops": f}
    if kind == "distill":
        N, d, V = case["N"], case["d"], case["V"]
        # the head, both hidden states and the gradient; the backward needs its probabilities, but not through memory
        return {"bytes": 2 * V * d + 3 * 2 * N * d + 4 * N, "flops": 3 * 2.0 * N * V * d}
    groups = _layer_groups(case["model"], case["layers"], case["g"], case["g_out"])
    G, L, D, H = sum(groups), len(groups), case["D"], case["H"]
    # heads: read by the forward; then weights and moments read and written once by the backward
    return {"bytes": 4.0 * (G * 2 * H * 7 + G * 9), "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind == "select":
        return {"rel": 1e-6}  # fp32 elementwise, exact counts
    if kind in ("step", "infer"):
        # Outputs rounded once to bf16 (1.7e-3 against 64 bits); soft selectors also round mask times weight.
        return {"rel": 9e-3 if case.get("soft") else 6e-3}
    if kind == "distill":
        return {"rel": 1e-2}  # dz and dH each rounded to bf16
    return {"rel": 1e-5}  # fp32 sums over up to a layer's selectors


# ---------------------------------------------------------------- 64 bits

def _expand(mask, g, go):
    m = mask.double()
    return m.repeat_interleave(g, 1).repeat_interleave(go, 0) if go > 1 else m.repeat_interleave(g, 1)


def _exact_select(case, seed):
    s = _select_inputs(case, seed)
    u = s["noise"].double()
    z = s["logits"].double() + torch.log(u) - torch.log1p(-u)
    y = torch.sigmoid(z / TAU)
    mask = (z > 0).double()
    off = s["offsets"].tolist()
    kept = torch.stack([mask[a:b].sum() for a, b in zip(off, off[1:])])
    G = (s["offsets"][1:] - s["offsets"][:-1]).double()
    p = s["params"].double()
    sp = float(((1 - kept / G) * p).sum() / p.sum())
    r = math.log(sp / TARGET)
    coeff = LAMBDA * (1.0 if r > 0 else -1.0 if r < 0 else 0.0) / sp * (-(p / G) / p.sum())
    per = torch.repeat_interleave(coeff, s["offsets"][1:] - s["offsets"][:-1])
    dl = (s["dgate"].double() + per) * y * (1 - y) / TAU
    return {"mask": mask, "soft": y, "kept": None, "loss": torch.tensor([LAMBDA * abs(r)], dtype=torch.float64),
            "coeff": coeff, "dlogits": dl}


def _exact_step(case, seed):
    s = _step_inputs(case, seed)
    g, go = case["g"], case["g_out"]
    X, W, dY = s["X"].double(), s["W"].double(), s["dY"].double()
    Wm = W * _expand(s["mask"], g, go)
    p = (dY.t() @ X) * W
    d_out, d_in = W.shape
    return {"Y": X @ Wm.t(), "dX": dY @ Wm, "dgate": p.view(d_out // go, go, d_in // g, g).sum((1, 3))}


def _exact_hyper(case, seed):
    s = _hyper_inputs(case, seed)
    H, D, L = case["H"], case["D"], s["z"].shape[0]
    G = s["A"].shape[0]
    off = s["offsets"].tolist()
    z, gru = s["z"].double().cpu(), s["gru"].double().cpu().requires_grad_()
    P = 3 * H * (D + H + 2)
    halves = []
    for d in range(2):  # the recurrence is small: on the CPU, by autograd
        p = gru[d * P:(d + 1) * P]
        wi, wh = p[:3 * H * D].view(3 * H, D), p[3 * H * D:3 * H * (D + H)].view(3 * H, H)
        bi, bh = p[3 * H * (D + H):3 * H * (D + H + 1)], p[3 * H * (D + H + 1):]
        h, hs = torch.zeros(H, dtype=torch.float64), [None] * L
        for t in range(L):
            l = t if d == 0 else L - 1 - t
            gi, gh = wi @ z[l] + bi, wh @ h + bh
            r, u = torch.sigmoid(gi[:H] + gh[:H]), torch.sigmoid(gi[H:2 * H] + gh[H:2 * H])
            n = torch.tanh(gi[2 * H:] + r * gh[2 * H:])
            h = (1 - u) * n + u * h
            hs[l] = h
        halves.append(torch.stack(hs))
    o_cpu = torch.cat(halves, 1)
    o = o_cpu.detach().cuda()
    dl = s["dlogits"].double()
    logits = torch.empty(G, device="cuda", dtype=torch.float64)
    do = torch.empty_like(o)
    b1, b2, lr, wd, eps, step = (ADAMW[k] for k in ("beta1", "beta2", "lr", "weight_decay", "eps", "step"))

    def adamw(p, gr, m, v):
        m, v = b1 * m + (1 - b1) * gr, b2 * v + (1 - b2) * gr * gr
        return p * (1 - lr * wd) - lr * (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + eps), m, v

    A, mA, vA = s["A"], s["mA"], s["vA"]
    out = {k: torch.empty(x.shape, device="cuda", dtype=torch.float64) for k, x in (("A", A), ("mA", mA), ("vA", vA))}
    for l in range(L):  # a layer at a time
        a, b = off[l], off[l + 1]
        Al = A[a:b].double()
        logits[a:b] = Al @ o[l] + s["c"][a:b].double()
        do[l] = dl[a:b] @ Al
        out["A"][a:b], out["mA"][a:b], out["vA"][a:b] = adamw(Al, dl[a:b, None] * o[l], mA[a:b].double(), vA[a:b].double())
    c, mc, vc = adamw(s["c"].double(), dl, s["mc"].double(), s["vc"].double())
    o_cpu.backward(do.cpu())
    return {"logits": logits, "dgru": gru.grad, "c": c, "mc": mc, "vc": vc, **out}


def exact(case, seed):
    kind = case["kind"]
    if kind == "select":
        return _exact_select(case, seed)
    if kind == "step":
        return _exact_step(case, seed)
    if kind == "infer":
        return [x["X"].double() @ (x["W"].double() * _expand(x["mask"], case["g"], 1)).t()
                for x in _infer_inputs(case, seed)]
    if kind == "distill":
        s = _distill_inputs(case, seed)
        W = s["W"].double()
        zt, zs = s["Ht"].double() @ W.t(), s["Hs"].double() @ W.t()
        lt, ls = torch.logsumexp(zt, 1, keepdim=True), torch.logsumexp(zs, 1, keepdim=True)
        pt = torch.exp(zt - lt)
        ce = (pt * (ls - zs)).sum(1)
        ok = torch.ones_like(ce) if s["valid"] is None else (s["valid"] != 0).double()
        nv = float(ok.sum())
        dz = (torch.exp(zs - ls) - pt) * (ok / max(nv, 1.0))[:, None]
        return {"loss": ((ce * ok).sum() / max(nv, 1.0)).view(1), "ce": ce, "dHs": dz @ W}
    return _exact_hyper(case, seed)
