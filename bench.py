#!/usr/bin/env python3
"""Throughput of the group-masked linear layer's mask-learning step on one MI355X.

A step is one pass of the whole hot path over one batch: gate (Gumbel-Sigmoid,
hard STE forward) -> masked forward -> backward (dX and dgate) -> gate backward.
The headline workload is the whole LLaMA-2-7B mask-learning step: all 224
masked linears (32 layers x q, k, v, o 4096x4096, gate, up 11008x4096, down
4096x11008), T = 4096 tokens (2 x 2048), 1x256 groups, per-matrix budgets from
a Beta(2,2) law rescaled to 50 % of the 25,296,896 groups, one gate and one
STE call over all selectors.

Counted work per step: kept FLOPs 2*T*nnz for the forward and for dX, dense
FLOPs 2*T*d_out*d_in for dgate (every selector receives a gradient).  Inputs
are seeded synthetic tensors resident in HBM before timing starts; the gate
inputs are independent draws (logits ~ N(0,1), u ~ U(0,1)) shifted per matrix,
with the library's own gate deciding, so that each matrix keeps its budget.

The JSON line also carries the roofline of the dominant kernel (dgate), the
gate's HBM bandwidth over all 25.3 M selectors with its near-threshold count,
the fp64 oracle timed on the host cores (every workload, sampled where stated),
the single-linear latency, the LLaMA-2-7B attention projection and MLP-trio
steps, the decode GEMV bandwidth on LLaMA-2-13B shapes, the LLaMA-2-13B group
size sweep and T = 512 forward, the sparsity-budget regulariser, square
groups, the distillation loss and the hypernetwork.

`--summarize-trace CSV` and `--summarize-counters CSV` print the rocprofv3
kernel-trace and counter summaries that profiles/ holds (per kernel and grid).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0       # MI355X HBM3E

HERE = os.path.dirname(os.path.abspath(__file__))
GEMM_SOURCES = ["paper_2609_33977_amd/csrc/gemm.hip", "paper_2609_33977_amd/csrc/gm_gemm.h", "paper_2609_33977_amd/csrc/gm_pipe.h",
                "paper_2609_33977_amd/csrc/gm_device.h", "paper_2609_33977_amd/csrc/gm_lists.h",
                "paper_2609_33977_amd/csrc/gm_dgate.h", "paper_2609_33977_amd/csrc/gm_plan.h"]

# HBM traffic of the roofline kernel, dgate_kernel<256, 1>, averaged over the
# launches of the headline step (128 of 4096x4096, 64 of 11008x4096, 32 of
# 4096x11008), from rocprofv3 --pmc FETCH_SIZE and --pmc WRITE_SIZE runs (KiB
# per dispatch), calibrated with a device-to-device copy of known size measured
# by the same counters (FETCH_SIZE read 0.5x and WRITE_SIZE 1.0x of the copied
# bytes).  The numbers describe the kernel built from sources whose code (comments
# excluded) has this digest, and are reported only while the sources still match
# it (None: not measured).
DGATE_TRAFFIC = {"sources_sha256": "b9bb1b66fc6d192e4b31caf9a11c9e487aa8acaeac16135cbeb6cf77bda25615",
                 "launch_mix": "separate", "fetch_kib": 218516.1, "write_kib": 596.4, "fetch_scale": 2.0, "write_scale": 1.0}


def _progress(msg: str) -> None:
    """One line per leg on stderr (stdout carries only the JSON line)."""
    print(f"[bench {time.strftime('%H:%M:%S')}] {msg}", file=sys.stderr, flush=True)


def _code_text(src: str) -> str:
    """C++ source with its comments removed and whitespace runs collapsed, so that an edit of a comment leaves the
    digest of the code unchanged (the GEMM sources hold no string literal that contains a comment marker)."""
    import re
    src = re.sub(r"/\*.*?\*/", " ", src, flags=re.S)
    src = re.sub(r"//[^\n]*", " ", src)
    return " ".join(src.split())


def _sources_digest():
    """sha256 over the code of the GEMM sources (comments and layout excluded), or None when one of them is absent
    (a tree with the built library only): the stored traffic figure is then not claimed."""
    import hashlib
    h = hashlib.sha256()
    for rel in GEMM_SOURCES:
        try:
            with open(os.path.join(HERE, rel), encoding="utf-8") as f:
                h.update(_code_text(f.read()).encode())
        except FileNotFoundError:
            return None
    return h.hexdigest()


def _dgate_traffic_bytes(launch_mix=None):
    """Calibrated HBM bytes per dgate launch of the roofline batches, while the GEMM sources and the launch mix
    (which linears the batches launch: "separate" or "stacked") are the ones the counters were taken on."""
    t = DGATE_TRAFFIC
    if t["sources_sha256"] is None or t["sources_sha256"] != _sources_digest():
        return None
    if launch_mix is not None and launch_mix != t["launch_mix"]:
        return None
    return (t["fetch_kib"] * t["fetch_scale"] + t["write_kib"] * t["write_scale"]) * 1024.0


def _parse():
    ap = argparse.ArgumentParser(description=__doc__.splitlines()[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20, help="timed headline steps (each about 0.12 s)")
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--reps", type=int, default=10, help="repetitions of each secondary measurement")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-gemv", action="store_true")
    ap.add_argument("--no-square", action="store_true")
    ap.add_argument("--no-distill", action="store_true")
    ap.add_argument("--no-hyper", action="store_true")
    ap.add_argument("--no-model", action="store_true",
                    help="skip the single-linear, attention-projection and MLP-trio steps")
    ap.add_argument("--no-sweep", action="store_true", help="skip the LLaMA-2-13B T=8192 sweep")
    ap.add_argument("--no-prefill", action="store_true", help="skip the LLaMA-2-13B T=512 forward")
    ap.add_argument("--gemv-layers", type=int, default=40)
    ap.add_argument("--profile-copy-mib", type=int, default=0,
                    help="also copy this many MiB device to device once (calibrates the HBM byte counters)")
    ap.add_argument("--summarize-trace", metavar="CSV", help="print the summary of a rocprofv3 kernel trace and exit")
    ap.add_argument("--summarize-counters", metavar="CSV",
                    help="print the per-dispatch summary of a rocprofv3 counter collection and exit")
    return ap.parse_args()


# ------------------------------------------------------------------ the step

class Step:
    """Buffers and the sequence of library calls of one mask-learning step."""

    def __init__(self, d, g, tau, g_out=1):
        import torch
        import paper_2609_33977_amd as gm
        self.gm, self.d, self.g, self.g_out, self.tau = gm, d, g, g_out, tau
        T, d_in = d["X"].shape
        d_out = d["W"].shape[0]
        G_in, G_out = d_in // g, d_out // g_out
        dev = "cuda"
        self.mask = torch.empty(G_out, G_in, dtype=torch.float32, device=dev)
        self.soft = torch.empty(G_out, G_in, dtype=torch.float32, device=dev)
        self.Y = torch.empty(T, d_out, dtype=torch.bfloat16, device=dev)
        self.dX = torch.empty(T, d_in, dtype=torch.bfloat16, device=dev)
        self.dgate = torch.empty(G_out, G_in, dtype=torch.float32, device=dev)
        self.dlogits = torch.empty(G_out, G_in, dtype=torch.float32, device=dev)
        self.ws = torch.empty(max(gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g, g_out), 16),
                              dtype=torch.uint8, device=dev)
        self.fws = torch.empty(max(gm.gm_workspace_size(gm.GM_OP_FWD, T, d_in, d_out, g, g_out), 16),
                               dtype=torch.uint8, device=dev)

    def gate(self):
        self.gm.gm_gate(self.d["logits"], self.d["noise"], self.tau, True, self.mask, self.soft)

    def fwd(self):
        self.gm.gm_masked_linear_fwd(self.d["X"], self.d["W"], self.mask, self.g, self.Y, self.fws, g_out=self.g_out)

    def bwd(self):
        self.gm.gm_masked_linear_bwd(self.d["dY"], self.d["X"], self.d["W"], self.mask, self.g, self.dX, self.dgate,
                                     self.ws, g_out=self.g_out)

    def gate_bwd(self):
        self.gm.gm_gate_bwd(self.dgate, self.soft, self.tau, self.dlogits)

    def dgate_only(self):
        self.gm.gm_masked_linear_bwd(self.d["dY"], self.d["X"], self.d["W"], self.mask, self.g, None, self.dgate,
                                     self.ws, g_out=self.g_out)

    def __call__(self):
        self.gate()
        self.fwd()
        self.bwd()
        self.gate_bwd()


def _events_ms(fn, n):
    """Average duration of fn() on the current stream, from HIP events around each call."""
    import torch
    starts = [torch.cuda.Event(enable_timing=True) for _ in range(n)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(n)]
    for i in range(n):
        starts[i].record()
        fn()
        ends[i].record()
    torch.cuda.synchronize()
    return float(np.mean([s.elapsed_time(e) for s, e in zip(starts, ends)]))


def _events_batch_ms(fn, n):
    """Average duration of n back-to-back fn() calls on the current stream: HIP events around the batch."""
    import torch
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(n):
        fn()
    end.record()
    torch.cuda.synchronize()
    return float(start.elapsed_time(end)) / n


def _graph_pass_ms(fn, outs, reps):
    """fn() captured once in a HIP graph and replayed: the average time of a replay between HIP events, or None
    when a replay's outputs (zeroed before each of two checked replays) differ from the eager call's."""
    import torch
    fn()
    torch.cuda.synchronize()
    want = [o.clone() for o in outs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn()
    for _ in range(2):
        for o in outs:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        if not all(torch.equal(o, w) for o, w in zip(outs, want)):
            return None
    ms = _events_ms(graph.replay, reps)
    del graph
    return ms


def _shift_to_budget(gm, logits, noise, sizes, kept, tau, iters=64):
    """Logits shifted by one offset per selector matrix so that the library's own hard gate keeps
    exactly kept[l] of matrix l's selectors (bisection on the offsets, all matrices at once; nothing
    here evaluates the gate's noise transform).  Returns the shifted logits."""
    import torch
    dev = logits.device
    L = len(sizes)
    seg = torch.repeat_interleave(torch.arange(L, device=dev), torch.tensor(sizes, device=dev))
    ends = torch.tensor(np.cumsum(sizes), dtype=torch.int64, device=dev)
    want = torch.tensor(kept, dtype=torch.float64, device=dev)

    def counts(m):  # kept selectors per matrix: a running sum read at the matrix ends
        cs = torch.cumsum(m.to(torch.int32), 0, dtype=torch.int64)[ends - 1]
        return torch.diff(cs, prepend=torch.zeros(1, dtype=torch.int64, device=dev)).double()

    lo = torch.full((L,), -24.0, dtype=torch.float64, device=dev)
    hi = torch.full((L,), 24.0, dtype=torch.float64, device=dev)
    mask = torch.empty_like(logits)
    for _ in range(iters):
        c = 0.5 * (lo + hi)
        gm.gm_gate(logits + c.float()[seg], noise, tau, True, mask)
        cnt = counts(mask)
        eq = cnt == want
        lo = torch.where(eq | (cnt < want), c, lo)
        hi = torch.where(eq | (cnt > want), c, hi)
        if bool(eq.all()):
            break
    c = 0.5 * (lo + hi)
    out = logits + c.float()[seg]
    del seg, mask
    return out


class ModelStep:
    """One mask-learning step over several masked linears whose selectors share one flat array: one gate
    call over all of them, every linear's forward, every linear's backward (dX and dgate, last linear
    first), one STE call.  The gate inputs are independent draws, logits ~ N(0,1) and u ~ U(0,1), with each
    matrix's logits shifted so that the library's gate keeps exactly that matrix's budget.

    groups (default: every linear alone) lists runs of consecutive linears that read one input, e.g. a
    layer's q, k and v: each run is stored and launched as one stacked linear (weights, selectors, output
    and output gradient of its members one after the other, as the fused layouts of inference and training
    frameworks keep them).  Its forward gives every member's Y, its dgate every member's selector gradient,
    and its dX the sum of the members' input gradients, which is what the shared input receives.  The
    members' selectors are contiguous in the flat array, so the gate and the budgets are those of the
    separate linears.  Each launch has its own X, W and dY (drawn on the device)."""

    def __init__(self, T, shapes, kept, g, tau, key, groups=None):
        import torch
        import paper_2609_33977_amd as gm
        import workloads
        self.gm, self.g, self.tau, self.T = gm, g, tau, T
        self.shapes = list(shapes)
        sizes = [d_out * (d_in // g) for d_out, d_in in self.shapes]
        self.offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        n = int(self.offsets[-1])
        logits, noise = workloads.independent_gate_inputs(workloads.gen.rng_for(*key), n)
        dev = "cuda"
        self.noise = torch.from_numpy(noise).to(dev)
        self.logits = _shift_to_budget(gm, torch.from_numpy(logits).to(dev), self.noise, sizes, kept, tau)
        self.mask, self.soft, self.dgate, self.dlogits = (torch.empty(n, device=dev) for _ in range(4))
        self.gate()
        seg_kept = [int(self.mask[int(a):int(b)].sum().item()) for a, b in zip(self.offsets[:-1], self.offsets[1:])]
        self.kept = seg_kept
        self.kept_total = int(sum(seg_kept))
        self.kept_target = int(sum(kept))
        gen = torch.Generator(device=dev)
        gen.manual_seed(workloads.SEED + 1000 * key[0] + key[1])
        self.groups = [(l,) for l in range(len(self.shapes))] if groups is None else [tuple(gr) for gr in groups]
        if sorted(l for gr in self.groups for l in gr) != list(range(len(self.shapes))) or any(
                list(gr) != list(range(gr[0], gr[0] + len(gr))) or len({self.shapes[l][1] for l in gr}) != 1
                for gr in self.groups):
            raise ValueError("groups must cover every linear once, as runs of consecutive linears of one d_in")
        self.lin = []
        fws = bws = 16
        for gr in self.groups:
            d_out, d_in = sum(self.shapes[l][0] for l in gr), self.shapes[gr[0]][1]
            lo, hi = int(self.offsets[gr[0]]), int(self.offsets[gr[-1] + 1])
            X = torch.randn(T, d_in, device=dev, generator=gen).to(torch.bfloat16)
            W = (torch.randn(d_out, d_in, device=dev, generator=gen) * 0.02).to(torch.bfloat16)
            dY = torch.randn(T, d_out, device=dev, generator=gen).to(torch.bfloat16)
            Y = torch.empty(T, d_out, dtype=torch.bfloat16, device=dev)
            dX = torch.empty(T, d_in, dtype=torch.bfloat16, device=dev)
            view = lambda t, lo=lo, hi=hi, d_out=d_out, d_in=d_in: t[lo:hi].view(d_out, d_in // g)
            self.lin.append((X, W, dY, Y, dX, view(self.mask), view(self.dgate)))
            fws = max(fws, gm.gm_workspace_size(gm.GM_OP_FWD, T, d_in, d_out, g))
            bws = max(bws, gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g))
        self.fws = torch.empty(fws, dtype=torch.uint8, device=dev)
        self.ws = torch.empty(bws, dtype=torch.uint8, device=dev)
        kept_params = [k * g for k in self.kept]
        self.flops = {"fwd": sum(2.0 * T * p for p in kept_params), "dx": sum(2.0 * T * p for p in kept_params),
                      "dgate": sum(2.0 * T * d_out * d_in for d_out, d_in in self.shapes)}

    def gate(self):
        self.gm.gm_gate(self.logits, self.noise, self.tau, True, self.mask, self.soft)

    def fwd(self):
        for X, W, _, Y, _, m, _ in self.lin:
            self.gm.gm_masked_linear_fwd(X, W, m, self.g, Y, self.fws)

    def bwd(self):
        for X, W, dY, _, dX, m, dg in reversed(self.lin):
            self.gm.gm_masked_linear_bwd(dY, X, W, m, self.g, dX, dg, self.ws)

    def dgate_only(self):
        for X, W, dY, _, _, m, dg in reversed(self.lin):
            self.gm.gm_masked_linear_bwd(dY, X, W, m, self.g, None, dg, self.ws)

    def gate_bwd(self):
        self.gm.gm_gate_bwd(self.dgate, self.soft, self.tau, self.dlogits)

    def near_threshold(self, band=1e-6):
        """Gates of the last gate pass whose relaxed value lies within band of 1/2 (the GPU's fp32 value)."""
        return int(((self.soft - 0.5).abs() <= band).sum().item())

    def __call__(self):
        self.gate()
        self.fwd()
        self.bwd()
        self.gate_bwd()


def _model_step(step, reps, workload):
    """Time a ModelStep: whole steps as one batch between HIP events, then each phase the same way."""
    import torch
    for _ in range(2):
        step()
    torch.cuda.synchronize()
    ms = _events_batch_ms(step, reps)
    ph = {name: _events_batch_ms(getattr(step, name), reps) for name in ("gate", "fwd", "bwd", "gate_bwd")}
    fl = step.flops
    total = sum(fl.values())
    return {"workload": workload, "linears": len(step.shapes), "selectors": int(step.offsets[-1]),
            "kept": step.kept_total, "TFLOP_per_step": total / 1e12, "ms_per_step": ms,
            "TFLOP/s": total / (ms / 1e3) / 1e12, "frac_of_bf16_peak": total / (ms / 1e3) / 1e12 / PEAK_BF16_TFLOPS,
            "breakdown_ms": ph, "fwd_kept_TFLOP/s": fl["fwd"] / (ph["fwd"] / 1e3) / 1e12,
            "bwd_TFLOP/s": (fl["dx"] + fl["dgate"]) / (ph["bwd"] / 1e3) / 1e12,
            "near_threshold_gates": step.near_threshold()}


def _dgate_roofline(step, reps):
    """Every linear's dgate-only backward (one dgate_kernel launch each) back to back between two HIP events
    on the launch stream: average launch duration and achieved TFLOP/s on the dense dgate FLOPs."""
    import torch
    step.dgate_only()
    torch.cuda.synchronize()
    batch = _events_batch_ms(step.dgate_only, reps)
    n = len(step.lin)
    return {"launches_per_batch": n, "avg_launch_ms": batch / n, "flops_per_launch": step.flops["dgate"] / n,
            "achieved_TFLOP/s": step.flops["dgate"] / (batch / 1e3) / 1e12}


def _single_linear(reps):
    """Single masked linear (T 128, 1024 x 1024, 1x256 groups, half of 4096 groups kept, tau 0.5): a
    latency figure (the step is far too small to fill the GPU)."""
    import workloads
    cfg = workloads.config("single_1024")
    _, d_out, d_in = cfg["linears"][0]
    g = cfg["g"]
    step = ModelStep(cfg["T"], [(d_out, d_in)], [d_out * (d_in // g) // 2], g, cfg["tau"], (1, 1))
    out = _model_step(step, reps, f"single masked linear: T {cfg['T']}, W {d_out}x{d_in}, 1x{g} groups, "
                                  f"2048 of 4096 kept, tau {cfg['tau']}")
    out["us_per_step"] = out["ms_per_step"] * 1e3
    out["breakdown_us"] = {k: v * 1e3 for k, v in out.pop("breakdown_ms").items()}
    out["graph_us_per_step"] = _graph_us(step, reps)
    return out


def _graph_us(step, reps):
    """The step captured once in a HIP graph and replayed: its time without the host's per-call cost.  Every
    replay's outputs (mask, Y, dX, dgate, logit gradient) are checked against the eager step's; None if they
    differ.  The single linear's path launches kernels only (no memset nodes)."""
    import torch
    step()
    torch.cuda.synchronize()
    X, W, dY, Y, dX, m, dg = step.lin[0]
    outs = lambda: [step.mask, Y, dX, step.dgate, step.dlogits]
    eager = [t.clone() for t in outs()]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(3):
        for t in outs():
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        if not all(torch.equal(a, b) for a, b in zip(outs(), eager)):
            return None
    ms = _events_batch_ms(graph.replay, max(reps, 50))
    del graph
    return ms * 1e3


def _attention_4096(reps):
    """LLaMA-2-7B attention projection (T 4096, W 4096 x 4096, 1x256 groups, half kept): the step, its
    per-phase times, its dgate roofline and the vendor dense GEMMs on the same tensors."""
    import workloads
    cfg = workloads.config("attn_4096")
    _, d_out, d_in = cfg["linears"][0]
    g = cfg["g"]
    step = ModelStep(cfg["T"], [(d_out, d_in)], [d_out * (d_in // g) // 2], g, cfg["tau"], (2, 1))
    out = _model_step(step, reps, f"LLaMA-2-7B attention projection: W {d_out}x{d_in}, X {cfg['T']} tokens "
                                  f"(2 x 2048), 1x{g} groups, 50% of {d_out * (d_in // g)} kept")
    out["dgate_roofline"] = _dgate_roofline(step, reps)
    X, W, dY = step.lin[0][0], step.lin[0][1], step.lin[0][2]
    out["dense_context"] = _dense_context(X, W, dY, out["breakdown_ms"], reps)
    out["_step"] = step
    return out


def _mlp_trio(reps):
    """LLaMA-2-7B MLP trio (gate/up 11008x4096, down 4096x11008), T 4096, per-matrix sparsity ~ U(0.3, 0.7)."""
    import workloads
    cfg = workloads.config("mlp_trio_7b")
    g = cfg["g"]
    shapes = [(d_out, d_in) for _, d_out, d_in in cfg["linears"]]
    kept, s = workloads.kept_counts_uniform_law(workloads.gen.rng_for(3, 0), [o * (i // g) for o, i in shapes],
                                                *cfg["law"][1:])
    step = ModelStep(cfg["T"], shapes, kept, g, cfg["tau"], (3, 1))
    out = _model_step(step, reps, "LLaMA-2-7B MLP trio: gate/up 11008x4096, down 4096x11008, T 4096, "
                                  "1x256 groups, sparsity ~ U(0.3, 0.7) per matrix")
    out["sparsity"] = [round(float(x), 4) for x in s]
    return out


def _llama2_7b_shapes():
    import workloads
    cfg = workloads.config("llama2_7b_step")
    g = cfg["g"]
    shapes = [(d_out, d_in) for _ in range(cfg["layers"]) for _, d_out, d_in in cfg["linears"]]
    sizes = [o * (i // g) for o, i in shapes]
    kept, _ = workloads.kept_counts_beta_law(workloads.gen.rng_for(4, 0), sizes, [o * i for o, i in shapes], 0.5)
    return cfg, shapes, kept


def _llama2_7b_groups(layers):
    """Per layer, q|k|v and gate|up (each run reads one input) as one stacked linear; o and down alone."""
    return [gr for l in range(layers) for gr in ((7 * l, 7 * l + 1, 7 * l + 2), (7 * l + 3,), (7 * l + 4, 7 * l + 5),
                                                 (7 * l + 6,))]


LLAMA2_7B_WORKLOAD = ("LLaMA-2-7B mask-learning step: all 224 masked linears (32 layers x q,k,v,o 4096x4096, "
                      "gate,up 11008x4096, down 4096x11008), T 4096 (2 x 2048), 1x256 groups, Beta(2,2) per-matrix "
                      "budgets at 50% of 25,296,896 groups; one gate and one STE call over all selectors")


def _sweep_13b(reps):
    """LLaMA-2-13B shapes at T 8192: forward and backward per call for g in {64, 128, 256, 512}, half kept."""
    import torch
    import paper_2609_33977_amd as gm
    import workloads
    cfg = workloads.config("llama2_13b_infer")
    T = cfg["T_sweep"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(workloads.SEED + 5)
    out = {"workload": f"LLaMA-2-13B q (5120x5120), gate (13824x5120), down (5120x13824), T {T}, 1xg groups, "
                       "50% kept at random"}
    for name, d_out, d_in in (cfg["linears"][0], cfg["linears"][4], cfg["linears"][6]):
        X = torch.randn(T, d_in, device="cuda", generator=gen).to(torch.bfloat16)
        W = (torch.randn(d_out, d_in, device="cuda", generator=gen) * 0.02).to(torch.bfloat16)
        dY = torch.randn(T, d_out, device="cuda", generator=gen).to(torch.bfloat16)
        Y = torch.empty(T, d_out, dtype=torch.bfloat16, device="cuda")
        dX = torch.empty(T, d_in, dtype=torch.bfloat16, device="cuda")
        for g in cfg["g_sweep"]:
            G = d_out * (d_in // g)
            m = torch.zeros(G, device="cuda")
            m[torch.randperm(G, device="cuda", generator=gen)[: G // 2]] = 1.0
            m = m.view(d_out, d_in // g)
            dg = torch.empty(d_out, d_in // g, device="cuda")
            ws = torch.empty(gm.gm_workspace_size(gm.GM_OP_BWD, T, d_in, d_out, g), dtype=torch.uint8, device="cuda")
            fwd = lambda: gm.gm_masked_linear_fwd(X, W, m, g, Y)
            bwd = lambda: gm.gm_masked_linear_bwd(dY, X, W, m, g, dX, dg, ws)
            for _ in range(3):
                fwd()
                bwd()
            torch.cuda.synchronize()
            tf, tb = _events_ms(fwd, reps), _events_ms(bwd, reps)
            kept_fl, dense_fl = 2.0 * T * (G // 2) * g, 2.0 * T * d_out * d_in
            out[f"{name}_g{g}"] = {"fwd_ms": tf, "bwd_ms": tb, "fwd_kept_TFLOP/s": kept_fl / (tf / 1e3) / 1e12,
                                   "bwd_TFLOP/s": (kept_fl + dense_fl) / (tb / 1e3) / 1e12,
                                   "TFLOP/s": (2 * kept_fl + dense_fl) / ((tf + tb) / 1e3) / 1e12}
        del X, W, dY, Y, dX
    return out


def _prefill_13b(reps):
    """LLaMA-2-13B forward at T 512 over the seven linears of one layer: 40 to 108 output tiles, so the
    forward splits K (its workspace is passed)."""
    import torch
    import paper_2609_33977_amd as gm
    import workloads
    cfg = workloads.config("llama2_13b_infer")
    T, g = 512, cfg["g"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(workloads.SEED + 6)
    mats, fl, by = [], 0.0, 0.0
    ws = torch.empty(max(max(gm.gm_workspace_size(gm.GM_OP_FWD, T, d_in, d_out, g) for _, d_out, d_in in cfg["linears"]),
                         16), dtype=torch.uint8, device="cuda")
    for _, d_out, d_in in cfg["linears"]:
        X = torch.randn(T, d_in, device="cuda", generator=gen).to(torch.bfloat16)
        W = (torch.randn(d_out, d_in, device="cuda", generator=gen) * 0.02).to(torch.bfloat16)
        G = d_out * (d_in // g)
        m = torch.zeros(G, device="cuda")
        m[torch.randperm(G, device="cuda", generator=gen)[: G // 2]] = 1.0
        mats.append((X, W, m.view(d_out, d_in // g), torch.empty(T, d_out, dtype=torch.bfloat16, device="cuda")))
        fl += 2.0 * T * (G // 2) * g
        by += (G // 2) * g * 2 + G * 4 + 2 * T * (d_in + d_out)

    def run():
        for X, W, m, Y in mats:
            gm.gm_masked_linear_fwd(X, W, m, g, Y, ws)
    for _ in range(3):
        run()
    torch.cuda.synchronize()
    ms = _events_ms(run, reps)
    return {"workload": "LLaMA-2-13B q,k,v,o,gate,up,down forward, T 512, 1x256 groups, 50% kept",
            "ms_per_layer": ms, "kept_TFLOP/s": fl / (ms / 1e3) / 1e12, "GB/s": by / (ms / 1e3) / 1e9}


def _dense_context(X, W, dY, breakdown, reps):
    """Context, not a target: the vendor dense GEMM (hipBLASLt through torch.matmul) on the three dense products
    of the same training step on the same tensors, Y = X W^T, dX = dY W and the weight gradient dW = dY^T X,
    every operand contiguous and row-major (the transposed ones copied beforehand).  The masked step computes
    the forward on kept groups, dX over kept groups and the per-group gradient instead of dW; the ratio of the
    dense time to the masked forward + backward time is the figure to set beside a dense layer."""
    import torch
    Wt = W.t().contiguous()
    dYt = dY.t().contiguous()
    T, d_in = X.shape
    d_out = W.shape[0]
    prods = {"fwd": lambda: torch.matmul(X, Wt), "dX": lambda: torch.matmul(dY, W),
             "dW": lambda: torch.matmul(dYt, X)}
    out = {"workload": f"dense bf16 GEMMs of the same step: {T} tokens, W {d_out}x{d_in} (hipBLASLt via torch.matmul)"}
    total = 0.0
    for name, fn in prods.items():
        for _ in range(10):
            fn()
        torch.cuda.synchronize()
        ms = _events_batch_ms(fn, reps)
        total += ms
        out[name + "_ms"] = ms
        out[name + "_TFLOP/s"] = 2.0 * T * d_in * d_out / (ms / 1e3) / 1e12
    masked = breakdown["fwd"] + breakdown["bwd"]
    out.update({"dense_fwd_bwd_ms": total, "masked_fwd_bwd_ms": masked, "speedup": total / masked})
    return out


# ------------------------------------------------------------------ CPU baseline

def _cpu_info():
    """Cores this process may run on, the BLAS thread pools NumPy uses, and the CPU model."""
    cores = len(os.sched_getaffinity(0))
    blas = []
    try:
        from threadpoolctl import threadpool_info
        blas = [{"library": i.get("internal_api"), "threads": int(i.get("num_threads", 1))} for i in threadpool_info()]
    except Exception:
        pass
    model = None
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    threads = max([b["threads"] for b in blas] or [cores])
    return cores, threads, blas, model


def _oracle_step_s(case, min_s):
    """Seconds per whole step of the oracle on one linear (gate, fwd, dX, dgate, STE), fp64 NumPy; repeated
    until min_s have passed (at least once).  The bf16 -> fp64 widening of the inputs is done beforehand."""
    import oracle
    X, W, dY = oracle.from_bf16(case.X), oracle.from_bf16(case.W), oracle.from_bf16(case.dY)
    reps, t0 = 0, time.perf_counter()
    while True:
        m, y = oracle.gate(case.logits, case.noise, case.tau, True)
        oracle.linear_fwd(X, W, m, case.g)
        _, dgate = oracle.linear_bwd(dY, X, W, m, case.g)
        oracle.gate_bwd(dgate, y, case.tau)
        reps += 1
        el = time.perf_counter() - t0
        if el >= min_s:
            return el / reps, reps


def _step_flops(T, d_in, d_out, kept, g):
    return 2.0 * T * kept * g * 2 + 2.0 * T * d_out * d_in


def _cpu_baseline(headline_flops):
    """The fp64 oracle, as it stands, timed on this host for every workload: the single linear, the attention
    projection and the MLP trio in full, the LLaMA-2-7B step as its first layer (7 linears) times 32, and the
    LLaMA-2-13B decode / T = 512 forward over one layer per token count."""
    import oracle
    import workloads
    cores, threads, blas, model = _cpu_info()
    per = {}
    c1 = workloads.config("single_1024")
    _, d_out, d_in = c1["linears"][0]
    case = workloads.make_linear_case((1, 0, 0), c1["T"], d_in, d_out, c1["g"], None, tau=c1["tau"])
    sec, reps = _oracle_step_s(case, 1.0)
    per["single_1024"] = {"s_per_step": sec, "reps": reps,
                          "TFLOP/s": _step_flops(c1["T"], d_in, d_out, case.kept, c1["g"]) / sec / 1e12}
    c2 = workloads.config("attn_4096")
    _, d_out, d_in = c2["linears"][0]
    case = workloads.make_linear_case((2, 0, 0), c2["T"], d_in, d_out, c2["g"], None, tau=c2["tau"])
    sec, reps = _oracle_step_s(case, 1.0)
    per["attn_4096"] = {"s_per_step": sec, "reps": reps,
                        "TFLOP/s": _step_flops(c2["T"], d_in, d_out, case.kept, c2["g"]) / sec / 1e12}
    c3 = workloads.config("mlp_trio_7b")
    g = c3["g"]
    kept3, _ = workloads.kept_counts_uniform_law(workloads.gen.rng_for(3, 0),
                                                 [o * (i // g) for _, o, i in c3["linears"]], *c3["law"][1:])
    sec3, fl3 = 0.0, 0.0
    for j, (_, d_out, d_in) in enumerate(c3["linears"]):
        case = workloads.make_linear_case((3, 0, j), c3["T"], d_in, d_out, g, kept3[j], tau=c3["tau"])
        sec3 += _oracle_step_s(case, 0.0)[0]
        fl3 += _step_flops(c3["T"], d_in, d_out, kept3[j], g)
        del case
    per["mlp_trio_7b"] = {"s_per_step": sec3, "TFLOP/s": fl3 / sec3 / 1e12}
    c4, shapes, kept4 = _llama2_7b_shapes()
    g = c4["g"]
    sec4 = 0.0
    for j, (d_out, d_in) in enumerate(shapes[:7]):
        case = workloads.make_linear_case((4, 0, j), c4["T"], d_in, d_out, g, kept4[j], tau=c4["tau"])
        sec4 += _oracle_step_s(case, 0.0)[0]
        del case
    per["llama2_7b_step"] = {"s_per_layer": sec4, "s_per_step": 32 * sec4,
                             "TFLOP/s": headline_flops / (32 * sec4) / 1e12,
                             "sample": "layer 0's seven linears, one whole step each; the step time is 32 x that"}
    c5 = workloads.config("llama2_13b_infer")
    g = c5["g"]
    r = workloads.gen.rng_for(5, 7)
    mats = []
    for _, d_out, d_in in c5["linears"]:
        W = oracle.from_bf16(workloads.bf16_bits_from_f32(r.standard_normal((d_out, d_in), dtype=np.float32)
                                                          * np.float32(0.02)))
        G = d_out * (d_in // g)
        m = workloads.random_kept_mask(r, G, G // 2).reshape(d_out, d_in // g).astype(np.float64)
        mats.append((W, m))
    kept_bytes = sum(int(m.sum()) * g * 2 for _, m in mats)
    for T in c5["T_decode"]:
        xs = {}
        t0 = time.perf_counter()
        for (W, m), src in zip(mats, ("a", "a", "a", "o", "m", "m", "d")):
            if (src, W.shape[1]) not in xs:
                xs[(src, W.shape[1])] = oracle.from_bf16(workloads.bf16_bits_from_f32(
                    r.standard_normal((T, W.shape[1]), dtype=np.float32)))
            oracle.linear_fwd(xs[(src, W.shape[1])], W, m, g)
        sec = time.perf_counter() - t0
        per[f"llama2_13b_T{T}"] = {"s_per_layer": sec, "kept_GB/s": kept_bytes / sec / 1e9,
                                   "kept_TFLOP/s": 2.0 * T * kept_bytes / 2 / sec / 1e12}
    del mats
    return {"value": per["llama2_7b_step"]["TFLOP/s"], "unit": "TFLOP/s", "cores": threads, "kind": "oracle",
            "sample": "LLaMA-2-7B step: layer 0's seven masked linears (q,k,v,o,gate,up,down at T 4096), one whole "
                      "step each (gate, fwd, dX, dgate, STE) in fp64 NumPy, times 32 layers; value counted like "
                      "the GPU figure (kept FLOPs for fwd and dX, dense for dgate)",
            "affinity_cores": cores, "blas": blas, "cpu_model": model, "per_config": per}


# ------------------------------------------------------------------ square groups

def _square_groups(X, W, dY, tau, reps):
    """The same step on the attention-projection tensors with g x g groups (g = 16 .. 128), half of the
    groups kept at random (gate inputs encode the kept set: the subject here is the GEMMs)."""
    import torch
    import workloads
    T, d_in = X.shape
    d_out = W.shape[0]
    d = dict(X=X, W=W, dY=dY)
    out = {"workload": f"attention-projection tensors (T {T}, W {d_out}x{d_in}) with square g x g groups, "
                       "50% kept at random"}
    for g in (16, 32, 64, 128):
        G = (d_out // g) * (d_in // g)
        r = workloads.gen.rng_for(2, 1, g)
        keep = workloads.random_kept_mask(r, G, G // 2)
        logits, noise = workloads.budgeted_gate_inputs(r, keep)
        shape = (d_out // g, d_in // g)
        dd = dict(d, logits=torch.from_numpy(np.ascontiguousarray(logits.reshape(shape), dtype=np.float32)).cuda(),
                  noise=torch.from_numpy(np.ascontiguousarray(noise.reshape(shape), dtype=np.float32)).cuda())
        step = Step(dd, g, tau, g_out=g)
        for _ in range(3):
            step()
        torch.cuda.synchronize()
        if int(step.mask.sum().item()) != G // 2:
            raise RuntimeError(f"gate kept count differs from the budget ({g}x{g})")
        nnz = (G // 2) * g * g
        fl = {"fwd": 2.0 * T * nnz, "dx": 2.0 * T * nnz, "dgate": 2.0 * T * d_out * d_in}
        ms = _events_ms(step, reps)
        br = {name: _events_ms(getattr(step, name), reps) for name in ("fwd", "bwd")}
        dg = _events_ms(step.dgate_only, reps)
        out[f"{g}x{g}"] = {"ms_per_step": ms, "TFLOP/s": sum(fl.values()) / (ms / 1e3) / 1e12,
                           "fwd_ms": br["fwd"], "fwd_kept_TFLOP/s": fl["fwd"] / (br["fwd"] / 1e3) / 1e12,
                           "bwd_ms": br["bwd"], "dgate_ms": dg,
                           "dgate_TFLOP/s": fl["dgate"] / (dg / 1e3) / 1e12}
        del step, dd
    return out


# ------------------------------------------------------------------ distillation loss

def _distill(reps):
    """Distillation loss (Eq. 4) through the LLaMA-2-7B LM head over one batch: forward and backward."""
    import torch
    import paper_2609_33977_amd as gm
    import workloads
    N, d, V = workloads.config("llama2_7b_step")["T"], 4096, 32000
    gen = torch.Generator(device="cuda")
    gen.manual_seed(workloads.SEED)
    Ht = torch.randn(N, d, device="cuda", generator=gen)
    Hs = (Ht + 0.3 * torch.randn(N, d, device="cuda", generator=gen)).to(torch.bfloat16)
    Ht = Ht.to(torch.bfloat16)
    W = (torch.randn(V, d, device="cuda", generator=gen) * (3.0 / d ** 0.5)).to(torch.bfloat16)
    ws = torch.empty(gm.gm_distill_workspace_size(N, d, V), dtype=torch.uint8, device="cuda")
    loss = torch.empty(1, device="cuda")
    dH = torch.empty(N, d, dtype=torch.bfloat16, device="cuda")

    def fwd():
        gm.gm_distill_fwd(Ht, Hs, W, None, loss, None, ws)

    def bwd():
        gm.gm_distill_bwd(W, dH, ws)

    fwd(); bwd()
    torch.cuda.synchronize()
    t_f = _events_ms(fwd, reps)
    t_b = _events_ms(bwd, reps)
    fl_f, fl_b = 4.0 * N * V * d, 2.0 * N * V * d
    return {"workload": f"LLaMA-2-7B LM head, V {V}, d {d}, {N} tokens of each pass (teacher, student)",
            "fwd_ms": t_f, "fwd_TFLOP/s": fl_f / (t_f / 1e3) / 1e12,
            "bwd_ms": t_b, "bwd_TFLOP/s": fl_b / (t_b / 1e3) / 1e12,
            "TFLOP/s": (fl_f + fl_b) / ((t_f + t_b) / 1e3) / 1e12,
            "logit_bytes_written": 8.0 * N * V, "loss": float(loss.item())}


# ------------------------------------------------------------------ hypernetwork

def _hyper(reps):
    """Hypernetwork over the 224 LLaMA-2-7B selector matrices (1x256 groups), D = H = 64: forward and backward."""
    import torch
    import paper_2609_33977_amd as gm
    import workloads
    cfg = workloads.config("llama2_7b_step")
    sizes = [do * di // cfg["g"] for _ in range(cfg["layers"]) for _, do, di in cfg["linears"]]
    L, D, H = len(sizes), 64, 64
    G = sum(sizes)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), dtype=torch.int64, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(workloads.SEED)
    P = 2 * 3 * H * (D + H + 2)
    z = torch.randn(L, D, device="cuda", generator=gen)
    gru = (torch.rand(P, device="cuda", generator=gen) * 2 - 1) / H ** 0.5
    A = (torch.rand(G, 2 * H, device="cuda", generator=gen) * 2 - 1) / (2 * H) ** 0.5
    c = (torch.rand(G, device="cuda", generator=gen) * 2 - 1) / (2 * H) ** 0.5
    dl = torch.randn(G, device="cuda", generator=gen) * 0.01
    mA, vA, mc, vc = torch.zeros_like(A), torch.zeros_like(A), torch.zeros_like(c), torch.zeros_like(c)
    logits = torch.empty(G, device="cuda")
    dgru = torch.empty(P, device="cuda")
    ws = torch.empty(gm.gm_hyper_workspace_size(L, D, H, G), dtype=torch.uint8, device="cuda")
    step = [0]

    def fwd():
        gm.gm_hyper_fwd(z, gru, A, c, offsets, H, logits, ws)

    def bwd():
        step[0] += 1
        gm.gm_hyper_bwd(dl, z, gru, A, c, mA, vA, mc, vc, H, 1e-3, 0.9, 0.999, 1e-8, 0.05, step[0], dgru, ws)

    fwd(); bwd()
    torch.cuda.synchronize()
    t_f = _events_ms(fwd, reps)
    t_b = _events_ms(bwd, reps)
    b_f = G * (2 * H * 4 + 4 + 4)                          # A, c read; logits written
    b_b = G * (2 * H * 4 * 6 + 4 + 3 * 4 * 2)              # A, mA, vA read and written; dlogits; c, mc, vc
    return {"workload": f"LLaMA-2-7B: {L} layers, {G} selectors, D {D}, H {H} (heads {G * 2 * H} fp32 weights)",
            "fwd_ms": t_f, "fwd_GB/s": b_f / (t_f / 1e3) / 1e9, "bwd_adamw_ms": t_b,
            "bwd_GB/s": b_b / (t_b / 1e3) / 1e9, "fwd_bytes": b_f, "bwd_bytes": b_b}


# ------------------------------------------------------------------ decode GEMV

def _gemv_bandwidth(n_layers, reps):
    """Decode forward (T=1) over the seven LLaMA-2-13B linears of n_layers distinct layers at 50 % sparsity.

    q, k and v read one input, gate and up another (as in the model).  Four
    schedules of the same work: eager launches in series; the same series
    captured in a HIP graph (no host gaps); a graph in which the projections
    that share their input run concurrently on side streams; and the fused
    layout that inference engines use, q|k|v and gate|up stacked into one
    weight (and mask) each, so a layer takes four launches instead of seven.
    Every graph replay and the fused outputs are checked bit for bit against
    the eager outputs before they are timed."""
    import torch
    import paper_2609_33977_amd as gm
    import workloads
    cfg = workloads.config("llama2_13b_infer")
    g = cfg["g"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(workloads.SEED)
    layers, fused, kept_bytes, other_bytes = [], [], 0, 0
    for _ in range(n_layers):
        mats, xs = [], {}
        for (name, d_out, d_in), src in zip(cfg["linears"], ("a", "a", "a", "o", "m", "m", "d")):
            if src not in xs:
                xs[src] = torch.randn(1, d_in, device="cuda", generator=gen).to(torch.bfloat16)
            W = (torch.randn(d_out, d_in, device="cuda", generator=gen) * 0.02).to(torch.bfloat16)
            G = d_out * (d_in // g)
            m = torch.zeros(G, device="cuda")
            m[torch.randperm(G, device="cuda", generator=gen)[: G // 2]] = 1.0
            Y = torch.empty(1, d_out, dtype=torch.bfloat16, device="cuda")
            mats.append((xs[src], W, m.view(d_out, d_in // g), Y))
            kept_bytes += (G // 2) * g * 2
            other_bytes += G * 4 + 2 * d_in + 2 * d_out
        layers.append(mats)

        def stack(part):
            W = torch.cat([mat[1] for mat in part])
            return (part[0][0], W, torch.cat([mat[2] for mat in part]),
                    torch.empty(1, W.shape[0], dtype=torch.bfloat16, device="cuda"))
        fused.append([stack(mats[0:3]), mats[3], stack(mats[4:6]), mats[6]])
    torch.cuda.synchronize()
    total = kept_bytes + other_bytes

    def run(mat, stream=None):
        X, W, m, Y = mat
        gm.gm_masked_linear_fwd(X, W, m, g, Y, stream=stream)

    def serial():
        for mats in layers:
            for mat in mats:
                run(mat)

    def serial_fused():
        for mats in fused:
            for mat in mats:
                run(mat)

    side = [torch.cuda.Stream() for _ in range(3)]  # default priority

    def concurrent():
        main = torch.cuda.current_stream()
        for mats in layers:
            for group, tail in ((mats[0:3], mats[3]), (mats[4:6], mats[6])):
                for s in side[:len(group)]:
                    s.wait_stream(main)
                for s, mat in zip(side, group):
                    run(mat, stream=s)
                for s in side[:len(group)]:
                    main.wait_stream(s)
                run(tail)

    serial()
    torch.cuda.synchronize()
    eager = [mat[3].clone() for mats in layers for mat in mats]
    out = {"workload": f"LLaMA-2-13B decode T=1, 7 linears x {n_layers} distinct layers, 1x{g} groups, 50% kept",
           "bytes_per_pass": total, "launches_per_pass": 7 * n_layers}
    ms = _events_ms(serial, reps)
    out["eager_GB/s"] = total / (ms / 1e3) / 1e9
    best, best_name = ms, "eager"
    serial_fused()
    torch.cuda.synchronize()
    same = all(torch.equal(f[0][3], torch.cat([m[0][3], m[1][3], m[2][3]], dim=1)) and torch.equal(f[2][3], torch.cat(
        [m[4][3], m[5][3]], dim=1)) for f, m in zip(fused, layers))
    if same:
        t = _events_ms(serial_fused, reps)
        out["fused_qkv_gateup_GB/s"] = total / (t / 1e3) / 1e9
        if t < best:
            best, best_name = t, "fused_qkv_gateup"
    else:
        out["fused_qkv_gateup_GB/s"] = None
    for name, body in (("graph", serial), ("graph_concurrent", concurrent)):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            body()
        ok = True
        for _ in range(2):
            for mats in layers:
                for mat in mats:
                    mat[3].zero_()
            graph.replay()
            torch.cuda.synchronize()
            got = [mat[3] for mats in layers for mat in mats]
            ok = ok and all(torch.equal(a, b) for a, b in zip(got, eager))
        if not ok:
            out[name + "_GB/s"] = None
            continue
        t = _events_ms(graph.replay, reps)
        out[name + "_GB/s"] = total / (t / 1e3) / 1e9
        if t < best:
            best, best_name = t, name
        del graph
    out.update({"GB/s": total / (best / 1e3) / 1e9, "frac_of_peak": total / (best / 1e3) / 1e9 / PEAK_HBM_GBS,
                "ms_per_pass": best, "schedule": best_name})
    # The group-compacted export (App. F) of the stacked layout: each row's kept
    # pieces contiguous, with their column and selector (8 bytes per piece) and
    # a row pointer instead of the dense selector array.  Same kept weights;
    # outputs checked bit for bit against the in-place stacked launches.
    packed, packed_bytes = [], 0
    for mats in fused:
        for X1, W, m, Y in mats:
            d_o, d_i = W.shape
            cap = int((m != 0).sum().item())
            Wp = torch.empty(cap, g, dtype=torch.bfloat16, device="cuda")
            chunk = torch.empty(cap, dtype=torch.int32, device="cuda")
            scale = torch.empty(cap, dtype=torch.float32, device="cuda")
            rowptr = torch.empty(d_o + 1, dtype=torch.int32, device="cuda")
            gm.gm_pack_rows(W, m, g, cap, Wp, chunk, scale, rowptr)
            packed.append((X1, Wp, chunk, scale, rowptr, d_o, torch.empty_like(Y), Y))
            packed_bytes += cap * (2 * g + 8) + 4 * (d_o + 1) + 2 * (d_i + d_o)

    def serial_packed():
        for X1, Wp, chunk, scale, rowptr, d_o, Yp, _ in packed:
            gm.gm_packed_linear_fwd(X1, Wp, chunk, scale, rowptr, d_o, g, Yp)

    serial_fused()
    serial_packed()
    torch.cuda.synchronize()
    t = _graph_pass_ms(serial_packed, [p[6] for p in packed], reps) \
        if all(torch.equal(Yp, Y) for *_, Yp, Y in packed) else None
    out["packed_stacked"] = None if t is None else {
        "bytes_per_pass": packed_bytes, "GB/s": packed_bytes / (t / 1e3) / 1e9,
        "frac_of_peak": packed_bytes / (t / 1e3) / 1e9 / PEAK_HBM_GBS, "ms_per_pass": t}
    # Each launch shape on its own: the same projection of all layers back to back (serialised on the stream,
    # as in the pass, captured in a HIP graph so that small launches are not timed against the host's per-call
    # cost; every replay's outputs checked against the eager launches); the rate of one kernel at one shape,
    # free of the pass's mix of small and large launches.
    per_shape = {}
    for j, name in enumerate(("qkv_stacked", "o", "gateup_stacked", "down")):
        mats = [f[j] for f in fused]
        nbytes = sum(2 * int((m != 0).sum().item()) * g + 4 * m.numel() + 2 * (W.shape[1] + W.shape[0])
                     for _, W, m, _ in mats)

        def one(mats=mats):
            for mat in mats:
                run(mat)
        t = _graph_pass_ms(one, [mat[3] for mat in mats], reps)
        per_shape[name] = None if t is None else {
            "rows_x_d_in": list(mats[0][1].shape), "us_per_launch": 1e3 * t / len(mats),
            "GB/s": nbytes / (t / 1e3) / 1e9}
    out["per_shape"] = per_shape
    # 8 and 16 tokens over the same weights and masks: seven launches per layer,
    # the stacked layout's four (q|k|v and gate|up read one input each, so the
    # stacked launches read it once), and the packed export of the stacked
    # layout (outputs checked bit for bit against the stacked in-place ones:
    # both layouts run the same MFMA kernel); each pass captured in a HIP graph,
    # since a 5120 x 5120 launch takes about as long on the GPU as the host
    # needs to issue it
    for T in (8, 16):
        xs = {}

        def x_for(X1):
            if id(X1) not in xs:
                xs[id(X1)] = torch.randn(T, X1.shape[1], device="cuda", generator=gen).to(torch.bfloat16)
            return xs[id(X1)]

        def y_for(d_o):
            return torch.empty(T, d_o, dtype=torch.bfloat16, device="cuda")

        sched = {}
        for name, mats_of in (("", lambda i: layers[i]), ("stacked_", lambda i: fused[i])):
            ys, nbytes = [], kept_bytes
            for i in range(n_layers):
                for X1, W, m, _ in mats_of(i):
                    ys.append((x_for(X1), W, m, y_for(W.shape[0])))
                    nbytes += 4 * m.numel() + 2 * T * (W.shape[0] + W.shape[1])
            sched[name] = (ys, nbytes, lambda ys=ys: [run(mat) for mat in ys], [mat[3] for mat in ys])
        pys, pbytes = [], 0
        for X1, Wp, chunk, scale, rowptr, d_o, _, _ in packed:
            pys.append((x_for(X1), Wp, chunk, scale, rowptr, d_o, y_for(d_o)))
            pbytes += Wp.numel() * 2 + chunk.numel() * 8 + 4 * (d_o + 1) + 2 * T * (X1.shape[1] + d_o)
        sched["packed_stacked_"] = (pys, pbytes, lambda: [gm.gm_packed_linear_fwd(x, Wp, c, sc, rp, d_o, g, y)
                                                          for x, Wp, c, sc, rp, d_o, y in pys], [p[6] for p in pys])
        for name, (ys, nbytes, fn, outs) in sched.items():
            t = _graph_pass_ms(fn, outs, reps)
            out[f"T{T}_{name}GB/s"] = None if t is None else nbytes / (t / 1e3) / 1e9
            out[f"T{T}_{name}ms_per_pass"] = t
        same = all(torch.equal(a, b) for a, b in zip(sched["packed_stacked_"][3], sched["stacked_"][3]))
        out[f"T{T}_packed_equals_in_place"] = bool(same)
        if not same:
            out[f"T{T}_packed_stacked_GB/s"] = None
        del sched, pys, xs
    del packed
    return out


# ------------------------------------------------------------------ budget regulariser

def _budget_bandwidth(reps):
    """Sparsity-budget regulariser over the 224 selector matrices of LLaMA-2-7B (one flat array)."""
    import torch
    import paper_2609_33977_amd as gm
    import workloads
    cfg = workloads.config("llama2_7b_step")
    g = cfg["g"]
    shapes = [(do, di) for _ in range(cfg["layers"]) for _, do, di in cfg["linears"]]
    sizes = [do * di // g for do, di in shapes]
    n = sum(sizes)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), dtype=torch.int64, device="cuda")
    params = torch.tensor([do * di for do, di in shapes], dtype=torch.int64, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(workloads.SEED)
    mask = (torch.rand(n, device="cuda", generator=gen) < 0.5).float()
    y = torch.rand(n, device="cuda", generator=gen) * 0.98 + 0.01
    dgate = torch.randn(n, device="cuda", generator=gen)
    dlog = torch.empty_like(dgate)
    L = len(sizes)
    kept = torch.empty(L, dtype=torch.int64, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    coeff = torch.empty(L, dtype=torch.float32, device="cuda")

    def reg():
        gm.gm_budget_loss(mask, offsets, params, 0.5, 16.0, False, kept, loss, coeff)

    def bwd():
        gm.gm_gate_bwd_budget(dgate, y, cfg["tau"], offsets, coeff, dlog)

    reg(); bwd()
    torch.cuda.synchronize()
    t_reg = _events_ms(reg, reps)
    t_bwd = _events_ms(bwd, reps)
    return {"workload": f"LLaMA-2-7B: {L} selector matrices, {n} selectors in one flat array, lambda 16, s_t 0.5",
            "loss_ms": t_reg, "loss_GB/s": 4.0 * n / (t_reg / 1e3) / 1e9,
            "gate_bwd_budget_ms": t_bwd, "gate_bwd_budget_GB/s": 12.0 * n / (t_bwd / 1e3) / 1e9}


# ------------------------------------------------------------------ main

# ------------------------------------------------------------------ rocprofv3 summaries

def _short_kernel(name: str) -> str:
    """`void gm::dgate_kernel<256, 1>(...)` -> `gm::dgate_kernel<256, 1>`; other names cut at 60 characters."""
    n = name[5:] if name.startswith("void ") else name
    depth, out = 0, []
    for ch in n:
        if ch == "(" and depth == 0:
            break
        depth += ch == "<"
        depth -= ch == ">"
        out.append(ch)
    n = "".join(out)
    return n if n.startswith("gm::") else n[:60]


def _runs(items, key):
    """Maximal runs of consecutive items (in start order) for which key(item) is true: list of (first, last)."""
    runs, start = [], None
    for k, it in enumerate(items):
        if key(it):
            start = k if start is None else start
        elif start is not None:
            runs.append((start, k - 1))
            start = None
    if start is not None:
        runs.append((start, len(items) - 1))
    return runs


def _trace_summary(path: str) -> str:
    """Markdown summary of a rocprofv3 kernel_trace.csv: per kernel and workgroup count, dispatches and
    duration statistics; then the longest back-to-back run of dgate_kernel<256, 1> dispatches (the
    bench's roofline batches: every linear's dgate-only backward) with its mean launch duration."""
    import csv
    rows = []
    with open(path, newline="") as f:
        for r in csv.DictReader(f):
            if r.get("Kind", "KERNEL_DISPATCH") != "KERNEL_DISPATCH":
                continue
            wg = int(r["Grid_Size_X"]) // max(int(r["Workgroup_Size_X"]), 1)
            rows.append((int(r["Start_Timestamp"]), int(r["End_Timestamp"]), _short_kernel(r["Kernel_Name"]), wg))
    rows.sort()
    total = sum(e - b for b, e, _, _ in rows) or 1
    agg = {}
    for b, e, k, wg in rows:
        agg.setdefault((k, wg), []).append((e - b) / 1e3)
    lines = [f"{len(rows)} dispatches, {total / 1e6:.2f} ms of kernel time", "",
             "| kernel | workgroups | calls | mean µs | median µs | min µs | max µs | % of kernel time |",
             "|---|---:|---:|---:|---:|---:|---:|---:|"]
    for (k, wg), d in sorted(agg.items(), key=lambda kv: -sum(kv[1]))[:40]:
        d = np.array(d)
        lines.append(f"| `{k}` | {wg} | {d.size} | {d.mean():.1f} | {np.median(d):.1f} | {d.min():.1f} | "
                     f"{d.max():.1f} | {100 * d.sum() * 1e3 / total:.2f} |")
    dg = "gm::dgate_kernel<256, 1>"
    runs = _runs(rows, lambda r: r[2] == dg)
    if runs:
        a, b = max(runs, key=lambda ab: ab[1] - ab[0])
        d = np.array([(rows[k][1] - rows[k][0]) / 1e3 for k in range(a, b + 1)])
        span = (rows[b][1] - rows[a][0]) / 1e3 / d.size
        mix = {}
        for k in range(a, b + 1):
            mix[rows[k][3]] = mix.get(rows[k][3], 0) + 1
        lines += ["", f"Longest back-to-back run of `{dg}`: {d.size} dispatches (workgroups: "
                      + ", ".join(f"{w} x {c}" for w, c in sorted(mix.items())) + f"), mean {d.mean():.2f} µs, "
                      f"median {np.median(d):.2f}, min {d.min():.2f}, max {d.max():.2f}; "
                      f"first start to last end / dispatches = {span:.2f} µs"]
    return "\n".join(lines)


def _counter_summary(path: str) -> str:
    """Markdown summary of a rocprofv3 counter_collection.csv: per kernel and workgroup count, the mean of
    each counter per dispatch (summed over the counter's instances within a dispatch)."""
    import csv
    per = {}
    with open(path, newline="") as f:
        for r in csv.DictReader(f):
            wg = int(r["Grid_Size"]) // max(int(r["Workgroup_Size"]), 1)
            key = (_short_kernel(r["Kernel_Name"]), wg)
            disp = per.setdefault(key, {}).setdefault(r["Dispatch_Id"], {})
            disp[r["Counter_Name"]] = disp.get(r["Counter_Name"], 0.0) + float(r["Counter_Value"])
    names = sorted({c for d in per.values() for v in d.values() for c in v})
    lines = ["| kernel | workgroups | dispatches | " + " | ".join(f"mean {n}" for n in names) + " |",
             "|---|---:|---:|" + "---:|" * len(names)]
    for (k, wg), d in sorted(per.items()):
        vals = [np.mean([v.get(n, 0.0) for v in d.values()]) for n in names]
        lines.append(f"| `{k}` | {wg} | {len(d)} | " + " | ".join(f"{x:.1f}" for x in vals) + " |")
    # the roofline batches: the longest run of consecutive dispatches that are all dgate_kernel<256, 1>
    dg = "gm::dgate_kernel<256, 1>"
    order = sorted(((int(i), k, wg) for (k, wg), d in per.items() for i in d), key=lambda x: x[0])
    runs = _runs(order, lambda x: x[1] == dg)
    if runs:
        a, b = max(runs, key=lambda ab: ab[1] - ab[0])
        sel = order[a:b + 1]
        lines += ["", f"Longest back-to-back run of `{dg}` (dispatches {sel[0][0]}-{sel[-1][0]}): {len(sel)} dispatches"]
        for wg in sorted({x[2] for x in sel}) + [None]:
            part = [per[(dg, x[2])][str(x[0])] for x in sel if wg is None or x[2] == wg]
            what = f"workgroups {wg}" if wg is not None else "all of the run"
            lines.append(f"- {what}: {len(part)} dispatches, mean " + ", ".join(
                f"{n} {np.mean([v.get(n, 0.0) for v in part]):.1f}" for n in names))
    return "\n".join(lines)


def main():
    args = _parse()
    if args.summarize_trace:
        print(_trace_summary(args.summarize_trace))
        return
    if args.summarize_counters:
        print(_counter_summary(args.summarize_counters))
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU; --gpus {args.gpus} is not supported (this build has no multi-GPU path).",
              file=sys.stderr)
        sys.exit(2)
    import torch
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(2)
    import paper_2609_33977_amd  # noqa: F401  (fails loudly when the HIP library is missing)

    # ---- headline: the whole LLaMA-2-7B mask-learning step (224 masked linears)
    _progress("headline: building the LLaMA-2-7B step (224 linears)")
    cfg, shapes, kept = _llama2_7b_shapes()
    step = ModelStep(cfg["T"], shapes, kept, cfg["g"], cfg["tau"], (4, 1))
    if step.kept_total != step.kept_target:
        raise RuntimeError(f"gate kept {step.kept_total} groups, budget {step.kept_target}")
    flops = step.flops
    flops_step = sum(flops.values())
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    _progress(f"headline: {args.steps} timed steps")
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    ms_per_step = (time.perf_counter() - t0) * 1e3 / args.steps
    tflops = flops_step / (ms_per_step / 1e3) / 1e12
    near = step.near_threshold()

    reps = max(3, args.reps)
    breakdown = {name: _events_batch_ms(getattr(step, name), reps) for name in ("gate", "fwd", "bwd", "gate_bwd")}
    roof = _dgate_roofline(step, reps)
    n_sel = int(step.offsets[-1])
    gate_leg = {"workload": f"the step's gate over all {n_sel} selectors (one call) and its STE backward",
                "selectors": n_sel, "gate_ms": breakdown["gate"],
                "gate_GB/s": 16.0 * n_sel / (breakdown["gate"] / 1e3) / 1e9,
                "gate_bwd_ms": breakdown["gate_bwd"],
                "gate_bwd_GB/s": 12.0 * n_sel / (breakdown["gate_bwd"] / 1e3) / 1e9,
                "bytes": {"gate": 16 * n_sel, "gate_bwd": 12 * n_sel},
                "near_threshold_gates": near,
                "near_threshold_rule": "GPU relaxed value within 1e-6 of 1/2 in the last timed step"}
    gate_leg["gate_frac_of_hbm_peak"] = gate_leg["gate_GB/s"] / PEAK_HBM_GBS
    del step
    torch.cuda.empty_cache()

    # The same step with the linears that read one input (q|k|v, gate|up) launched as one stacked linear each
    # (four launches per layer and phase, as fused layouts keep them): the same counted work, another schedule.
    _progress("headline step with q|k|v and gate|up stacked")
    stk = ModelStep(cfg["T"], shapes, kept, cfg["g"], cfg["tau"], (4, 1), groups=_llama2_7b_groups(cfg["layers"]))
    for _ in range(2):
        stk()
    torch.cuda.synchronize()
    stk_ms = _events_batch_ms(stk, max(3, args.steps // 2))
    stacked = {"launches_per_phase": len(stk.lin), "ms_per_step": stk_ms,
               "TFLOP/s": flops_step / (stk_ms / 1e3) / 1e12,
               "breakdown_ms": {name: _events_batch_ms(getattr(stk, name), reps) for name in ("fwd", "bwd")}}
    del stk
    torch.cuda.empty_cache()

    if args.profile_copy_mib:
        src = torch.empty(args.profile_copy_mib << 20, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    single = attn = mlp = None
    square = None
    if not args.no_model:
        _progress("single linear, attention projection, square groups, MLP trio")
        single = _single_linear(max(reps, 50))
        attn = _attention_4096(reps)
        a_step = attn.pop("_step")
        if not args.no_square:
            square = _square_groups(a_step.lin[0][0], a_step.lin[0][1], a_step.lin[0][2], a_step.tau, reps)
        del a_step
        torch.cuda.empty_cache()
        mlp = _mlp_trio(reps)
        torch.cuda.empty_cache()

    _progress("decode GEMV, budget, distillation, hypernetwork, sweep, T=512 forward")
    gemv = None if args.no_gemv else _gemv_bandwidth(args.gemv_layers, reps)
    torch.cuda.empty_cache()
    budget = _budget_bandwidth(reps)
    distill = None if args.no_distill else _distill(reps)
    torch.cuda.empty_cache()
    hyper = None if args.no_hyper else _hyper(reps)
    torch.cuda.empty_cache()
    sweep = None if args.no_sweep else _sweep_13b(reps)
    prefill = None if args.no_prefill else _prefill_13b(reps)
    torch.cuda.empty_cache()

    _progress("oracle on the host")
    cpu = None if args.no_cpu_baseline else _cpu_baseline(flops_step)
    _progress("done")

    out = {
        "metric": "masked-linear fwd+bwd TFLOP/s & % bf16 MFMA peak; sparse GEMV GB/s",
        "value": tflops,
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic",
        "config": {"workload": LLAMA2_7B_WORKLOAD, "T": cfg["T"], "linears": len(shapes), "g": cfg["g"],
                   "selectors": n_sel, "kept_groups": sum(kept), "tau": cfg["tau"],
                   "TFLOP_per_step": flops_step / 1e12,
                   "counting": "kept FLOPs 2*T*nnz for fwd and dX, dense 2*T*d_out*d_in for dgate"},
        "frac_of_bf16_peak": tflops / PEAK_BF16_TFLOPS,
        "roofline": {"bound": "mfma", "achieved": roof["achieved_TFLOP/s"], "peak": PEAK_BF16_TFLOPS,
                     "unit": "TFLOP/s", "frac": roof["achieved_TFLOP/s"] / PEAK_BF16_TFLOPS,
                     "traffic": _dgate_traffic_bytes("separate")},
        "kernels": {"dominant": "dgate_kernel<256, 1> (X^T dY tile + fused W-weighted group reduction), one launch "
                                "per linear: 128 of 4096x4096, 64 of 11008x4096, 32 of 4096x11008 per step",
                    "dgate_flops_per_launch": roof["flops_per_launch"], "dgate_avg_launch_ms": roof["avg_launch_ms"],
                    "dgate_launches_per_batch": roof["launches_per_batch"],
                    "dgate_algorithmic_bytes_per_launch": sum(2.0 * cfg["T"] * (di + do) + 2.0 * do * di
                                                              + 4.0 * do * (di // cfg["g"]) for do, di in shapes)
                                                          / len(shapes),
                    "sources_sha256": _sources_digest(), "breakdown_ms": breakdown,
                    "fwd_kept_TFLOP/s": flops["fwd"] / (breakdown["fwd"] / 1e3) / 1e12,
                    "bwd_TFLOP/s": (flops["dx"] + flops["dgate"]) / (breakdown["bwd"] / 1e3) / 1e12,
                    "stacked_launches": stacked},
        "gate": gate_leg,
        "cpu_baseline": cpu,
        "single_linear": single,
        "attn_4096": attn,
        "mlp_trio": mlp,
        "gemv": gemv,
        "budget": budget,
        "square_groups": square,
        "distill": distill,
        "hypernetwork": hyper,
        "sweep_13b": sweep,
        "prefill_13b": prefill,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
