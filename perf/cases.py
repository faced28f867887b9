"""Workloads whose time matters to a user of this library, in a form that can be timed and checked.

A case is a dict of plain values.  `listed()` are the fixed ones, `draw(rng)` gives more of the same ranges,
`prepare(case, seed)` makes what a training program holds before the call (an optimizer state as it is in the middle of
a run, two gradient buffers, the hyper-parameters), `run(state)` is one pass through the public entry points, and
`exact(case, seed)` is what the floating-point outputs of that pass are in 64 bits.

Successive passes take the two gradient buffers in turn, as a training loop sees another gradient in every step: the
amax of a tensor moves between them by its sampling noise, so the scales of some tensors change and those of most stay.

Layouts are those of the paper's model table (Tab. 1: hidden 768 / 4096 / 5120 / 12288) with a Megatron-style tensor list,
whole or one layer of them, the one flat tensor of configuration 1, and ragged lists of many small tensors.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2310_18313_amd import binding as B
from paper_2310_18313_amd import synth
from paper_2310_18313_amd.allreduce_study import Fp8AllReduce
from paper_2310_18313_amd.state import OptimizerState

DEVICE = "cuda:0"
SRC = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}
FMT = {"e5m2": B.E5M2, "e4m3": B.E4M3}
WCOPY = {"e4m3": B.WCOPY_E4M3, "bf16": B.WCOPY_BF16}
STATE = {"f16": B.STATE_F16, "bf16": B.STATE_BF16, "e4m3": B.STATE_E4M3, "f32": B.STATE_F32}
MODE = {"exact": B.MSCALE_EXACT_PASS, "predicted": B.MSCALE_PREDICTED, "cast": B.MSCALE_FROM_CAST}
FMAX = {B.E5M2: 57344.0, B.E4M3: 448.0}


def listed():
    return [
        # one flat tensor of 2^20 parameters, the smallest configuration: a step is a dozen launches and their latency
        {"name": "step flat 1M", "kind": "step", "layout": "flat", "n": 1 << 20, "sigma": 1e-3, "path": "spec"},
        # many small tensors of odd sizes (adapters, norms, biases), some empty: per-tensor work and remainders; half
        # precision gradients, E4M3, a bf16 weight copy, the three entry points one after the other
        {"name": "step 600 ragged tensors", "kind": "step", "layout": "ragged", "tensors": 600, "largest": 70001, "sizes": 3,
         "sigma": 0.0, "path": "jit", "src": "fp16", "fmt": "e4m3", "wcopy": "bf16"},
        # a whole small model: the default path of a single-GPU step (just-in-time scales, speculative quantisation)
        {"name": "step GPT-125M", "kind": "step", "layout": "gpt", "hidden": 768, "layers": 12, "ffn": 3072, "vocab": 50304,
         "pos": 2048, "sigma": 0.0, "path": "spec"},
        # the same model with delayed scaling and a predicted first-moment scale: one pass over the gradient, one over the state
        {"name": "step GPT-125M single pass", "kind": "step", "layout": "gpt", "hidden": 768, "layers": 12, "ffn": 3072,
         "vocab": 50304, "pos": 2048, "sigma": 0.0, "path": "single", "fmt": "e4m3", "hist": 16},
        # one layer of the 7B model (a pipeline stage, or the unit of a layer-wise optimizer), the cast measuring for the step
        {"name": "step GPT-7B layer fused", "kind": "step", "layout": "gpt", "hidden": 4096, "layers": 1, "ffn": 16384, "vocab": 0,
         "pos": 0, "sigma": 1e-4, "path": "spec-fused", "hist": 4},
        # two layers of the 13B model, the step with a pair of first-moment buffers
        {"name": "step GPT-13B 2 layers, m pair", "kind": "step", "layout": "gpt", "hidden": 5120, "layers": 2, "ffn": 20480,
         "vocab": 0, "pos": 0, "sigma": 1e-4, "path": "spec-m2"},
        # one layer of the 175B model, heavy-tailed gradients: the largest, bound by memory
        {"name": "step GPT-175B layer", "kind": "step", "layout": "gpt", "hidden": 12288, "layers": 1, "ffn": 49152, "vocab": 0,
         "pos": 0, "sigma": 1e-4, "path": "spec", "tails": True},
        # gradients accumulated in fp32 (micro-batches), quantised before they are communicated
        {"name": "quantize GPT-7B layer fp32", "kind": "quantize", "layout": "gpt", "hidden": 4096, "layers": 1, "ffn": 16384,
         "vocab": 0, "pos": 0, "sigma": 1e-4, "src": "fp32", "fmt": "e4m3"},
        # the optimizer of a data-parallel rank (the FP8 gradient arrives from the all-reduce), with fp32 master weights
        {"name": "adam GPT-125M fp32 master", "kind": "adam", "layout": "gpt", "hidden": 768, "layers": 12, "ffn": 3072,
         "vocab": 50304, "pos": 2048, "sigma": 0.0, "master": "f32"},
        # the same with a bf16 weight copy and the counters of every output, for a caller that cannot allocate
        {"name": "adam GPT-125M static, counters", "kind": "adam", "layout": "gpt", "hidden": 768, "layers": 12, "ffn": 3072,
         "vocab": 50304, "pos": 2048, "sigma": 0.0, "wcopy": "bf16", "stats": True, "static": True, "fmt": "e4m3"},
        # the arithmetic of the FP8 gradient all-reduce, eight ranks: quantise, shared scale, re-quantise, sum
        {"name": "all-reduce GPT-125M 8 ranks", "kind": "allreduce", "layout": "gpt", "hidden": 768, "layers": 12, "ffn": 3072,
         "vocab": 50304, "pos": 2048, "sigma": 0.0, "ranks": 8, "fmt": "e4m3"},
        # monitoring: signal, noise, underflow and overflow of an FP8 gradient against its fp32 source
        {"name": "error stats GPT-125M fp32", "kind": "stats", "layout": "gpt", "hidden": 768, "layers": 12, "ffn": 3072,
         "vocab": 50304, "pos": 2048, "sigma": 0.0, "src": "fp32", "fmt": "e5m2"},
    ]


def _log_int(rng: random.Random, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["step"] * 6 + ["quantize", "adam", "adam", "allreduce", "stats"])
    case = {"kind": kind}
    shape = rng.choice(["flat", "ragged", "gpt", "gpt"])
    ranks = rng.choice([2, 3, 4, 8, 8, 12]) if kind == "allreduce" else 1
    if shape == "flat":
        case.update(layout="flat", n=_log_int(rng, 1 << 17, (1 << 29) // ranks))
    elif shape == "ragged":
        case.update(layout="ragged", tensors=_log_int(rng, 50, 2000), largest=_log_int(rng, 5000, 200000), sizes=rng.randrange(1000))
    else:
        layers, hidden = _log_int(rng, 1, 12), _log_int(rng, 200, 4096 / math.sqrt(ranks))
        while 12 * hidden * hidden * layers > 6e8:
            layers -= 1
        case.update(layout="gpt", hidden=hidden, layers=max(1, layers), ffn=4 * hidden, vocab=rng.choice([0, 0, 1000, 32003]),
                    pos=rng.choice([0, 2048]))
    case["sigma"] = rng.choice([0.0, 1e-4, 1e-3])
    case["src"] = rng.choice(["bf16", "bf16", "fp16", "fp32"])
    case["fmt"] = rng.choice(["e5m2", "e4m3"])
    if kind == "step":
        case["path"] = rng.choice(["spec", "spec", "jit", "single", "spec-fused", "spec-m2"])
        case["hist"] = rng.choice([1, 1, 4, 16])
        case["wcopy"] = rng.choice(["e4m3", "bf16"])
        case["tails"] = rng.random() < 0.25
    elif kind == "adam":
        if rng.random() < 0.5:
            case["master"] = rng.choice(["f16", "bf16", "e4m3", "f32"])
            case["v"] = rng.choice(["f16", "e4m3"])
        else:
            case["wcopy"] = rng.choice(["e4m3", "bf16"])
            case["stats"] = rng.random() < 0.5
        case["mode"] = rng.choice(["exact", "exact", "predicted"])
        case["static"] = rng.random() < 0.3
    elif kind == "allreduce":
        case["ranks"] = ranks
        case["src"] = "bf16"
    return case


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _layout(case) -> synth.Layout:
    if case["layout"] == "flat":
        return synth.flat_layout(case["n"])
    if case["layout"] == "gpt":
        return synth.gpt_layout(case["hidden"], case["layers"], case["ffn"], case["vocab"], pos=case["pos"])
    sizes = random.Random(case["sizes"])
    numels = [0 if sizes.random() < 0.02 else _log_int(sizes, 1, case["largest"]) for _ in range(case["tensors"])]
    return synth.Layout([f"t{i}" for i in range(len(numels))], numels)


def _workload(case) -> synth.Workload:
    return synth.Workload(case["kind"], _layout(case), lr=3e-4, grad_kind="student_t" if case.get("tails") else "normal",
                          sigma=case["sigma"] or None, hist_window=case.get("hist", 1))


def _gradients(case, wl, seed, count=2):
    dtype = SRC[case.get("src", "bf16")]
    out = []
    for k in range(count):
        g = torch.zeros(wl.layout.total, dtype=dtype, device=DEVICE)
        synth.fill_gradients(g, wl, seed, k)
        out.append(g)
    return out


def _tensors(wl):
    return [(t, off, n) for t, (off, n) in enumerate(wl.layout.tensors()) if n]


def _amaxes(buf, wl) -> np.ndarray:
    """max |x| per tensor, on the host."""
    out = np.zeros(wl.layout.n_tensors)
    which = _tensors(wl)
    if which:
        got = torch.stack([buf[o:o + n].abs().amax().float() for _, o, n in which]).cpu().numpy()
        out[[t for t, _, _ in which]] = got
    return out


def _pow2(fmax: float, amax: float) -> float:
    """The largest power of two s with s * amax <= fmax."""
    e = math.floor(math.log2(fmax / amax))
    while math.ldexp(amax, e) > fmax:
        e -= 1
    while math.ldexp(amax, e + 1) <= fmax:
        e += 1
    return math.ldexp(1.0, e)


def _encode(x: torch.Tensor, kind: str) -> torch.Tensor:
    """fp32 payloads as they are stored."""
    if kind == "e4m3":
        return x.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    if kind == "e5m2":
        return x.clamp(-57344.0, 57344.0).to(torch.float8_e5m2).view(torch.uint8)
    return x.clamp(-65504.0, 65504.0).to(torch.float16)


def _fill_moment(dst, meta, wl, sigmas, seed, kind, second):
    """A first or second moment as a run of some hundred steps leaves it, with its metadata (as on resuming a run)."""
    fmax = 65504.0 if kind == "f16" else 448.0
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed * 2 + (1 if second else 0) + 12345)
    rows, which = [], _tensors(wl)
    for t, off, n in which:
        s = float(sigmas[t])
        x = torch.randn(n, generator=gen, device=DEVICE, dtype=torch.float32)
        x = x.mul_(0.16 * s * s).add_(s * s).abs_() if second else x.mul_(0.23 * s)
        amax = x.abs().amax()
        scale = torch.exp2(torch.floor(torch.log2(fmax / amax.double()))).float()
        code = _encode(x.mul_(scale), kind)
        dst[off:off + n] = code
        rows.append(torch.stack([scale, 1.0 / scale, amax, _decode_max(code, kind) / scale]))
    arr = B.meta_to_numpy(meta, wl.layout.n_tensors)
    if rows:
        got = torch.stack(rows).cpu().numpy()
        for j, field in enumerate(("scale", "inv_scale", "amax", "amax_deq")):
            arr[field][[t for t, _, _ in which]] = got[:, j]
    meta.copy_(B.meta_from_numpy(arr, DEVICE))


def _decode_max(code, kind):
    if kind == "f16":
        return code.abs().amax().float()
    top = (code & 0x7F).amax()
    return top.view(1).view(torch.float8_e4m3fn if kind == "e4m3" else torch.float8_e5m2).float()[0]


def _optimizer(case, wl, seed, **kw) -> OptimizerState:
    """The optimizer state of a run under way: weights, moments and the metadata that goes with them."""
    cfg = B.autoscale_cfg(ramp_steps=wl.ramp_steps, hist_window=wl.hist_window)
    st = OptimizerState(wl.layout.tensors(), wl.layout.total, cfg, grad_fmt=FMT[case.get("fmt", "e5m2")],
                        wcopy=WCOPY[case.get("wcopy", "e4m3")], master_fmt=STATE[case.get("master", "f16")],
                        v_fmt=STATE[case.get("v", "f16")], **kw)
    w0 = torch.zeros(wl.layout.total, dtype=torch.bfloat16, device=DEVICE)
    synth.fill_weights(w0, wl.layout, seed)
    st.init_master(w0)
    sig = synth.per_tensor_sigma(wl, seed)
    _fill_moment(st.m, st.m_meta, wl, sig, seed, "e4m3", False)
    _fill_moment(st.v, st.v_meta, wl, sig, seed, case.get("v", "f16"), True)
    return st


def _seed_history(meta, wl, grad):
    """The amax history as it is when the steps before saw gradients like `grad`."""
    amax = _amaxes(grad, wl)
    arr = B.meta_to_numpy(meta, wl.layout.n_tensors)
    arr["amax_hist"][:, :wl.hist_window] = amax[:, None]
    meta.copy_(B.meta_from_numpy(arr, DEVICE))


def prepare(case, seed):
    wl = _workload(case)
    kind = case["kind"]
    S = {"case": case, "wl": wl, "k": 100}
    if kind == "step":
        S["grads"] = _gradients(case, wl, seed)
        S["st"] = st = _optimizer(case, wl, seed, second_m=case["path"] == "spec-m2")
        _seed_history(st.g_meta, wl, S["grads"][1])
    elif kind == "quantize":
        S["grads"] = _gradients(case, wl, seed)
        S["cfg"] = cfg = B.autoscale_cfg(hist_window=wl.hist_window)
        S["ctx"] = ctx = B.Context(wl.layout.tensors())
        S["meta"] = ctx.new_meta(cfg)
        S["g8"] = torch.zeros(wl.layout.total, dtype=torch.uint8, device=DEVICE)
    elif kind == "adam":
        S["st"] = st = _optimizer(case, wl, seed)
        grad = _gradients(case, wl, seed, 1)[0]
        st.quantize_grad(grad)
    elif kind == "allreduce":
        n = case["ranks"]
        common = torch.zeros(wl.layout.total, dtype=torch.bfloat16, device=DEVICE)
        S["grads"] = []
        for k in range(2):
            synth.fill_gradients(common, wl, seed, k)
            ranks = []
            for r in range(n):
                g = torch.zeros(wl.layout.total, dtype=torch.bfloat16, device=DEVICE)
                synth.fill_gradients(g, wl, seed, 2 + 2 * r + k)
                ranks.append(g.add_(common, alpha=0.25))
            S["grads"].append(ranks)
        ctx = B.Context(wl.layout.tensors())
        S["group"] = Fp8AllReduce(ctx, n, wl.layout.total, FMT[case["fmt"]], B.autoscale_cfg(), "auto")
    else:
        S["grad"] = grad = _gradients(case, wl, seed, 1)[0]
        cfg = B.autoscale_cfg()
        S["ctx"] = ctx = B.Context(wl.layout.tensors())
        S["meta"] = ctx.new_meta(cfg)
        S["g8"] = torch.zeros(wl.layout.total, dtype=torch.uint8, device=DEVICE)
        ctx.amax_scale(grad, FMT[case["fmt"]], S["meta"], cfg)
        ctx.cast_fp8(grad, S["g8"], FMT[case["fmt"]], S["meta"], cfg)
    return S


# ---- one pass -------------------------------------------------------------------------------------------------------
def run(S):
    case = S["case"]
    kind = case["kind"]
    if kind == "step":
        st, path = S["st"], case["path"]
        grad = S["grads"][S["k"] & 1]
        S["k"] += 1
        mode = {"spec-fused": B.MSCALE_FROM_CAST, "single": B.MSCALE_PREDICTED}.get(path, B.MSCALE_EXACT_PASS)
        hp = B.adam_hparams(S["wl"].lr, S["k"], wcopy=st.wcopy_kind, m_scale_mode=mode)
        st.step(grad, hp, delayed=path == "single", speculative=path.startswith("spec"), pair_m=path == "spec-m2")
        return {"g8": st.g8, "m": st.m, "v": st.v, "w": st.w, "wq": st.wq, "g_meta": st.g_meta, "m_meta": st.m_meta,
                "v_meta": st.v_meta, "w_meta": st.w_meta, "q_meta": st.q_meta}
    if kind == "quantize":
        grad = S["grads"][S["k"] & 1]
        S["k"] += 1
        fmt = FMT[case["fmt"]]
        S["ctx"].amax_scale(grad, fmt, S["meta"], S["cfg"])
        S["ctx"].cast_fp8(grad, S["g8"], fmt, S["meta"], S["cfg"])
        return {"g8": S["g8"], "meta": S["meta"]}
    if kind == "adam":
        st = S["st"]
        S["k"] += 1
        hp = B.adam_hparams(S["wl"].lr, S["k"], wcopy=st.wcopy_kind, stats=int(case.get("stats", False)),
                            m_scale_mode=MODE[case.get("mode", "exact")], master_fmt=st.master_fmt, v_fmt=st.v_fmt)
        if case.get("static"):
            B.adam_step_fp8_static(st.tensors, st.g8, st.grad_fmt, st.g_meta, st.m, st.m_meta, st.v, st.v_meta, st.w, st.w_meta,
                                   st.wq, st.q_meta, hp)
        else:
            st.adam(hp)
        return {"m": st.m, "v": st.v, "w": st.w, "wq": st.wq, "m_meta": st.m_meta, "v_meta": st.v_meta, "w_meta": st.w_meta,
                "q_meta": st.q_meta}
    if kind == "allreduce":
        grp = S["group"]
        grads = S["grads"][S["k"] & 1]
        S["k"] += 1
        grp.step(grads)
        return {"summed": grp.summed, "summed_meta": grp.summed_meta, "payloads": grp.shared_payload, "metas": grp.shared_meta}
    got = S["ctx"].quant_error_stats(S["grad"], S["g8"], FMT[case["fmt"]], S["meta"])
    return {f: got[f].astype(np.int64) if got[f].dtype.kind == "u" else got[f] for f in got.dtype.names}


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def work(case):
    n = _layout(case).n_params
    src = 4 if case.get("src") == "fp32" else 2
    kind = case["kind"]
    if kind == "quantize":
        return {"bytes": n * (src + 1), "flops": n * 3}
    if kind == "stats":
        return {"bytes": n * (src + 1), "flops": n * 6}
    if kind == "allreduce":
        # every rank: its gradient in, its payload and its re-quantised payload out; and the sum
        return {"bytes": n * (case["ranks"] * 4 + 1), "flops": n * case["ranks"] * 6}
    v = B.STATE_BYTES[STATE[case.get("v", "f16")]]
    w = B.STATE_BYTES[STATE[case.get("master", "f16")]]
    state = 2 * (1 + v + w) + (2 if case.get("wcopy") == "bf16" else 1)       # moments and weights in and out, the copy out
    return {"bytes": n * (state + 1 + (src if kind == "step" else 0)), "flops": n * 20}


def tolerance(case):
    # Codes, scales and counters follow from one rounding per written operation and are the same whatever the order of the
    # work.  The error statistics are sums in float64 whose order is free: 4e-16 against torch's order over 1.3e8 elements.
    if case["kind"] == "stats":
        return {"rel": 4e-15, "max": 1e-13}
    return "exact"


# ---- the floating-point outputs in 64 bits --------------------------------------------------------------------------
def _value(code, kind):
    if kind in ("e4m3", "e5m2"):
        return code.view(torch.float8_e4m3fn if kind == "e4m3" else torch.float8_e5m2).double()
    return code.double()


def exact(case, seed):
    if case["kind"] not in ("step", "adam", "stats"):
        return None                                            # codes and metadata only
    wl = _workload(case)
    fmt = case.get("fmt", "e5m2")
    S = prepare(case, seed)
    if case["kind"] == "stats":
        meta = B.meta_to_numpy(S["meta"], wl.layout.n_tensors)
        signal, noise = np.zeros(wl.layout.n_tensors), np.zeros(wl.layout.n_tensors)
        for t, off, n in _tensors(wl):
            r = S["grad"][off:off + n].double()
            signal[t] = float((r * r).sum())
            noise[t] = float((r - _value(S["g8"][off:off + n], fmt) / float(meta["scale"][t])).square().sum())
        return {"signal": signal, "noise": noise, "n_nonzero": None, "n_underflow": None, "n_overflow": None, "n_nonfinite": None}
    st = S["st"]
    nt = wl.layout.n_tensors
    metas = {k: B.meta_to_numpy(getattr(st, k + "_meta"), nt) for k in "gmvw"}
    vk, wk = case.get("v", "f16"), case.get("master", "f16")
    v_out = torch.zeros(st.v.numel(), dtype=torch.float64, device=DEVICE) if vk == "f16" else None
    w_out = torch.zeros(st.w.numel(), dtype=torch.float64, device=DEVICE) if wk != "e4m3" else None
    q_out = torch.zeros(st.wq.numel(), dtype=torch.float64, device=DEVICE) if case.get("wcopy") == "bf16" else None
    step, lr, b1, b2, eps, wd = S["k"] + 1, wl.lr, 0.9, 0.95, 1e-8, 0.1
    grad = S["grads"][S["k"] & 1] if case["kind"] == "step" else None
    amax = _amaxes(grad, wl) if grad is not None else None
    for t, off, n in _tensors(wl):
        sl = slice(off, off + n)
        if grad is not None:
            # the gradient's scale and its FP8 code, then the value that the code stands for
            hist = metas["g"]["amax_hist"][t].astype(np.float64)
            if case["path"] == "single":
                bound = float(hist[:wl.hist_window].max())
            else:
                bound = max(float(amax[t]), float(hist[1:wl.hist_window].max()) if wl.hist_window > 1 else 0.0)
            s = _pow2(FMAX[FMT[fmt]], bound) if bound > 0 else float(metas["g"]["scale"][t])
            g = _value(_encode(grad[sl].float() * s, fmt), fmt) / s
            g_deq = float(g.abs().amax())
        else:
            g = _value(st.g8[sl], fmt) / float(metas["g"]["scale"][t])
            g_deq = float(metas["g"]["amax_deq"][t])
        M, V, W = metas["m"][t], metas["v"][t], metas["w"][t]
        m = b1 * (_value(st.m[sl], "e4m3") / float(M["scale"])) + (1 - b1) * g
        v = b2 * (_value(st.v[sl], vk) / float(V["scale"])) + (1 - b2) * g * g
        del g
        w = _value(st.w[sl], wk) / float(W["scale"])
        w = w * (1 - lr * wd) - lr * (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + eps)
        if v_out is not None:
            bound = b2 * float(V["amax_deq"]) + (1 - b2) * g_deq ** 2
            v_out[sl] = v * (_pow2(65504.0, bound) if bound > 0 else float(V["scale"]))
        if w_out is not None:
            bound = float(W["amax_deq"])
            w_out[sl] = w * ((_pow2(65504.0, bound) / 2 if bound > 0 else float(W["scale"])) if wk == "f16" else 1.0)
        if q_out is not None:
            q_out[sl] = w
    out = dict.fromkeys(("m", "m_meta", "v_meta", "w_meta", "q_meta"))
    if case["kind"] == "step":
        out.update(g8=None, g_meta=None)
    out.update(v=v_out, w=w_out, wq=q_out)
    return out
