"""The measured cases: what a user of this package has it do, from one small linear to a ViT-Large layer.

Every case goes through the public entry points of `paper_2607_12505_amd.nmspmm` on device tensors.  Three forms:

* `linear`: one GEMM, sparse (any N:M) or the dense one (`entry` "dense"), with int32, fp16 and/or int8 outputs.
* `layer`:  the four linears of a transformer block (qkv, proj, fc1, fc2), each with its own activations, as a
            network's sequence of layers runs them.  `mode` says how a program issues them: "eager" (four calls),
            "graph" (captured once, one replay per pass) or "carried" (plans made once with the carried-expansion
            hint, every launch expanding the next linear's weight).
* `mlp`:    the INT8 chain fp16 -> nm_quantize_f16 -> fc1 with the int8 epilogue -> fc2 with fp16 output.

Weights are pruned by magnitude to N:M, quantised per row and packed with `nmspmm.compress` in `prepare`: that is
done once, before deployment.  Activations are int8 uniform on [-127, 127], or fp16 N(0, 1) where they are quantised.
"""
import math

import torch

from paper_2607_12505_amd import nmspmm

# The patterns of the library: 1:4 and 2:4, 1:8 ... 5:8; 8:8 is a layer that stays dense.
PATTERNS = ("1:4", "2:4", "1:8", "2:8", "3:8", "4:8", "5:8", "8:8")
OUTS = ("i32", "f16", "i32+f16", "i8")
# No case costs more multiply-adds than the ViT-Large layer, nor writes more outputs than the Swin-B one.
MOST_MACS = 18464 * 12 * 1024 * 1024
MOST_OUTPUTS = 100352 * 9 * 128


def listed():
    return [
        # DeiT-Tiny, one image, fc1: the smallest call, one eager launch.
        {"name": "deit_tiny_fc1_b1", "form": "linear", "m": 197, "k": 192, "n": 768, "pattern": "2:4", "out": "i32"},
        # A ragged call: tokens, channels and reduction that no tile divides, the fp16 and int32 results at once.
        {"name": "ragged_3of8", "form": "linear", "m": 333, "k": 1168, "n": 1004, "pattern": "3:8", "out": "i32+f16"},
        # A serving loop at one image per request: a DeiT-Base layer captured in a graph, a pattern per linear.
        {"name": "deit_base_layer_b1_graph", "form": "layer", "m": 197, "c": 768, "hidden": 3072,
         "patterns": "2:4,1:4,2:8,1:8", "out": "i32", "mode": "graph"},
        # A small batch: a DeiT-Base layer of eight images, 1:4 throughout, four eager calls.
        {"name": "deit_base_layer_b8", "form": "layer", "m": 1576, "c": 768, "hidden": 3072,
         "patterns": "1:4,1:4,1:4,1:4", "out": "f16", "mode": "eager"},
        # DeiT-Small, batch 64, int32 and fp16 results: short reductions, bound by the output stream.
        {"name": "deit_small_layer_b64", "form": "layer", "m": 12608, "c": 384, "hidden": 1536,
         "patterns": "2:4,2:4,2:4,2:4", "out": "i32+f16", "mode": "eager"},
        # Swin-B stage 1, batch 32: the most tokens and the shortest reduction.
        {"name": "swin_b_stage1_layer_b32", "form": "layer", "m": 100352, "c": 128, "hidden": 512,
         "patterns": "2:4,2:8,2:4,2:8", "out": "i32", "mode": "eager"},
        # Swin-B stage 4, batch 32: the int8 MLP with few tokens and wide layers.
        {"name": "swin_b_stage4_mlp_b32", "form": "mlp", "m": 1568, "c": 1024, "hidden": 4096, "patterns": "2:8,2:8"},
        # DeiT-Base, batch 128: the int8 MLP of a throughput run.
        {"name": "deit_base_mlp_b128", "form": "mlp", "m": 25216, "c": 768, "hidden": 3072, "patterns": "2:4,2:4"},
        # ViT-Large at 384 px, batch 32, a searched layer-wise assignment, expansions carried: the flagship workload.
        {"name": "vit_large_layer_b32_carried", "form": "layer", "m": 18464, "c": 1024, "hidden": 4096,
         "patterns": "2:4,2:8,4:8,1:4", "out": "i32", "mode": "carried"},
        # The same network's fc2 left dense: the GEMM that every speedup is quoted over.
        {"name": "vit_large_fc2_b32_dense", "form": "linear", "m": 18464, "k": 4096, "n": 1024, "pattern": "8:8",
         "out": "i32", "entry": "dense"},
        # The same network's qkv, 1:8, fp16 results, one eager call that expands its own weight.
        {"name": "vit_large_qkv_b32_1of8", "form": "linear", "m": 18464, "k": 1024, "n": 3072, "pattern": "1:8",
         "out": "f16"},
    ]


def _log(rng, lo, hi, step):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def draw(rng):
    """One more case: a form, then sizes over the ranges above, most of them multiples of no tile."""
    while True:
        form = rng.choice(("linear", "linear", "linear", "layer", "layer", "mlp"))
        if form == "linear":
            c = {"form": form, "m": _log(rng, 16, 50000, 1), "k": _log(rng, 128, 4096, 16),
                 "n": _log(rng, 128, 4096, 4), "pattern": rng.choice(PATTERNS), "out": rng.choice(OUTS)}
            if c["pattern"] == "8:8":
                c["entry"] = rng.choice(("dense", "sparse"))
        elif form == "layer":
            width = _log(rng, 128, 1024, 32)
            c = {"form": form, "m": _log(rng, 49, 100352, 1), "c": width, "hidden": 4 * width,
                 "patterns": ",".join(rng.choice(PATTERNS) for _ in range(4)), "out": rng.choice(OUTS[:3]),
                 "mode": rng.choice(("eager", "carried"))}
            if c["m"] <= 512:
                c["mode"] = "graph"
        else:
            width = _log(rng, 128, 1024, 32)
            c = {"form": form, "m": _log(rng, 49, 100352, 1), "c": width, "hidden": 4 * width,
                 "patterns": ",".join(rng.choice(PATTERNS[:7]) for _ in range(2))}
        gemms = _gemms(c)
        if sum(m * k * n for m, k, n, _ in gemms) <= MOST_MACS and sum(m * n for m, _, n, _ in gemms) <= MOST_OUTPUTS:
            return c


def _pattern(text):
    return tuple(int(v) for v in text.split(":"))


def _gemms(case):
    """The case's GEMMs as (m, k, n, pattern)."""
    if case["form"] == "linear":
        return [(case["m"], case["k"], case["n"], case["pattern"])]
    m, c, h, p = case["m"], case["c"], case["hidden"], case["patterns"].split(",")
    if case["form"] == "mlp":
        return [(m, c, h, p[0]), (m, h, c, p[1])]
    return [(m, c, 3 * c, p[0]), (m, c, c, p[1]), (m, c, h, p[2]), (m, h, c, p[3])]


def _weight(n, k, pattern, gen):
    """int8 weight [n, k] with at most N nonzeros per window of M, and its per-row scale, on the GPU."""
    N, M = _pattern(pattern)
    w = torch.randn((n, k // M, M), generator=gen, device="cuda") * 0.02
    if N < M:
        kept = w.abs().topk(N, dim=2).indices
        w = w * torch.zeros_like(w).scatter_(2, kept, 1.0)
    w = w.reshape(n, k)
    top = w.abs().amax(dim=1)
    s_w = torch.where(top > 0, top / 127, torch.ones_like(top))
    return (w / s_w[:, None]).round().clamp(-127, 127).to(torch.int8), s_w


def _inputs(case, seed):
    """The inputs in plain tensors: a list of (X, W, s_w) and, for the MLP (whose X are made on the way), the fp16
    activations."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    gemms, x16 = [], None
    if case["form"] == "mlp":
        x16 = torch.randn((case["m"], case["c"]), generator=gen, device="cuda").half()
    for m, k, n, pattern in _gemms(case):
        x = None
        if x16 is None:
            x = torch.randint(-127, 128, (m, k), generator=gen, device="cuda", dtype=torch.int32).to(torch.int8)
        gemms.append((x, *_weight(n, k, pattern, gen)))
    return gemms, x16


S_X = 4.0 / 127  # scale of quantised N(0, 1) activations


def _mlp_scales(case, gemms):
    """qscale of fc1 (to int8 codes with a per-tensor scale s_y) and scale of fc2 (to fp16)."""
    N, M = _pattern(case["patterns"].split(",")[0])
    s_y = 4 * 0.02 * math.sqrt(case["c"] * min(1.0, 2.5 * N / M)) / 127
    return gemms[0][2] * (S_X / s_y), gemms[1][2] * s_y


def _packed(w, pattern):
    return nmspmm.DeviceWeight.from_packed(nmspmm.compress(w.cpu().numpy(), *_pattern(pattern)))


def _outputs(m, n, out):
    o = {}
    if "i32" in out:
        o["Y"] = torch.empty((m, n), dtype=torch.int32, device="cuda")
    if "f16" in out:
        o["Yh"] = torch.empty((m, n), dtype=torch.float16, device="cuda")
    if "i8" in out:
        o["Yq"] = torch.empty((m, n), dtype=torch.int8, device="cuda")
    return o


def _multipliers(out, k, s_w):
    """fp16: activations of scale 1/127.  int8: codes that use the range, whatever the reduction's length."""
    a = {}
    if "f16" in out:
        a["scale"] = s_w / 127
    if "i8" in out:
        a["qscale"] = s_w / (0.05 * math.sqrt(k))
    return a


def _carried(state):
    """Plans of a layer whose launches carry the next linear's expansion, and its buffers: made once."""
    calls, mode = state["calls"], (nmspmm.NM_OUT_I32 if "Y" in state["outs"][0] else 0) | (
        nmspmm.NM_OUT_F16 if "Yh" in state["outs"][0] else 0)
    plans = [nmspmm.spmm_plan(w.desc, x.shape[0], mode | nmspmm.NM_PLAN_EXPAND_CARRIED) for x, w, _ in calls]
    state["jobs"], state["weights"] = [None] * 4, [w for _, w, _ in calls]
    for i in range(1, 4):
        w = calls[i][1]
        if plans[i].expand:
            buf = torch.empty(nmspmm.expand_size(w.desc)[1], dtype=torch.uint8, device="cuda")
            state["jobs"][i - 1], state["weights"][i] = nmspmm.expand_job(w, buf)
            # the plan of the expanded weight: the compact plan's tile and split
            plans[i] = nmspmm.make_plan(state["weights"][i].desc.kind, plans[i].tile, plans[i].split_k)
    state["plans"] = plans


def prepare(case, seed):
    gemms, x16 = _inputs(case, seed)
    form = case["form"]
    weights = [w if case.get("entry") == "dense" else _packed(w, g[3]) for (_, w, _), g in zip(gemms, _gemms(case))]
    state = {"form": form, "mode": case.get("mode", "eager"), "entry": case.get("entry", "sparse")}
    if form == "mlp":
        m, c, h = case["m"], case["c"], case["hidden"]
        qscale, scale = _mlp_scales(case, gemms)
        state.update(x=x16, w1=weights[0], w2=weights[1], qscale=qscale, scale=scale,
                     xq=torch.empty((m, c), dtype=torch.int8, device="cuda"),
                     hq=torch.empty((m, h), dtype=torch.int8, device="cuda"),
                     y=torch.empty((m, c), dtype=torch.float16, device="cuda"))
        return state
    shapes = _gemms(case)
    state["outs"] = [_outputs(m, n, case["out"]) for m, _, n, _ in shapes]
    state["calls"] = [(x, w, {**o, **_multipliers(case["out"], g[1], s_w)})
                      for (x, _, s_w), w, o, g in zip(gemms, weights, state["outs"], shapes)]
    if state["mode"] == "carried":
        _carried(state)
    if state["mode"] == "graph":
        _layer(state)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _layer(state)
    return state


def _layer(state):
    for x, w, args in state["calls"]:
        nmspmm.spmm(x, w, **args)


def run(state):
    form = state["form"]
    if form == "mlp":
        nmspmm.quantize_f16(state["x"], 1.0 / S_X, xq=state["xq"])
        nmspmm.spmm(state["xq"], state["w1"], Yq=state["hq"], qscale=state["qscale"])
        nmspmm.spmm(state["hq"], state["w2"], Yh=state["y"], scale=state["scale"])
        return {"xq": state["xq"], "hq": state["hq"], "y": state["y"]}
    if state["entry"] == "dense":
        x, w, args = state["calls"][0]
        nmspmm.gemm_i8_dense(x, w, **args)
    elif state["mode"] == "graph":
        state["graph"].replay()
    elif state["mode"] == "carried":
        for (x, _, args), w, plan, job in zip(state["calls"], state["weights"], state["plans"], state["jobs"]):
            nmspmm.spmm(x, w, plan=plan, job=job, **args)
    else:
        _layer(state)
    return state["outs"]


def _stored_bytes(n, k, pattern):
    """Bytes of a weight in its packed form: N/M values and their positions or masks (a dense one as it is)."""
    if pattern == "8:8":
        return n * k
    d = nmspmm.compress_size(n, k, *_pattern(pattern))
    return d.vals_bytes + d.meta_bytes


def work(case):
    """Activations, packed weights and multipliers read once, outputs written once; 2 m n k operations of the equivalent
    dense product, halved where the pattern fits the 4:2 structured-sparse matrix instruction."""
    nbytes = flops = 0
    for i, (m, k, n, pattern) in enumerate(_gemms(case)):
        N, M = _pattern(pattern)
        nbytes += _stored_bytes(n, k, pattern) if case.get("entry") != "dense" else n * k
        flops += 2 * m * n * k // (2 if N <= 2 else 1)
        out = ("i8", "f16")[i] if case["form"] == "mlp" else case["out"]
        nbytes += m * n * sum(s for o, s in (("i32", 4), ("f16", 2), ("i8", 1)) if o in out)
        nbytes += 4 * n * sum(o in out for o in ("f16", "i8")) + m * k
        if case["form"] == "mlp" and i == 0:
            nbytes += 2 * m * k + m * k  # fp16 activations read, their codes written (and read by fc1, above)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Whole numbers are the same.  fp16 results are one rounding of an exact int32 times a binary32 multiplier: off by
    2.1e-4 from 64 bits (2-norm), and by no more than one code (2^-10) where a correct implementation rounds a tie
    through binary32."""
    if case["form"] == "mlp" or "f16" in case.get("out", ""):
        return {"rel": 8e-4, "max": 2e-3}
    return "exact"


def exact(case, seed):
    """The same products in 64 bits (exact: every sum is below 2^53)."""
    gemms, x16 = _inputs(case, seed)
    if case["form"] == "mlp":
        # the int8 codes are defined in binary32: q8(v) = round to nearest even, saturated
        qscale, scale = _mlp_scales(case, gemms)
        inv = torch.tensor(1.0 / S_X, dtype=torch.float32, device="cuda")
        xq = (x16.float() * inv).round().clamp(-127, 127)
        y1 = xq.double() @ gemms[0][1].double().T
        hq = (y1.float() * qscale).round().clamp(-127, 127)
        y = (hq.double() @ gemms[1][1].double().T) * scale.double()
        return {"xq": xq.to(torch.int8), "hq": hq.to(torch.int8), "y": y}
    res = []
    for (x, w, s_w), (_, k, _, _) in zip(gemms, _gemms(case)):
        y = x.double() @ w.double().T
        o, mul = {}, _multipliers(case["out"], k, s_w)
        if "i32" in case["out"]:
            o["Y"] = y.to(torch.int32)
        if "f16" in case["out"]:
            o["Yh"] = y * mul["scale"].double()
        if "i8" in case["out"]:
            o["Yq"] = (y.float() * mul["qscale"]).round().clamp(-127, 127).to(torch.int8)
        res.append(o)
    return res
