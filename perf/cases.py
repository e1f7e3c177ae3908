"""Workloads of the Sherry 3:4 ternary product, for timing and comparing builds.

A case is one piece of what a program that serves (or packs) a 1.25-bit model
does with this library, through its public calls:

* ``linear``: one product on its own: fp32 activations of m tokens in, quantized
  per token, times one packed matrix (m = 1: the fused call);
* ``layer``: the seven projections of one decoder layer, in the order a model
  needs them (q/k/v, o, gate/up, down: four inputs, four products or groups);
* ``step``: the projections of every layer in one grouped launch, as the
  benchmark runs a decode step;
* ``pack``: fp32 weights to packed bytes, on the device, in both layouts.

Options in use: one weight scale per tensor, per output channel or per 128
weights of a channel; tiled weights or (up to 16 tokens) lane-interleaved ones;
int32 sums beside the fp32 outputs; row lengths that are not whole units.
"""
from __future__ import annotations

import math
import zlib

import torch

import paper_2601_07892_amd as sh

GROUP = 128  # weights per scale with "group" scales


def listed():
    return [
        # the smallest call: one token through one 2048 x 2048 projection
        dict(name="linear_1tok_2048", op="linear", m=1, n=2048, k=2048, scales="tensor",
             layout="tiled", acc=False, outliers=False),
        # a decoder layer (LLaMA-3.2-3B) at one token, launch after launch, as
        # a model with attention between the products runs it
        dict(name="layer_1tok_3b", op="layer", m=1, hidden=3072, kv=1024, inter=8192,
             scales="channel", layout="il", outliers=False),
        # the benchmark's decode step: every projection of LLaMA-3.2-1B, one launch
        dict(name="step_1tok_1b", op="step", m=1, hidden=2048, kv=512, inter=8192, layers=16,
             scales="tensor", layout="il", outliers=False),
        # the same at 8B scale on the tiled layout: the largest weight stream
        dict(name="step_1tok_8b", op="step", m=1, hidden=4096, kv=1024, inter=14336, layers=32,
             scales="tensor", layout="tiled", outliers=False),
        # small batches of a served LLaMA-3.2-3B: 4 tokens with the paper's
        # default granularity (one scale per 128 weights), 16 tokens interleaved
        dict(name="step_4tok_3b_group", op="step", m=4, hidden=3072, kv=1024, inter=8192,
             layers=28, scales="group", layout="tiled", outliers=False),
        dict(name="step_16tok_3b", op="step", m=16, hidden=3072, kv=1024, inter=8192, layers=28,
             scales="channel", layout="il", outliers=False),
        # a larger decode batch at 8B scale
        dict(name="step_64tok_8b", op="step", m=64, hidden=4096, kv=1024, inter=14336, layers=32,
             scales="tensor", layout="tiled", outliers=False),
        # a short prompt, sizes that fill neither tiles nor units
        dict(name="layer_37tok_ragged", op="layer", m=37, hidden=1204, kv=300, inter=3380,
             scales="channel", layout="tiled", outliers=True),
        # prefill of a LLaMA-3.2-3B layer: 2048 tokens, outlier channels; and a
        # shorter prompt with one scale per 128 weights
        dict(name="layer_2048tok_3b", op="layer", m=2048, hidden=3072, kv=1024, inter=8192,
             scales="tensor", layout="tiled", outliers=True),
        dict(name="layer_512tok_3b_group", op="layer", m=512, hidden=3072, kv=1024, inter=8192,
             scales="group", layout="tiled", outliers=True),
        # the largest product: an 8B-scale gate projection over a long prompt batch
        dict(name="linear_8192tok_8b_gate", op="linear", m=8192, n=14336, k=4096,
             scales="channel", layout="tiled", acc=False, outliers=True),
        # loading a model: ternarize, pack and interleave an 8B-scale down projection
        dict(name="pack_8b_down", op="pack", n=4096, k=14336),
    ]


MAX_OPS = 8.9e11  # multiply-adds x 2 of a drawn case (the largest listed ones have 8.9e11 and 9.6e11)
MAX_WEIGHTS = 7.0e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A row length or row count: mostly whole units, some ragged (a multiple of 4)."""
    g = rng.choice([128, 128, 128, 64, 4])
    return max(lo, min(hi, _log_int(rng, lo, hi) // g * g)) // 4 * 4


def draw(rng):
    op = rng.choice(["linear", "linear", "linear", "layer", "layer", "layer", "step", "step",
                     "step", "pack"])
    if op == "pack":
        return dict(op="pack", n=_size(rng, 256, 8192), k=_size(rng, 256, 14336))
    scales = rng.choice(["tensor", "channel", "group"])
    outliers = rng.random() < 0.5
    if op == "linear":
        n, k = _size(rng, 512, 14336), _size(rng, 512, 14336)
        m = _log_int(rng, 1, max(1, min(16384, int(MAX_OPS / (2 * n * k)))))
        acc = rng.random() < 0.25
        return dict(op=op, m=m, n=n, k=k, scales=scales, layout="tiled", acc=acc,
                    outliers=outliers)
    hidden = _size(rng, 768, 4096)
    kv = max(64, hidden // rng.choice([1, 2, 4, 8]) // 4 * 4)
    g = rng.choice([128, 128, 4])
    inter = min(14336, int(hidden * rng.uniform(2.0, 4.0)) // g * g)
    per_layer = 2 * hidden * hidden + 2 * kv * hidden + 3 * hidden * inter
    c = dict(op=op, hidden=hidden, kv=kv, inter=inter)
    if op == "layer":
        c["m"] = _log_int(rng, 1, min(4096, int(MAX_OPS / (2 * per_layer))))
    else:
        c["layers"] = max(2, min(_log_int(rng, 2, 32), int(MAX_WEIGHTS / per_layer)))
        most = max(1, min(64, int(MAX_OPS / (2 * per_layer * c["layers"]))))
        c["m"] = min(most, rng.choice([1, 1, rng.randint(2, 4), rng.randint(5, 16),
                                       rng.randint(17, 64)]))
    il = c["m"] <= 16 and scales != "group" and rng.random() < 0.6
    c.update(scales=scales, layout="il" if il else "tiled", outliers=outliers)
    return c


# ---- inputs -------------------------------------------------------------------

def _gen(seed, *key):
    g = torch.Generator(device="cuda")
    g.manual_seed(zlib.crc32(repr((int(seed),) + key).encode()) + (int(seed) << 32))
    return g


def _dense(seed, n, k, *key):
    """Latent fp32 weights ~ N(0, 0.02^2)."""
    return torch.randn((n, k), generator=_gen(seed, "w", n, k, *key), device="cuda") * 0.02


def _acts(seed, m, k, outliers, *key):
    """fp32 activations ~ N(0, 1); with outliers, 1% of the channels x 20."""
    g = _gen(seed, "x", m, k, *key)
    x = torch.randn((m, k), generator=g, device="cuda")
    if outliers:
        ch = torch.randperm(k, generator=g, device="cuda")[:max(1, k // 100)]
        x[:, ch] *= 20.0
    return x


def _w_scale(seed, *key):
    u = zlib.crc32(repr((int(seed), "s") + key).encode()) / 2.0 ** 32
    return float(torch.tensor(0.01 + 0.04 * u, dtype=torch.float32))


def _group_scales(seed, n, k, *key):
    return torch.rand((n, -(-k // GROUP)), generator=_gen(seed, "gs", n, k, *key),
                      device="cuda") * 0.04 + 0.01


class _Linear:
    """One packed projection as a program keeps it."""

    def __init__(self, case, seed, n, k, *key):
        self.n, self.k, self.key = n, k, key
        w = _dense(seed, n, k, *key)
        tiled = torch.empty(sh.sherry_packed_bytes(n, k), dtype=torch.uint8, device="cuda")
        alpha = torch.empty(n, dtype=torch.float32, device="cuda")
        sh.sherry_ternarize_pack(w, n, k, tiled, alpha)
        self.w = tiled
        if case["layout"] == "il":
            self.w = torch.empty_like(tiled)
            sh.sherry_interleave(tiled, self.w, n, k)
        self.scale, self.channel, self.group = 0.0, None, None
        if case["scales"] == "tensor":
            self.scale = _w_scale(seed, *key)
        elif case["scales"] == "channel":
            self.channel = alpha
        else:
            self.group = _group_scales(seed, n, k, *key)

    def fill(self, d, x, x_scale, y, m=None):
        d.w, d.x, d.x_scale, d.y = self.w.data_ptr(), x.data_ptr(), x_scale.data_ptr(), y.data_ptr()
        d.acc = None
        d.w_scales = self.channel.data_ptr() if self.channel is not None else None
        d.w_group_scales = self.group.data_ptr() if self.group is not None else None
        d.n, d.k, d.w_scale = self.n, self.k, self.scale
        if m is not None:
            d.m = m


def _to_device(descs):
    return torch.from_numpy(sh.descs_to_bytes(descs)).cuda()


def _layer_groups(case):
    """(input length, projections (name, n)) of the four inputs of a layer."""
    h, kv, it = case["hidden"], case["kv"], case["inter"]
    return [(h, [("q", h), ("k", kv), ("v", kv)]), (h, [("o", h)]),
            (h, [("gate", it), ("up", it)]), (it, [("down", h)])]


class _Group:
    """Products that read one input (or, in a step, many inputs), in one launch."""

    def __init__(self, case, m, linears, xs, sxs, ys, qs):
        self.m, self.il, self.count = m, case["layout"] == "il", len(linears)
        if m == 1:
            descs = (sh.sherry_gemv_f32_desc * self.count)()
            for d, lin, x, sx, y in zip(descs, linears, xs, sxs, ys):
                lin.fill(d, x, sx, y)
            prepare = sh.sherry_gemv_f32_il_batched_prepare if self.il else \
                sh.sherry_gemv_f32_batched_prepare
            self.blocks = prepare(descs)
        else:
            descs = (sh.sherry_gemm_desc * self.count)()
            for d, lin, q, sx, y in zip(descs, linears, qs, sxs, ys):
                lin.fill(d, q, sx, y, m)
            prepare = sh.sherry_gemm_il_batched_prepare if self.il else \
                sh.sherry_gemm_batched_prepare
            self.blocks, self.value = prepare(descs)
        self.descs = _to_device(descs)

    def run(self):
        if self.m == 1:
            call = sh.sherry_gemv_f32_il_batched if self.il else sh.sherry_gemv_f32_batched
            call(self.descs, self.count, self.blocks)
        else:
            call = sh.sherry_gemm_il_batched if self.il else sh.sherry_gemm_batched
            call(self.descs, self.count, self.blocks, self.value)


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    op = case["op"]
    st = {"op": op, "case": case}
    if op == "pack":
        n, k = case["n"], case["k"]
        st["w"] = _dense(seed, n, k, "pack")
        st["packed"] = _empty(sh.sherry_packed_bytes(n, k), torch.uint8)
        st["il"] = torch.empty_like(st["packed"])
        st["alpha"] = _empty(n, torch.float32)
        return st
    m = case["m"]
    if op == "linear":
        st["lin"] = _Linear(case, seed, case["n"], case["k"], "linear")
        st["x"] = _acts(seed, m, case["k"], case["outliers"], "linear")
        st["q"] = _empty((m, case["k"]), torch.int8)
        st["sx"] = _empty(m, torch.float32)
        st["y"] = _empty((m, case["n"]), torch.float32)
        st["acc"] = _empty((m, case["n"]), torch.int32) if case["acc"] else None
        return st
    if op == "layer":
        st["parts"] = []
        for i, (k, projs) in enumerate(_layer_groups(case)):
            p = {"lins": [_Linear(case, seed, n, k, name) for name, n in projs],
                 "x": _acts(seed, m, k, case["outliers"], i), "q": _empty((m, k), torch.int8),
                 "sx": _empty(m, torch.float32),
                 "ys": [_empty((m, n), torch.float32) for _, n in projs]}
            count = len(projs)
            if count > 1 or (m <= 16 and case["layout"] == "il"):
                p["group"] = _Group(case, m, p["lins"], [p["x"]] * count, [p["sx"]] * count,
                                    p["ys"], [p["q"]] * count)
            st["parts"].append(p)
        return st
    # step: one flat output buffer, one input per product group
    lins, xs, qs, sxs, ys, quant = [], [], [], [], [], []
    groups = _layer_groups(case)
    st["y"] = _empty(case["layers"] * m * sum(n for _, ps in groups for _, n in ps), torch.float32)
    st["sx"] = _empty(case["layers"] * len(groups) * m, torch.float32)
    at, row = 0, 0
    for layer in range(case["layers"]):
        for i, (k, projs) in enumerate(groups):
            x = _acts(seed, m, k, case["outliers"], layer, i)
            q = _empty((m, k), torch.int8)
            sx = st["sx"][row:row + m]
            row += m
            quant.append((x, q, sx, k))
            for name, n in projs:
                lins.append(_Linear(case, seed, n, k, layer, name))
                xs.append(x)
                qs.append(q)
                sxs.append(sx)
                ys.append(st["y"][at:at + m * n])
                at += m * n
    st["keep"] = (lins, xs, qs)
    st["group"] = _Group(case, m, lins, xs, sxs, ys, qs)
    if m > 1:
        descs = (sh.sherry_quant_desc * len(quant))()
        for d, (x, q, sx, k) in zip(descs, quant):
            d.x, d.q, d.x_scale, d.m, d.k = x.data_ptr(), q.data_ptr(), sx.data_ptr(), m, k
        st["quant_rows"], st["quant_k"] = sh.sherry_quantize_act_batched_prepare(descs)
        st["quant"], st["quant_count"] = _to_device(descs), len(quant)
    return st


# ---- one pass -----------------------------------------------------------------

def _product(lin, x, q, sx, y, acc, m):
    """One product of m tokens from fp32 activations (m > 1: q and sx are quantized already)."""
    n, k = lin.n, lin.k
    if m == 1:
        if lin.group is not None:
            sh.sherry_gemv_f32_group(lin.w, x, sx, lin.group, y, acc, n, k)
        elif lin.channel is not None:
            sh.sherry_gemv_f32_channel(lin.w, x, sx, lin.channel, y, acc, n, k)
        else:
            sh.sherry_gemv_f32(lin.w, x, sx, lin.scale, y, acc, n, k)
    elif lin.group is not None:
        sh.sherry_gemm_group(lin.w, q, sx, lin.group, y, acc, m, n, k)
    elif lin.channel is not None:
        sh.sherry_gemm_channel(lin.w, q, sx, lin.channel, y, acc, m, n, k)
    else:
        sh.sherry_gemm(lin.w, q, sx, lin.scale, y, acc, m, n, k)


def run(state):
    op = state["op"]
    if op == "pack":
        n, k = state["case"]["n"], state["case"]["k"]
        sh.sherry_ternarize_pack(state["w"], n, k, state["packed"], state["alpha"])
        sh.sherry_interleave(state["packed"], state["il"], n, k)
        return {"packed": state["packed"], "il": state["il"], "alpha": state["alpha"]}
    m = state["case"]["m"]
    if op == "linear":
        if m > 1:
            sh.sherry_quantize_act(state["x"], state["q"], state["sx"])
        _product(state["lin"], state["x"], state["q"], state["sx"], state["y"], state["acc"], m)
        out = {"y": state["y"], "sx": state["sx"]}
        if m > 1:
            out["q"] = state["q"]
        if state["acc"] is not None:
            out["acc"] = state["acc"]
        return out
    if op == "layer":
        for p in state["parts"]:
            if m > 1:
                sh.sherry_quantize_act(p["x"], p["q"], p["sx"])
            if "group" in p:
                p["group"].run()
            else:
                _product(p["lins"][0], p["x"], p["q"], p["sx"], p["ys"][0], None, m)
        return {"ys": [y for p in state["parts"] for y in p["ys"]],
                "sx": [p["sx"] for p in state["parts"]]}
    if m > 1:
        sh.sherry_quantize_act_batched(state["quant"], state["quant_count"], state["quant_rows"],
                                       state["quant_k"])
    state["group"].run()
    return {"y": state["y"], "sx": state["sx"]}


# ---- what a pass cannot do without --------------------------------------------

def _product_work(case, n, k):
    m = case["m"]
    packed = -(-n // 64) * 64 * (-(-k // 128) * 128) * 5 / 32
    scales = {"tensor": 0, "channel": 4 * n, "group": 4 * n * -(-k // GROUP)}[case["scales"]]
    return packed + scales + 4 * m * n, 2.0 * m * n * k


def work(case):
    """Packed weights, scales and fp32 activations read once, outputs written
    once; 2mnk int8 operations (each weight as the dense matrix units take it)."""
    if case["op"] == "pack":
        n, k = case["n"], case["k"]
        packed = -(-n // 64) * 64 * (-(-k // 128) * 128) * 5 / 32
        return {"bytes": 4.0 * n * k + 2 * packed + 4 * n, "flops": 0.0}
    m = case["m"]
    if case["op"] == "linear":
        b, f = _product_work(case, case["n"], case["k"])
        b += 4 * m * case["k"] + 4 * m + (4 * m * case["n"] if case["acc"] else 0)
        return {"bytes": b + (m * case["k"] if m > 1 else 0), "flops": f}
    b = f = 0.0
    for k, projs in _layer_groups(case):
        b += 4 * m * k + 4 * m
        for _, n in projs:
            pb, pf = _product_work(case, n, k)
            b, f = b + pb, f + pf
    times = case.get("layers", 1)
    return {"bytes": times * b, "flops": times * f}


def tolerance(case):
    # int32 sums are exact; y = float(sum) * (sx * sw) rounds twice (measured
    # 4e-8 off the fp64 result), and another order of the scale products would
    # round elsewhere.  Per-group sums add up to 64 scaled terms in fp32, in an
    # order of the kernel's choice (measured 1e-7).  About four times each.
    if case["op"] == "pack":
        return {"rel": 1.2e-7}  # alpha's fp64 sum in another order: the last bit of fp32
    if case["scales"] == "group":
        return {"rel": 4e-7, "max": 5e-6}
    return {"rel": 1.6e-7, "max": 5e-7}


# ---- 64-bit reference ----------------------------------------------------------

def _ternary(w):
    """(Eq. 4 ternary matrix, Eq. 5 mean |w| per row) of fp32 weights, in fp64."""
    n, k = w.shape
    b = w.double().view(n, k // 4, 4)
    a = b.abs()
    lo = a.amin(dim=2, keepdim=True)
    first = (a == lo).to(torch.int32).cumsum(dim=2) == 1
    drop = first & (a == lo)  # the lowest position of the smallest magnitude
    t = torch.where(b < 0, -1.0, 1.0).double().masked_fill(drop, 0.0)
    alpha = a.masked_fill(drop, 0.0).sum(dim=(1, 2)) / (3 * (k // 4))
    return t.view(n, k), alpha


def _quantized(x):
    """Per-token int8 values (as fp64) and scales: s = absmax / 127 and x / s in fp32."""
    s = (x.abs().amax(dim=1).double() / 127.0).float()
    # the fp64 quotient of two fp32 numbers rounds to the fp32 quotient
    q = (x.double() / s.double()[:, None]).float().round().clamp(-127, 127)
    return q.double(), s.double()


def _exact_product(case, seed, q, s, n, k, *key):
    t, alpha = _ternary(_dense(seed, n, k, *key))
    if case["scales"] == "group":
        g = _group_scales(seed, n, k, *key).double()
        t = t * g.repeat_interleave(GROUP, dim=1)[:, :k]
        return (q @ t.t().contiguous()) * s[:, None], None
    acc = q @ t.t().contiguous()
    scale = _w_scale(seed, *key) if case["scales"] == "tensor" else alpha.float().double()
    return acc * s[:, None] * scale, acc


def exact(case, seed):
    op = case["op"]
    if op == "pack":
        _, alpha = _ternary(_dense(seed, case["n"], case["k"], "pack"))
        return {"packed": None, "il": None, "alpha": alpha}
    m = case["m"]
    if op == "linear":
        q, s = _quantized(_acts(seed, m, case["k"], case["outliers"], "linear"))
        y, _ = _exact_product(case, seed, q, s, case["n"], case["k"], "linear")
        out = {"y": y, "sx": s}
        if m > 1:
            out["q"] = None
        if case["acc"]:
            out["acc"] = None
        return out
    ys, sxs = [], []
    for layer in range(case["layers"] if op == "step" else 1):
        for i, (k, projs) in enumerate(_layer_groups(case)):
            key = (layer, i) if op == "step" else (i,)
            q, s = _quantized(_acts(seed, m, k, case["outliers"], *key))
            sxs.append(s)
            for name, n in projs:
                wkey = (layer, name) if op == "step" else (name,)
                ys.append(_exact_product(case, seed, q, s, n, k, *wkey)[0])
    if op == "layer":
        return {"ys": ys, "sx": sxs}
    return {"y": torch.cat([y.reshape(-1) for y in ys]), "sx": torch.cat(sxs)}
