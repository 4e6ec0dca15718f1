"""The work that a user of this library has it do, as timed cases.

Each case is one call (or the few calls that belong together) of the public
Python entry points on the shapes of Gemma-3-1B (hidden 1152, FFN 6912,
vocabulary 262144, 26 layers, heads of 256), on ragged batch sizes of them and
on some generic FFN shapes.  Inputs follow the recipe of
``paper_2608_28003_amd.synth``, drawn on the GPU: activations N(0, 1) with 1 %
outlier channels x 30, weights N(0, 0.02^2), keys and values N(0, 2^2).

``exact`` evaluates the same definitions with plain torch in binary64; the
roundings that define the result (codes, scales, bf16 activations between
stages) are kept, sums and the GELU are binary64.
"""

import math

import numpy as np
import torch

from paper_2608_28003_amd import w8a8

D, F, V, LAYERS, HEAD = 1152, 6912, 262144, 26, 256
MAPS = {"bf16": (0, 0), "5+5": (5, 5), "10+10": (10, 10), "all26": (26, 0)}
DEV = "cuda"

# hidden and FFN widths of the drawn blocks: the model's, and generic ones
BLOCKS = [(1152, 6912), (640, 2048), (1536, 4608), (2560, 10240)]
# attention projections (fused QKV, O), one FFN projection each way, a ragged one
LINEARS = [(1536, 1152), (1152, 1024), (6912, 1152), (1152, 6912), (1000, 1168)]


def listed():
    return [
        # one decode step of the FFN stack: every layer INT8, INT8 lm_head
        {"name": "decode_step", "kind": "stack", "m": 1, "map": "all26"},
        # one FFN block in decode with a handful of sequences
        {"name": "ffn_int8_8", "kind": "ffn", "dt": "int8", "m": 8, "d": D, "f": F},
        # the same block on a short prompt
        {"name": "ffn_int8_128", "kind": "ffn", "dt": "int8", "m": 128, "d": D, "f": F},
        # the same block on a long prompt
        {"name": "ffn_int8_2048", "kind": "ffn", "dt": "int8", "m": 2048, "d": D, "f": F},
        # a layer that the precision map keeps in bf16, on a ragged prompt
        {"name": "ffn_bf16_1021", "kind": "ffn", "dt": "bf16", "m": 1021, "d": D, "f": F},
        # the FP8 variant of the block
        {"name": "ffn_fp8_1500", "kind": "ffn", "dt": "fp8", "m": 1500, "d": D, "f": F},
        # the attention block's fused QKV projection on a ragged prompt
        {"name": "qkv_int8_777", "kind": "linear", "m": 777, "n": 1536, "k": D, "x": "bf16", "y": "bf16"},
        # logits of a decode batch
        {"name": "lm_head_64", "kind": "lm_head", "dt": "int8", "m": 64},
        # append one token to a long INT8 cache and attend it
        {"name": "attn_int8_32768", "kind": "attn", "rows": 32768, "window": 32768, "heads": 4, "int8": True},
        # a prompt through the stack under the paper's 10+10 map
        {"name": "prefill_10+10_512", "kind": "stack", "m": 512, "map": "10+10"},
        # the benchmark's step: a long prompt, every layer and the lm_head INT8
        {"name": "prefill_all26_2048", "kind": "stack", "m": 2048, "map": "all26"},
        # loading a model: smoothing factors and codes of the lm_head's weights
        {"name": "quantise_lm_head", "kind": "weights", "n": V, "k": D, "w": "bf16"},
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ffn", "ffn", "ffn", "linear", "lm_head", "attn", "stack", "weights"])
    if kind == "ffn":
        d, f = rng.choice(BLOCKS)
        return {"kind": kind, "dt": rng.choice(["int8", "int8", "bf16", "fp8"]),
                "m": _spread(rng, 1, 4096), "d": d, "f": f}
    if kind == "linear":
        n, k = rng.choice(LINEARS)
        return {"kind": kind, "m": _spread(rng, 1, 4096), "n": n, "k": k,
                "x": rng.choice(["bf16", "bf16", "f32"]), "y": rng.choice(["bf16", "f32"])}
    if kind == "lm_head":
        return {"kind": kind, "dt": rng.choice(["int8", "int8", "bf16", "fp8"]), "m": _spread(rng, 1, 512)}
    if kind == "attn":
        rows = _spread(rng, 300, 131072)
        return {"kind": kind, "rows": rows, "window": rng.choice([rows, min(rows, 1024)]),
                "heads": rng.choice([1, 2, 4, 4, 8]), "int8": rng.random() < 0.6}
    if kind == "stack":
        return {"kind": kind, "m": _spread(rng, 1, 1024), "map": rng.choice(sorted(MAPS))}
    k = rng.choice([D, D, 1024, 2560, F])
    return {"kind": kind, "n": _spread(rng, 1000, V * D // max(k, D)), "k": k, "w": rng.choice(["bf16", "bf16", "f32"])}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _normal(g, shape, sigma=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=g, device=DEV) * sigma).to(dtype)


def _acts(g, m, k, dtype=torch.bfloat16):
    """m tokens and the calibration maximum of 64 more, with the same outlier channels."""
    factor = torch.ones(k, device=DEV)
    factor[torch.randperm(k, generator=g, device=DEV)[:max(1, round(0.01 * k))]] = 30.0
    x = torch.randn((m + 64, k), generator=g, device=DEV) * factor
    return x[:m].to(dtype).contiguous(), x[m:].to(torch.bfloat16).abs().amax(0).float(), x[m:].to(torch.bfloat16)


def _delta(act_amax, weights):
    w = weights[0].abs().amax(0).float()
    for other in weights[1:]:
        w = torch.maximum(w, other.abs().amax(0).float())
    a, w = act_amax.double().clamp_min(1e-5), w.double().clamp_min(1e-5)
    return (a.sqrt() / w.sqrt()).float()


def _ffn_weights(g, d, f):
    return _normal(g, (f, d), 0.02), _normal(g, (f, d), 0.02), _normal(g, (d, f), 0.02)


def _ffn_deltas(w, act_amax, x_cal):
    """Smoothing of the block's two inputs; the down input's statistic is gathered on the calibration tokens."""
    wg, wu, wd = w
    xc = x_cal.float()
    h = torch.nn.functional.gelu(xc @ wg.float().t(), approximate="tanh") * (xc @ wu.float().t())
    return _delta(act_amax, [wg, wu]), _delta(h.abs().amax(0), [wd])


def _bytes(n):
    return torch.empty(max(1, int(n)), dtype=torch.uint8, device=DEV)


def _prec(case):
    lo, hi = MAPS[case["map"]]
    return np.array([1 if l < lo or l >= LAYERS - hi else 0 for l in range(LAYERS)], np.uint8)


def _tensors(case, seed):
    """The plain tensors of a case, the same ones for prepare() and exact()."""
    g, kind = _gen(seed), case["kind"]
    if kind == "ffn":
        w = _ffn_weights(g, case["d"], case["f"])
        x, amax, x_cal = _acts(g, case["m"], case["d"])
        return {"x": x, "w": w, "deltas": _ffn_deltas(w, amax, x_cal)}
    if kind == "linear":
        dt = {"bf16": torch.bfloat16, "f32": torch.float32}[case["x"]]
        w = _normal(g, (case["n"], case["k"]), 0.02, dt)
        x, amax, _ = _acts(g, case["m"], case["k"], dt)
        return {"x": x, "w": w, "delta": _delta(amax, [w])}
    if kind == "lm_head":
        w = _normal(g, (V, D), 0.02)
        x, amax, _ = _acts(g, case["m"], D)
        return {"x": x, "w": w, "delta": _delta(amax, [w])}
    if kind == "attn":
        k, v = (_normal(g, (case["rows"], HEAD), 2.0) for _ in range(2))
        ch = torch.randperm(HEAD, generator=g, device=DEV)[:8]
        k[:, ch] *= 8.0
        qkv = _normal(g, ((case["heads"] + 2) * HEAD,), 2.0)
        qkv[case["heads"] * HEAD + ch] *= 8.0
        return {"k": k, "v": v, "qkv": qkv}
    if kind == "weights":
        w = _normal(g, (case["n"], case["k"]), 0.02, {"bf16": torch.bfloat16, "f32": torch.float32}[case["w"]])
        return {"w": w, "amax": _acts(g, 1, case["k"])[1]}
    x, amax, x_cal = _acts(g, case["m"], D)
    return {"x": x, "x_cal": x_cal, "g": g}  # the layers follow on the same generator, see _layer


def _rms(x):
    return (x.double() / (x.double().square().mean(-1, keepdim=True) + 1e-6).sqrt()).to(torch.bfloat16)


def _layer(t):
    """The next layer's weights and smoothing; its block input is a normalised token stream."""
    w = _ffn_weights(t["g"], D, F)
    x_cal = _rms(t["x_cal"])
    return w, _ffn_deltas(w, x_cal.abs().amax(0).float(), x_cal)


def _head(t):
    w = _normal(t["g"], (V, D), 0.02)
    return w, _delta(_rms(t["x_cal"]).abs().amax(0).float(), [w])


# ------------------------------------------------------------------ the calls

def prepare(case, seed):
    t, kind = _tensors(case, seed), case["kind"]
    s = {"kind": kind, "dt": case.get("dt")}
    if kind == "ffn":
        m, d, f = case["m"], case["d"], case["f"]
        if case["dt"] == "bf16":
            s["layer"], need = w8a8.FfnBF16.from_weights(*t["w"]), w8a8.bf16_ffn_workspace_bytes(m, d, f)
        elif case["dt"] == "fp8":
            s["layer"], need = w8a8.fp8_ffn_layer(*t["w"], *t["deltas"]), w8a8.fp8_ffn_workspace_bytes(m, d, f)
        else:
            s["layer"], need = w8a8.FfnW8A8.from_weights(*t["w"], *t["deltas"]), w8a8.ffn_workspace_bytes(m, d, f)
        s.update(x=t["x"], ws=_bytes(need), out=torch.empty((m, d), dtype=torch.bfloat16, device=DEV))
    elif kind == "linear":
        s["layer"] = w8a8.LinearW8A8.from_weight(t["w"], t["delta"])
        s.update(x=t["x"], ws=_bytes(w8a8.linear_workspace_bytes(case["m"], case["n"], case["k"])),
                 out=torch.empty((case["m"], case["n"]), device=DEV,
                                 dtype={"bf16": torch.bfloat16, "f32": torch.float32}[case["y"]]))
    elif kind == "lm_head":
        m = case["m"]
        if case["dt"] == "bf16":
            s["layer"], need = w8a8.pack_bf16(t["w"]), w8a8.bf16_linear_workspace_bytes(m, V, D)
        elif case["dt"] == "fp8":
            s["layer"], need = w8a8.fp8_linear_layer(t["w"], t["delta"]), w8a8.fp8_linear_workspace_bytes(m, V, D)
        else:
            s["layer"], need = w8a8.LinearW8A8.from_weight(t["w"], t["delta"]), w8a8.lm_head_workspace_bytes(m, V, D)
        s.update(x=t["x"], ws=_bytes(need), out=torch.empty((m, V), dtype=torch.bfloat16, device=DEV))
    elif kind == "attn":
        cache = w8a8.KVCache(case["rows"], int8=case["int8"], device=DEV)
        if case["rows"] > 1:
            cache.fill(0, t["k"][:-1], t["v"][:-1])
        s.update(cache=cache, qkv=t["qkv"], pos=case["rows"] - 1, window=case["window"], heads=case["heads"],
                 ws=_bytes(w8a8.attn_decode_workspace_bytes(case["rows"])),
                 out=torch.empty(case["heads"] * HEAD, dtype=torch.bfloat16, device=DEV))
    elif kind == "weights":
        s.update(w=t["w"], amax=t["amax"])
    else:
        prec, int8, bf16, unused = _prec(case), [], [], None
        for l in range(LAYERS):
            w, deltas = _layer(t)
            int8.append(w8a8.FfnW8A8.from_weights(*w, *deltas) if prec[l] else None)
            if not prec[l] or unused is None:
                unused = w8a8.FfnBF16.from_weights(*w)
            bf16.append(unused)  # a layer that the map sets to INT8 never reads its bf16 form
        w, delta = _head(t)
        stack = w8a8.Stack(int8, bf16, w8a8.LinearW8A8.from_weight(w, delta), None, V)
        s.update(stack=stack, prec=prec, x=t["x"], ws=_bytes(w8a8.stack_workspace_bytes(case["m"], D, F, V)),
                 out=torch.empty((case["m"], V), dtype=torch.bfloat16, device=DEV))
    return s


def run(s):
    kind, dt = s["kind"], s["dt"]
    if kind == "ffn":
        call = {"int8": w8a8.ffn, "bf16": w8a8.bf16_ffn, "fp8": w8a8.fp8_ffn}[dt]
        return call(s["layer"], s["x"], out=s["out"], ws=s["ws"])
    if kind == "linear":
        return w8a8.linear(s["layer"], s["x"], out=s["out"], ws=s["ws"])
    if kind == "lm_head":
        if dt == "bf16":
            return w8a8.bf16_linear(s["x"], s["layer"], V, D, out=s["out"], ws=s["ws"])
        return (w8a8.fp8_lm_head if dt == "fp8" else w8a8.lm_head)(s["layer"], s["x"], out=s["out"], ws=s["ws"])
    if kind == "attn":
        c = s["cache"]
        out = w8a8.attn_decode(s["qkv"], c, s["pos"], s["window"], n_heads=s["heads"], out=s["out"], ws=s["ws"])
        return [out, c.k, c.v, c.sk, c.sv] if c.int8 else [out, c.k, c.v]
    if kind == "weights":
        delta = w8a8.smooth_calibrate(s["amax"], [s["w"]])
        codes, scales = w8a8.quantize_weights(s["w"], delta)
        return [delta, codes, scales]
    return s["stack"].run(s["x"], s["prec"], True, out=s["out"], ws=s["ws"])


# ------------------------------------------------------------------ what the path cannot do without

def _block_bytes(d, f, dt):
    return 3 * d * f * 2 if dt == "bf16" else 3 * d * f + 4 * (2 * f + d) + 4 * (d + f)


def work(case):
    kind, m = case["kind"], case.get("m", 1)
    if kind == "ffn":
        d, f = case["d"], case["f"]
        return {"bytes": _block_bytes(d, f, case["dt"]) + 2 * m * d * 2, "flops": 6 * m * d * f}
    if kind == "linear":
        n, k = case["n"], case["k"]
        size = {"bf16": 2, "f32": 4}
        return {"bytes": n * k + 4 * n + 4 * k + m * k * size[case["x"]] + m * n * size[case["y"]], "flops": 2 * m * n * k}
    if kind == "lm_head":
        return {"bytes": V * D * (2 if case["dt"] == "bf16" else 1) + 4 * V + 4 * D + 2 * m * (D + V), "flops": 2 * m * V * D}
    if kind == "attn":
        rows = case["window"]
        return {"bytes": rows * (2 * HEAD + 8 if case["int8"] else 4 * HEAD) + 2 * (2 * case["heads"] + 2) * HEAD,
                "flops": 4 * case["heads"] * rows * HEAD}
    if kind == "weights":
        n, k = case["n"], case["k"]
        return {"bytes": n * k * ({"bf16": 2, "f32": 4}[case["w"]] + 1) + 4 * n + 8 * k, "flops": 0}
    layers = sum(_block_bytes(D, F, "int8" if p else "bf16") for p in _prec(case))
    return {"bytes": layers + V * D + 4 * V + 4 * D + 2 * m * (D + V), "flops": 6 * m * D * F * LAYERS + 2 * m * V * D}


def tolerance(case):
    kind = case["kind"]
    if kind == "weights":
        return "exact"
    if kind == "linear" and case["y"] == "f32":
        return {"rel": 1e-6}  # exact integer sums, two binary32 products
    if kind == "attn":
        return {"rel": 7e-3, "differ": 0.0}
    if kind == "stack":
        return {"rel": 3e-2}  # bf16 activations and codes through 26 normalised layers
    if kind == "ffn" and case["dt"] == "fp8":
        return {"rel": 1.5e-2}  # E4M3 codes of h follow its last bf16 bit
    return {"rel": 7e-3}  # one bf16 rounding of the result


# ------------------------------------------------------------------ the same in 64 bits

def _codes(v, dt="int8"):
    """Per-row codes (binary64) and scales (binary32) of binary32 rows."""
    s = v.abs().amax(1) / (448.0 if dt == "fp8" else 127.0)
    q = torch.where(s[:, None] > 0, v / s[:, None], torch.zeros_like(v))
    q = q.clamp(-448, 448).to(torch.float8_e4m3fn) if dt == "fp8" else q.round().clamp(-127, 127)
    return q.double(), s


def _linear64(x, w, delta, dt="int8"):
    qx, sx = _codes(x.float() / delta, dt)
    out = torch.empty((x.shape[0], w.shape[0]), dtype=torch.float64, device=DEV)
    for n in range(0, w.shape[0], 32768):
        qw, sw = _codes(w[n:n + 32768].float() * delta, dt)
        out[:, n:n + 32768] = (qx @ qw.t()) * sx.double()[:, None] * sw.double()
    return out


def _ffn64(x, w, deltas, dt):
    wg, wu, wd = w
    if dt == "bf16":
        g, u = x.double() @ wg.double().t(), x.double() @ wu.double().t()
    else:
        g, u = _linear64(x, wg, deltas[0], dt), _linear64(x, wu, deltas[0], dt)
    h = (torch.nn.functional.gelu(g, approximate="tanh") * u).to(torch.bfloat16)
    return h.double() @ wd.double().t() if dt == "bf16" else _linear64(h, wd, deltas[1], dt)


def exact(case, seed):
    t, kind = _tensors(case, seed), case["kind"]
    if kind == "ffn":
        return _ffn64(t["x"], t["w"], t["deltas"], case["dt"])
    if kind == "linear":
        return _linear64(t["x"], t["w"], t["delta"])
    if kind == "lm_head":
        if case["dt"] == "bf16":
            return torch.cat([t["x"].double() @ t["w"][n:n + 32768].double().t() for n in range(0, V, 32768)], 1)
        return _linear64(t["x"], t["w"], t["delta"], case["dt"])
    if kind == "attn":
        h, first = case["heads"], max(0, case["rows"] - case["window"])
        rows = [torch.cat([c[:-1], t["qkv"][(h + i) * HEAD:(h + i + 1) * HEAD][None]]) for i, c in enumerate((t["k"], t["v"]))]
        if case["int8"]:
            (qk, sk), (qv, sv) = (_codes(c.float()) for c in rows)
            k, v = qk * sk.double()[:, None], qv * sv.double()[:, None]
        else:
            k, v = (c.double() for c in rows)
        q = t["qkv"][:h * HEAD].double().view(h, HEAD)
        out = (torch.softmax(q @ k[first:].t() / 16.0, 1) @ v[first:]).reshape(-1)
        return [out, qk, qv, sk.double(), sv.double()] if case["int8"] else [out, k, v]
    if kind == "weights":
        delta = _delta(t["amax"], [t["w"]])
        s = torch.cat([(t["w"][n:n + 32768].float() * delta).abs().amax(1) / 127.0 for n in range(0, case["n"], 32768)])
        return [delta.double(), None, s.double()]
    x, prec = t["x"], _prec(case)
    for l in range(LAYERS):
        w, deltas = _layer(t)
        y = _ffn64(_rms(x), w, deltas, "int8" if prec[l] else "bf16").to(torch.bfloat16)
        x = (x.double() + _rms(y).double()).to(torch.bfloat16)
    w, delta = _head(t)
    return _linear64(_rms(x), w, delta)
