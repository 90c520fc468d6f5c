"""Workloads that stand for what a decoder does with this library.

A case is a pass over `layers` layers of a stack: every layer has weights and an input of its
own, so that, as in a decoder, the weights of a pass come from memory and not from a cache.
The calls of a pass are marshalled once with the package's prepare(), as a decode loop does.

op          what one layer of the pass calls
  proj      one projection, y = s_t(x) W^T (the attention output projection, or any single matrix)
  qkv       W_q, W_k, W_v in one call that forms its input from the hidden state (normalisation)
  gate_up   W_gate, W_up in one call on a state that is already normalised
  down      W_down on SiLU(gate) * up, formed in the call
  mlp       gate, up, SiLU(gate) * up and W_down in one launch
  block     a decoder block: qkv, proj, gate_up on the normalised state, down (four calls)
  batch     a decoder block for a small batch of hidden states (four grouped calls)
  calibrate thresholds of one activation site from a sample of tokens
fmt is the weight format (bf16, w8, w4); rows "padded" stores the bf16 matrices of grouped calls
256 bytes per row further apart; p is the share of input channels that are dropped.  Thresholds
are estimated from the distribution and not from the input itself, as an offline calibration does.
"""
import math

import torch

import paper_2408_14690_amd as T

EPS = 1e-5
GROUP = 128
LEVELS = [0.25, 0.4, 0.5, 0.65]
BITS = {"bf16": 16, "w8": 8, "w4": 4}


def _case(name, op, m, n=0, kv=0, f=0, fmt="bf16", rows="packed", p=0.5, batch=1, layers=1):
    return {"name": name, "op": op, "m": m, "n": n, "kv": kv, "f": f, "fmt": fmt, "rows": rows,
            "p": p, "batch": batch, "layers": layers}


def listed():
    return [
        # the smallest calls of a decode step: a square projection of a small model
        _case("proj_2048", "proj", 2048, n=2048, layers=32),
        # attention output projection, Llama-2-7B
        _case("o_7b", "proj", 4096, n=4096, layers=12),
        # q, k, v with grouped-query heads, input formed from the residual stream, Llama-3-8B
        _case("qkv_8b", "qkv", 4096, n=4096, kv=1024, layers=8),
        # gate and up of Llama-3-8B, matrices in padded rows
        _case("gate_up_8b", "gate_up", 4096, f=14336, rows="padded", layers=3),
        # W_down of Llama-3-8B on the gated intermediate
        _case("down_8b", "down", 4096, f=14336, layers=4),
        # the whole MLP of Llama-3-8B, one dependent launch
        _case("mlp_8b", "mlp", 4096, f=14336, rows="padded", layers=2),
        # the largest: decoder blocks of 70B shape
        _case("block_70b", "block", 8192, n=8192, kv=1024, f=28672, rows="padded", layers=3),
        # weight-only int8: Llama-3-8B blocks
        _case("block_8b_w8", "block", 4096, n=4096, kv=1024, f=14336, fmt="w8", layers=2),
        # weight-only int4 in groups of 128: a 70B-shaped block
        _case("block_70b_w4", "block", 8192, n=8192, kv=1024, f=28672, fmt="w4", layers=1),
        # a small batch of requests through a Llama-3-8B block
        _case("block_8b_batch8", "batch", 4096, n=4096, kv=1024, f=14336, batch=8, layers=1),
        # sizes that divide into nothing, at a low sparsity
        _case("ragged_25", "proj", 5000, n=3416, p=0.25, layers=8),
        # offline calibration of one site: 16384 tokens of a 4096-wide state
        _case("calibrate_4096", "calibrate", 4096, n=16384),
    ]


def _round(v, k):
    return max(k, int(v) // k * k)


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choice(["proj", "proj", "qkv", "gate_up", "down", "mlp", "block", "block", "batch",
                     "calibrate"])
    if op == "calibrate":
        return _sized(_case("", op, _round(_log(rng, 1024, 8192), 8), n=int(_log(rng, 1024, 16384))))
    fmt = "bf16" if op in ("gate_up", "batch") else rng.choice(["bf16", "bf16", "w8", "w4"])
    unit = {"bf16": 8, "w8": 16, "w4": 128}[fmt]
    if rng.random() < 0.5:
        unit = max(unit, 128)                    # half of the models are in round sizes
    m = _round(_log(rng, 1024, 8192), unit)
    n = _round(_log(rng, 1024, 8192), unit) if op == "proj" else m
    kv = _round(m / rng.choice([1, 4, 8]), unit)
    f = _round(m * rng.choice([2.6875, 3.5]), unit)
    rows = rng.choice(["packed", "padded"]) if fmt == "bf16" and op in ("gate_up", "mlp", "block") else "packed"
    p = rng.choice([0.0, 0.25, 0.4, 0.5, 0.5, 0.65, 0.8])
    batch = rng.randint(2, 8) if op == "batch" else 1
    return _sized(_case("", op, m, n, kv, f, fmt, rows, p, batch))


def _sized(case):
    """Without a name, with as many layers as make the pass read about 150 MB."""
    case.pop("name")
    case["layers"] = 1
    if case["op"] != "calibrate":
        outputs = sum(len(widths) for _, _, widths in _calls(case))
        case["layers"] = max(1, min(16, 60 // outputs, round(150e6 / work(case)["bytes"])))
    return case


# ---- what a layer consists of ----------------------------------------------------------------


def _calls(case):
    """The calls of one layer: (kind, input channels, output widths)."""
    op, m, n, kv, f = case["op"], case["m"], case["n"], case["kv"], case["f"]
    if op == "proj":
        return [("plain", m, [n])]
    if op == "qkv":
        return [("norm", m, [n, kv, kv])]
    if op == "gate_up":
        return [("plain", m, [f, f])]
    if op == "down":
        return [("swiglu", f, [m])]
    if op == "mlp":
        return [("mlp", m, [f, f, m])]
    if op == "block":
        return [("norm", m, [n, kv, kv]), ("plain", n, [m]), ("norm", m, [f, f]), ("swiglu", f, [m])]
    return [("batch", m, [n, kv, kv]), ("batch", n, [m]), ("batch", m, [f, f]), ("batch", f, [m])]


def _depths(kind, m, widths):
    """Input channels of each matrix of a call."""
    return [m, m, widths[0]] if kind == "mlp" else [m] * len(widths)


def work(case):
    if case["op"] == "calibrate":
        return {"bytes": 2 * case["m"] * case["n"] + 8 * T.TEAL_HIST_BINS + 4 * len(LEVELS), "flops": 0}
    bits, batch, by, fl = BITS[case["fmt"]], case["batch"], 0, 0
    for kind, m, widths in _calls(case):
        by += batch * m * {"plain": 2, "batch": 2, "mlp": 2, "norm": 8, "swiglu": 8}[kind]
        for depth, n in zip(_depths(kind, m, widths), widths):
            kept = round((1.0 - case["p"]) * depth)
            by += kept * n * bits // 8 + 4 * n * batch
            by += {"bf16": 0, "w8": 2 * n, "w4": 2 * n * (depth // GROUP)}[case["fmt"]]
            fl += 2 * kept * n * batch
    return {"bytes": by * case["layers"], "flops": fl * case["layers"]}


def tolerance(case):
    if case["op"] == "calibrate":
        return "exact"                           # counts, and thresholds that are order statistics
    if case["op"] == "mlp":
        # the intermediate is rounded to 16 bits and thresholded: where gate or up differ in the
        # last bit of their 32-bit sums one channel next to the threshold may be kept or dropped
        return {"rel": 1e-2}
    return {"rel": 2e-6}                         # 32-bit sums of exact products; measured 1e-7 .. 5e-7


# ---- inputs ------------------------------------------------------------------------------------


def _gen(seed, *at):
    g = torch.Generator(device="cuda")
    k = int(seed)
    for a in at:
        k = k * 1009 + a + 1
    g.manual_seed(k % (1 << 62))
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _laplace(g, *shape):
    u = torch.rand(shape, generator=g, device="cuda", dtype=torch.float32) - 0.4999999
    return -torch.sign(u) * torch.log1p(-2 * u.abs())


def _norm_inputs(g, m):
    """Residual stream with a few very large channels, and the weights of the normalisation."""
    h = 2.5 * _randn(g, m)
    big = torch.rand(m, generator=g, device="cuda") < 1.0 / 512.0
    return torch.where(big, 40.0 * h, h), 0.5 + 0.1 * _randn(g, m)


def _normalised(h, gamma):
    """x = binary16(binary32(binary32(h r) gamma)), r = binary32(1 / sqrt(mean(h^2) + eps))."""
    ss = h.double().square().sum()
    r = (1.0 / torch.sqrt(ss / h.numel() + EPS)).float()
    return ((h * r) * gamma).half()


def _gated(g, u):
    """SiLU(g) * u in the binary32 steps of teal.h, then binary16.  A fused multiply-add is a
    product and a sum in binary64, rounded once to binary32."""
    def f32(v):
        return v.float()

    def fma(a, b, c):
        return f32(a.double() * b + c)

    def const(v):
        return float(torch.tensor(v, dtype=torch.float32))
    z = (-g).clamp(-80.0, 80.0)
    k = torch.round(f32(z.double() * const(1.44269502)))
    r = fma(k, const(-0.693145752), z.double())
    r = fma(k, const(-1.42860677e-06), r.double())
    s = torch.full_like(r, const(1.0 / 5040.0))
    for c in (1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5, 1.0, 1.0):
        s = f32(s.double() * r.double() + const(c))
    e = f32(torch.ldexp(s.double(), k.double()))
    sg = f32(1.0 / f32(1.0 + e.double()).double())
    return f32(f32(g.double() * sg.double()).double() * u.double()).half()


def _threshold(kind, p, batch, dist):
    """The p-quantile of the magnitudes of a sample of the input's distribution that the passes
    never see, a little off it so that it is no fp16 value."""
    if p <= 0.0:
        return 0.0
    g = _gen(77, batch)
    count = 1 << 16
    if kind == "norm":
        s = _normalised(*_norm_inputs(g, count)).float().abs()
    elif kind == "swiglu":
        s = _gated(1.5 * _randn(g, count), _randn(g, count)).float().abs()
    elif kind == "batch":
        s = (_randn(g, batch, count) if dist == "gaussian" else _laplace(g, batch, count)).abs().mean(0)
    else:
        s = (_randn(g, count) if dist == "gaussian" else _laplace(g, count)).abs()
    return float(torch.sort(s).values[int(p * count)]) * 1.0001


def _matrix(g, m, n, fmt, pitch):
    """Weights N(0, 0.02^2), input-channel-major, in the format; and the values they stand for."""
    w = 0.02 * _randn(g, m, pitch)
    if fmt == "bf16":
        return {"W": w.to(torch.bfloat16), "n": n, "pitch": pitch}
    if fmt == "w8":
        scale = (w.abs().amax(0) / 127.0).half()
        q = torch.round(w / scale.float()).clamp(-127, 127).to(torch.int8)
        return {"W": q, "scale": scale, "n": n, "pitch": n}
    scale = (w.view(m // GROUP, GROUP, n).abs().amax(1) / 7.0).half()
    q = torch.round(w.view(m // GROUP, GROUP, n) / scale.float()[:, None, :]).clamp(-7, 7)
    q = q.to(torch.int8).view(m, n)
    return {"W": ((q[:, 0::2] & 15) | ((q[:, 1::2] & 15) << 4)).view(torch.uint8).contiguous(),
            "scale": scale, "n": n, "pitch": n}


def _dense(mat, fmt):
    """The matrix in 64 bits, [m][n]."""
    if fmt == "bf16":
        return mat["W"][:, :mat["n"]].double()
    if fmt == "w8":
        return mat["W"].double() * mat["scale"].double()
    b = mat["W"].view(torch.int8)
    lo, hi = ((b << 4) >> 4), (b >> 4)
    q = torch.stack([lo, hi], dim=2).view(b.shape[0], -1)
    return q.double() * mat["scale"].double().repeat_interleave(GROUP, 0)


def _inputs(case, seed):
    """The calls of every layer with their matrices, thresholds and inputs."""
    fmt, p, batch, got = case["fmt"], case["p"], case["batch"], []
    for layer in range(case["layers"]):
        for i, (kind, m, widths) in enumerate(_calls(case)):
            # states behind a normalisation are Gaussian-shaped, the others Laplacian
            dist = "laplace" if (case["op"] == "proj" or i in (1, 3)) else "gaussian"
            g = _gen(seed, layer, i)
            pad = 128 if case["rows"] == "padded" and (len(widths) > 1) else 0
            c = {"kind": kind, "m": m}
            c["mats"] = [_matrix(g, d, n, fmt, n + pad) for d, n in zip(_depths(kind, m, widths), widths)]
            t = _threshold(kind if kind != "mlp" else "plain", p, batch, dist)
            c["t"] = [t] * len(widths)
            if kind == "norm":
                c["h"], c["gamma"] = _norm_inputs(g, m)
            elif kind == "swiglu":
                c["gate"], c["up"] = 1.5 * _randn(g, m), _randn(g, m)
            elif kind == "batch":
                c["x"] = (_randn(g, batch, m) if dist == "gaussian" else _laplace(g, batch, m)).half()
            else:
                c["x"] = (_randn(g, m) if dist == "gaussian" else _laplace(g, m)).half()
            if kind == "mlp":
                # gate and up are N(0, s^2), s^2 = 0.02^2 sum of the kept x^2: the threshold of
                # their gated product, from a sample of that
                x = c["x"].float()
                s = 0.02 * float(x[x.abs() > t].square().sum().sqrt())
                v = _gated(s * _randn(_gen(78), 1 << 16), s * _randn(_gen(79), 1 << 16)).float().abs()
                c["t"][2] = 0.0 if p <= 0.0 else float(torch.sort(v).values[int(p * (1 << 16))]) * 1.0001
            got.append(c)
    return got


def _sample(case, seed):
    return _randn(_gen(seed), case["n"], case["m"]).half()


# ---- the pass ------------------------------------------------------------------------------------


def _workspace(nbytes):
    return torch.zeros(nbytes, dtype=torch.uint8, device="cuda")


def _issue(c, fmt, batch, ws):
    """One call through the library's entry points; outputs in c["out"]."""
    kind, m, mats, t, out = c["kind"], c["m"], c["mats"], c["t"], c["out"]
    W, n = [a["W"] for a in mats], [a["n"] for a in mats]
    pitch, scale = [a["pitch"] for a in mats], [a.get("scale") for a in mats]
    padded = pitch != n
    if kind == "batch":
        return T.teal_sparse_gemv_bf16_batch_multi(W, t, out, n, c["x"], batch, m, ws)
    if kind == "mlp":
        args = (c["x"], *t, *out, m, n[0], n[2], ws)
        if fmt == "bf16":
            return T.teal_sparse_mlp_bf16(*W, *args, shape=c["shape"])
        if fmt == "w8":
            return T.teal_sparse_mlp_w8(*W, *scale, *args, shape=c["shape"])
        return T.teal_sparse_mlp_w4(*W, *scale, GROUP, *args, shape=c["shape"])
    if kind == "norm":
        args = (t, out, n, c["h"], c["gamma"], EPS, m, ws)
        if fmt == "bf16" and padded:
            return T.teal_sparse_gemv_bf16_rmsnorm_multi_pitch(W, pitch, *args)
        if fmt == "bf16":
            return T.teal_sparse_gemv_bf16_rmsnorm_multi(W, *args)
        if fmt == "w8":
            return T.teal_sparse_gemv_w8_rmsnorm_multi(W, scale, *args)
        return T.teal_sparse_gemv_w4_rmsnorm_multi(W, scale, GROUP, *args)
    if kind == "swiglu":
        args = (c["gate"], c["up"], t[0], out[0], m, n[0], ws)
        if fmt == "bf16":
            return T.teal_sparse_gemv_bf16_swiglu(W[0], *args)
        if fmt == "w8":
            return T.teal_sparse_gemv_w8_swiglu(W[0], scale[0], *args)
        return T.teal_sparse_gemv_w4_swiglu(W[0], scale[0], GROUP, *args)
    if len(W) > 1:
        if padded:
            return T.teal_sparse_gemv_bf16_multi_pitch(W, pitch, t, out, n, c["x"], m, ws)
        return T.teal_sparse_gemv_bf16_multi(W, t, out, n, c["x"], m, ws)
    args = (c["x"], t[0], out[0], m, n[0], ws)
    if fmt == "bf16":
        return T.teal_sparse_gemv_bf16(W[0], *args)
    if fmt == "w8":
        return T.teal_sparse_gemv_w8(W[0], scale[0], *args)
    return T.teal_sparse_gemv_w4(W[0], scale[0], GROUP, *args)


def prepare(case, seed):
    if case["op"] == "calibrate":
        x = _sample(case, seed)
        hist = torch.zeros(T.TEAL_HIST_BINS, dtype=torch.int64, device="cuda")
        t = torch.zeros(len(LEVELS), dtype=torch.float32, device="cuda")

        def site():
            T.check(T.teal_abs_histogram(x, x.numel(), hist))
            T.check(T.teal_histogram_thresholds(hist, LEVELS, t))
        return {"go": T.prepare(site), "hist": hist, "out": [hist, t], "keep": x}
    fmt, batch = case["fmt"], case["batch"]
    bits = BITS[fmt]
    calls = _inputs(case, seed)
    need = 0
    for c in calls:
        n = [a["n"] for a in c["mats"]]
        if c["kind"] == "mlp":
            need = max(need, T.teal_workspace_bytes_mlp(c["m"], n[0], n[2]))
            pitches = [c["mats"][0]["pitch"], c["mats"][2]["pitch"]] if fmt == "bf16" else [0, 0]
            status, c["shape"] = T.teal_mlp_plan(bits, c["m"], n[0], n[2], *pitches)
            T.check(status)
        elif c["kind"] == "batch":
            need = max(need, T.teal_workspace_bytes_batch(c["m"], sum(n), batch))
        else:
            need = max(need, T.teal_workspace_bytes(c["m"], sum(n)))
        c["out"] = [torch.empty((batch, k) if c["kind"] == "batch" else k, dtype=torch.float32,
                                device="cuda") for k in n]
    ws = _workspace(need)                        # one workspace, the calls run in order

    def layers():
        for c in calls:
            T.check(_issue(c, fmt, batch, ws))
    return {"go": T.prepare(layers), "out": [c["out"] for c in calls], "keep": (calls, ws)}


def run(state):
    if "hist" in state:
        state["hist"].zero_()                    # a new site begins with empty counts
    T.check(state["go"]())
    return state["out"]


# ---- the same in 64 bits, by plain torch -------------------------------------------------------


def _product(x, kept, mat, fmt):
    """Rows of x (64 bits) times the matrix, dropped channels left out."""
    m, n = mat["W"].shape[0], mat["n"]
    y = torch.zeros((x.shape[0], n), dtype=torch.float64, device="cuda")
    part = max(GROUP, (1 << 26) // n // GROUP * GROUP)
    for i in range(0, m, part):
        rows = dict(mat, W=mat["W"][i:i + part])
        if fmt == "w4":
            rows["scale"] = mat["scale"][i // GROUP:(i + part) // GROUP]
        y += (x[:, i:i + part] * kept[i:i + part]) @ _dense(rows, fmt)
    return y


def exact(case, seed):
    if case["op"] == "calibrate":
        mag = _sample(case, seed).view(torch.int16).to(torch.int32) & 0x7FFF
        hist = torch.bincount(mag.view(-1), minlength=T.TEAL_HIST_BINS)
        below = torch.cumsum(hist, 0)
        bins = [int((below < math.ceil(p * mag.numel() - 1e-9)).sum()) for p in LEVELS]
        t = torch.tensor(bins, dtype=torch.int16, device="cuda").view(torch.float16).float()
        return [hist, t]
    fmt, batch, got = case["fmt"], case["batch"], []
    for c in _inputs(case, seed):
        kind, mats, t = c["kind"], c["mats"], c["t"]
        if kind == "batch":
            x = c["x"].double()
            size = x.abs().sum(0)
            got.append([_product(x, size > batch * t[0], a, fmt) for a in mats])
            continue
        if kind == "norm":
            x = _normalised(c["h"], c["gamma"])
        elif kind == "swiglu":
            x = _gated(c["gate"], c["up"])
        else:
            x = c["x"]

        def y(v, k):
            kept = v.float().abs() > torch.tensor(t[k], dtype=torch.float32, device="cuda")
            return _product(v.double()[None], kept, mats[k], fmt)[0]
        if kind == "mlp":
            gate, up = y(x, 0), y(x, 1)
            got.append([gate, up, y(_gated(gate.float(), up.float()), 2)])
        else:
            got.append([y(x, k) for k in range(len(mats))])
    return got
