"""Workloads of the affinity path whose speed is watched, each through the public entry points.

A calibration run streams tokens through `dtp_affinity_accumulate*` layer by layer, folds
each layer's weights once (`dtp_layer_set_weights`), forms the down edge's weight factor
once per layer (`dtp_down_weights`), optimises the layout (`dtp_coordinate_ascent`) and
permutes the weights (`dtp_apply_layout`).  A case is one such call, or the two calls that
always go together, with everything a program holds at that point made by `prepare`.

Kinds of case and their fields:
  affinity  dtype, d, I, H, G, dh, T, score ("fo", "down": FO with the down-edge statistic,
            "add"), load (the weights are folded in the same pass)
  down      the down edge's weight factor and S_down at d, I, H, G, dh
  ascent    N layers of G x I, L devices, down (with S_down between the layers)
  apply     the seven weight matrices of a layer moved to a layout over L devices
"""
import math

import torch

from paper_2609_13846_amd import dtp

EPS = 1e-6
_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
_DTP = {"bf16": dtp.DTP_BF16, "f32": dtp.DTP_F32}

QWEN = dict(dtype="bf16", d=1024, I=3072, H=16, G=8, dh=128)
DANUBE = dict(dtype="bf16", d=1536, I=4096, H=16, G=8, dh=96)
CLASS8B = dict(dtype="bf16", d=4096, I=14336, H=32, G=8, dh=128)


def _affinity(name, shape, T, score, load=False):
    return dict(name=name, kind="affinity", T=T, score=score, load=load, **shape)


def listed():
    return [
        # The smallest layer of the workload list, in fp32: latency and launches.
        _affinity("tiny-f32", dict(dtype="f32", d=64, I=128, H=8, G=4, dh=16), 512, "fo"),
        # The reference-precision path on a small model's layer, weights folded and streamed.
        _affinity("block-f32", dict(dtype="f32", d=512, I=1536, H=8, G=4, dh=64), 2048, "down", True),
        # The headline calibration: one Qwen3-0.6B-shaped layer, 64 x 1024 tokens in one call.
        _affinity("qwen-65536", QWEN, 65536, "fo"),
        # A quick look at a layer with a few documents, ragged, with the simpler ADD score.
        _affinity("qwen-1000-add", QWEN, 1000, "add"),
        # One chunk of the full-model stream (16,384 tokens) with the down edge, 96-wide heads.
        _affinity("danube-16384-down", DANUBE, 16384, "down"),
        # The same chunk of an 8B-class layer.
        _affinity("8b-16384-down", CLASS8B, 16384, "down"),
        # Widths off the usual powers of two: 80-wide heads, d of 65 x 16, ragged neurons, tokens.
        _affinity("odd-5000", dict(dtype="bf16", d=1040, I=2810, H=12, G=4, dh=80), 5000, "fo"),
        # A new 8B-class layer: its weights folded, then its first short batch of tokens.
        _affinity("8b-load-256", CLASS8B, 256, "fo", True),
        # The weight factor of an 8B-class layer's down edge, and S_down from it.
        dict(name="8b-down-weights", kind="down", **CLASS8B),
        # The layout of one layer over two devices, as every calibration step ends.
        dict(name="ascent-1x3072", kind="ascent", N=1, G=8, I=3072, L=2, down=False),
        # The layout of a whole 28-layer model over four devices, chained by the down edges.
        dict(name="ascent-28x3072", kind="ascent", N=28, G=8, I=3072, L=4, down=True),
        # The chosen layout realised on an 8B-class layer's weights.
        dict(name="8b-apply", kind="apply", L=4, **CLASS8B),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _layer_shape(rng, dtype, d_max, I_max):
    """A layer of the widths that decoder layers come in: heads of 32 to 128, d and I odd
    multiples of 16 and any integer among them."""
    dh = rng.choice([32, 48, 64, 80, 96, 128])
    G = rng.choice([1, 2, 4, 8])
    hpg = rng.choice([1, 2, 3, 4])
    while G * hpg * dh > 4096:
        G //= 2
    d = 16 * _log_int(rng, 8, d_max // 16)
    if rng.random() < 0.5:
        d = max(128, d // 128 * 128)
    I = _log_int(rng, 256, I_max)
    if rng.random() < 0.5:
        I = max(256, I // 128 * 128)
    return dict(dtype=dtype, d=d, I=I, H=G * hpg, G=G, dh=dh)


def draw(rng):
    kind = rng.choice(["bf16", "bf16", "bf16", "bf16", "f32", "down", "ascent", "apply"])
    if kind in ("bf16", "f32"):
        big = kind == "bf16"
        s = _layer_shape(rng, kind, 4096 if big else 768, 14336 if big else 2048)
        T = _log_int(rng, 64, 65536 if big else 4096)
        per_token = 4.0 * s["I"] * (s["H"] * s["dh"] + s["d"])
        T = max(64, min(T, int((6e12 if big else 1.2e10) / per_token)))
        return dict(kind="affinity", T=T, score=rng.choice(["fo", "down", "add"]),
                    load=rng.random() < 0.25, **s)
    if kind in ("down", "apply"):
        s = _layer_shape(rng, "bf16", 4096, 14336)
        s["I"] = s["I"] // 8 * 8
        if kind == "down":
            return dict(kind="down", **s)
        return dict(kind="apply", L=rng.choice([l for l in (1, 2, 4) if s["G"] % l == 0]), **s)
    G, L = rng.choice([(2, 2), (4, 2), (4, 4), (8, 2), (8, 4), (8, 8)])
    N = _log_int(rng, 1, 28)
    I = max(256, _log_int(rng, 256, min(14336, 90000 // N)) // L * L)
    return dict(kind="ascent", N=N, G=G, I=I, L=L, down=N > 1 and rng.random() < 0.7)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)


def _layer_weights(c, gen):
    dt, d, I, HD = _TORCH[c["dtype"]], c["d"], c["I"], c["H"] * c["dh"]
    return {"w_o": (0.02 * _normal(gen, d, HD)).to(dt), "gamma": (1 + 0.1 * _normal(gen, d)).to(dt),
            "w_gate": (0.02 * _normal(gen, I, d)).to(dt), "w_up": (0.02 * _normal(gen, I, d)).to(dt),
            "w_down": (0.02 * _normal(gen, d, I)).to(dt)}


def _tokens(c, w, gen):
    """The residual entering the FFN pre-norm (a few channels of massive activations, plus the
    attention output), the per-head attention outputs, and the next layer's residual."""
    dt, d, T, HD = _TORCH[c["dtype"]], c["d"], c["T"], c["H"] * c["dh"]
    x = _normal(gen, T, d)
    x[:, torch.randperm(d, generator=gen, device="cuda")[:4]] *= 50.0
    attn = _normal(gen, T, HD).to(dt)
    for t in range(0, T, 8192):
        x[t:t + 8192] += attn[t:t + 8192].float() @ w["w_o"].float().t()
    out = {"x": x.to(dt), "attn": attn.view(T, c["H"], c["dh"]), "x_next": None}
    if c["score"] == "down":
        x[:, torch.randperm(d, generator=gen, device="cuda")[:4]] *= 50.0
        out["x_next"] = x.to(dt)
    return out


def _down_inputs(c, gen):
    dt, d, I, HD, GD = _TORCH[c["dtype"]], c["d"], c["I"], c["H"] * c["dh"], c["G"] * c["dh"]
    return {"w_q": (0.02 * _normal(gen, HD, d)).to(dt), "w_k": (0.02 * _normal(gen, GD, d)).to(dt),
            "w_v": (0.02 * _normal(gen, GD, d)).to(dt), "gamma": (1 + 0.1 * _normal(gen, d)).to(dt),
            "w_down": (0.02 * _normal(gen, d, I)).to(dt), "s_down": 100 * torch.exp(_normal(gen, I))}


def _ascent_inputs(c, gen):
    """Affinities as the calibration leaves them: a scale per neuron (its write and activity)
    times a milder preference of each neuron among the groups."""
    N, G, I = c["N"], c["G"], c["I"]
    up = torch.exp(0.7 * _normal(gen, N, 1, I) + 0.3 * _normal(gen, N, G, I))
    down = torch.exp(0.7 * _normal(gen, N - 1, I, 1) + 0.1 * _normal(gen, N - 1, I, G)) if c["down"] else None
    return up.contiguous(), down


class _Layer:
    """A layer handle that is destroyed with the state that holds it."""

    def __init__(self, c):
        self.handle = dtp.dtp_layer_create(c["d"], c["I"], c["H"], c["G"], c["dh"], EPS, _DTP[c["dtype"]])

    def __del__(self):
        dtp.dtp_layer_destroy(self.handle)


def prepare(case, seed):
    c, gen = case, _generator(seed)
    s = {"case": c}
    if c["kind"] == "affinity":
        s["w"] = w = _layer_weights(c, gen)
        s["t"] = _tokens(c, w, gen)
        s["layer"] = _Layer(c)
        if not c["load"]:
            _load(s)
        s["A"] = torch.zeros(c["G"], c["I"], dtype=torch.float32, device="cuda")
        s["s_down"] = torch.zeros(c["I"], dtype=torch.float32, device="cuda")
    elif c["kind"] == "down":
        s["w"] = _down_inputs(c, gen)
        s["B"] = torch.empty(c["G"], c["I"], dtype=torch.float32, device="cuda")
        s["A_down"] = torch.empty(c["I"], c["G"], dtype=torch.float32, device="cuda")
    elif c["kind"] == "ascent":
        s["up"], s["down"] = _ascent_inputs(c, gen)
    else:
        w = _layer_weights(c, gen)
        w.update({k: v for k, v in _down_inputs(c, gen).items() if k in ("w_q", "w_k", "w_v")})
        s["src"] = {k: w[k] for k in dtp.WEIGHT_ORDER}
        s["dst"] = {k: torch.empty_like(v) for k, v in s["src"].items()}
        h, nu = dtp.dtp_random_layout(1, c["G"], c["I"], c["L"], int(seed))
        s["h"], s["nu"] = h[0], nu[0]
    return s


def _load(s):
    w = s["w"]
    dtp.dtp_layer_set_weights(s["layer"].handle, w["w_o"], w["gamma"], w["w_gate"], w["w_up"], w["w_down"])


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "affinity":
        t, layer, A = s["t"], s["layer"].handle, s["A"]
        if c["load"]:
            _load(s)
        A.zero_()
        if c["score"] == "down":
            s["s_down"].zero_()
            dtp.dtp_affinity_accumulate_down(layer, t["x"], t["attn"], t["x_next"], EPS, c["T"], A, s["s_down"])
            return {"A": A, "s_down": s["s_down"]}
        if c["score"] == "add":
            dtp.dtp_affinity_accumulate_add(layer, t["x"], t["attn"], c["T"], A)
        else:
            dtp.dtp_affinity_accumulate(layer, t["x"], t["attn"], c["T"], A)
        return {"A": A}
    if c["kind"] == "down":
        w = s["w"]
        dtp.dtp_down_weights(c["d"], c["I"], c["H"], c["G"], c["dh"], _DTP[c["dtype"]], w["w_q"], w["w_k"],
                             w["w_v"], w["gamma"], w["w_down"], s["B"])
        dtp.dtp_down_affinity(c["I"], c["G"], w["s_down"], s["B"], s["A_down"])
        return {"B": s["B"], "A_down": s["A_down"]}
    if c["kind"] == "ascent":
        return dtp.dtp_coordinate_ascent(c["N"], c["G"], c["I"], c["L"], s["up"], s["down"])
    dtp.dtp_apply_layout(c["d"], c["I"], c["H"], c["G"], c["dh"], _DTP[c["dtype"]], c["L"], s["h"], s["nu"],
                         s["src"], s["dst"])
    return s["dst"]


def work(case):
    c = case
    if c["kind"] == "ascent":  # every code of every matrix is read and added once
        entries = c["N"] * c["G"] * c["I"] + (c["N"] - 1) * c["I"] * c["G"] * c["down"]
        return {"bytes": 4.0 * entries + 4.0 * c["N"] * (c["G"] + c["I"]), "flops": 2.0 * entries}
    es = 2 if c["dtype"] == "bf16" else 4
    d, I, HD, GD = c["d"], c["I"], c["H"] * c["dh"], c["G"] * c["dh"]
    if c["kind"] == "down":
        return {"bytes": es * ((HD + 2.0 * GD) * d + d + d * I) + 4.0 * (I + 2 * c["G"] * I),
                "flops": 2.0 * (HD + 2 * GD) * d * I}
    if c["kind"] == "apply":
        return {"bytes": 2.0 * es * (2 * HD * d + 2 * GD * d + 3 * d * I), "flops": 0.0}
    T = c["T"]
    tokens = es * T * (d + HD + (d if c["score"] == "down" else 0))
    weights = es * (d * HD + d + 3.0 * d * I) if c["load"] else es * 2.0 * I * (d + HD) + 4 * I
    flops = 4.0 * I * (HD + d) * T
    if c["load"]:
        flops += 4.0 * HD * d * I + 2.0 * d * I
    return {"bytes": tokens + weights + 4.0 * c["G"] * I, "flops": flops}


def tolerance(case):
    if case["kind"] in ("ascent", "apply"):
        return "exact"  # integers, and weights moved as they are
    # About four times the distance from 64-bit results that was measured.
    if case["dtype"] == "f32":
        return {"rel": 2e-6}  # 1.2e-7: fp32 products and sums, fp64 split sums
    if case["kind"] == "down" or case["score"] == "add":
        return {"rel": 2.5e-3}  # 2e-4 to 6e-4: one bf16 rounding per operand, no cancellation
    return {"rel": 1e-2}  # 1e-3 to 3e-3: the folded weights' bf16 rounding through g, u and Delta


def exact(case, seed):
    c = case
    if c["kind"] in ("ascent", "apply"):
        return None
    gen = _generator(seed)
    if c["kind"] == "down":
        w = {k: v.double() for k, v in _down_inputs(c, gen).items()}
        scaled = w["gamma"][:, None] * w["w_down"]
        B = torch.zeros(c["G"], c["I"], dtype=torch.float64, device="cuda")
        for name in ("w_q", "w_k", "w_v"):
            B += ((w[name] @ scaled) ** 2).view(c["G"], -1, c["I"]).sum(1)
        return {"B": B, "A_down": (w["s_down"][None, :] * B).t().contiguous()}
    wb = _layer_weights(c, gen)
    t = _tokens(c, wb, gen)
    w = {k: v.double() for k, v in wb.items()}
    H, G, dh, I = c["H"], c["G"], c["dh"], c["I"]
    gate, up = (w["w_gate"] * w["gamma"]).t().contiguous(), (w["w_up"] * w["gamma"]).t().contiguous()
    w_oT = w["w_o"].t().contiguous()
    f_gate, f_up = w_oT @ gate, w_oT @ up  # [H * dh, I]
    A = torch.zeros(G, I, dtype=torch.float64, device="cuda")
    s_down = torch.zeros(I, dtype=torch.float64, device="cuda")
    for t0 in range(0, c["T"], 4096):
        x, a = t["x"][t0:t0 + 4096].double(), t["attn"][t0:t0 + 4096].double()
        r = torch.sqrt((x * x).mean(1, keepdim=True) + EPS)
        g, u = (x / r) @ gate, (x / r) @ up
        sig = torch.sigmoid(g)
        c1, c2 = sig * (1 + g * (1 - sig)) * u / r, g * sig / r
        if c["score"] == "down":
            xn = t["x_next"][t0:t0 + 4096].double()
            s_down += ((g * sig * u) ** 2 / ((xn * xn).mean(1, keepdim=True) + EPS)).sum(0)
        for h in range(H):
            ah = a[:, h].contiguous()
            pg, pu = ah @ f_gate[h * dh:(h + 1) * dh], ah @ f_up[h * dh:(h + 1) * dh]
            if c["score"] == "add":
                A[h // (H // G)] += ((pg / r) ** 2 + (pu / r) ** 2).sum(0)
            else:
                A[h // (H // G)] += ((c1 * pg + c2 * pu) ** 2).sum(0)
    if c["score"] != "add":
        A *= (w["w_down"] ** 2).sum(0)
    return {"A": A, "s_down": s_down} if c["score"] == "down" else {"A": A}
