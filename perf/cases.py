"""Performance cases of the FP8 MoE expert layer: the calls a training or serving program makes
through the public entry points (`ExpertLayerFP8` and the `ff8` operators), over their range of
sizes, scale formats, paddings and routings.

A case is a dict of plain values.  Kinds:
  step      one training step of a layer: weight cast, forward, backward (all gradients out)
  forward   the forward alone, with the weights quantized beforehand
  cast      1x128 quantization of an activation and, with transpose, its scaling-aware transpose
  dispatch  permute + pad + quantize the tokens, and the weighted combine of an expert output
  wgrad     one grouped weight-gradient product of transposed FP8 operands

`exact` restates the recipe in float64 torch: power-of-two scales 2^T with the smallest T that
keeps a tile's largest magnitude at or below 448 * 2^T, e4m3 round-to-nearest-even, bf16 at the
two GEMM outputs of each direction.
"""

import math

import torch

from paper_2511_02302_amd import ff8
from paper_2511_02302_amd.layer import ExpertLayerFP8

_OPTS = {"align": 128, "scale_fmt": "f32", "fp8_checkpoint": False, "router_grad": False, "routing": "iid"}


def _layer(kind, T, H, E, k, I, **opts):
    return {"kind": kind, "T": T, "H": H, "E": E, "k": k, "I": I, **_OPTS, **opts}


def listed():
    return [
        # the layer of the parity tests and of a unit-size model: every kernel runs for a few
        # microseconds, so launches and latency count
        {"name": "step_tiny", **_layer("step", 1024, 256, 8, 2, 512)},
        # a training step of one expert-parallel rank at the benchmark's size
        {"name": "step_share", **_layer("step", 16384, 7168, 32, 8, 2048)},
        # the skewed routing of an untrained or collapsed router, with the options of a
        # memory-bound run: the FP8 checkpoint of A and the router's gradient
        {"name": "step_skew", **_layer("step", 8192, 7168, 32, 8, 2048, routing="zipf", fp8_checkpoint=True,
                                       router_grad=True)},
        # a pipeline micro-batch: an eighth of the tokens, the paper's 16-row padding, byte scales
        {"name": "step_micro", **_layer("step", 2048, 7168, 32, 8, 2048, align=16, scale_fmt="e8m0")},
        # many narrow experts whose widths are odd multiples of the tile
        {"name": "step_fine", **_layer("step", 4096, 2048, 64, 6, 1408, router_grad=True)},
        # evaluation or prefill of a ragged batch
        {"name": "forward_prefill", **_layer("forward", 3001, 7168, 32, 8, 2048)},
        # a decoding batch: a few rows per expert, the weights are the traffic
        {"name": "forward_decode", **_layer("forward", 64, 7168, 32, 8, 2048, align=16)},
        # a handful of sequences on the narrow experts
        {"name": "forward_few", **_layer("forward", 7, 2048, 64, 6, 1408, align=16)},
        # an activation with outliers, cast at the layer's entry and turned for the weight gradient
        {"name": "cast_activation", "kind": "cast", "rows": 32768, "cols": 7168, "scale_fmt": "f32", "transpose": True},
        # a ragged small activation, cast only
        {"name": "cast_ragged", "kind": "cast", "rows": 1027, "cols": 1408, "scale_fmt": "e8m0", "transpose": False},
        # dispatch and combine around experts that another library computes
        {"name": "dispatch_combine", "kind": "dispatch", "T": 5000, "H": 4096, "E": 64, "k": 4, "align": 16,
         "scale_fmt": "f32", "routing": "iid"},
        # the weight gradient of one linear layer of the experts
        {"name": "wgrad_mid", "kind": "wgrad", "T": 4096, "E": 16, "k": 2, "N": 2816, "K": 2048, "align": 128,
         "scale_fmt": "f32", "routing": "iid"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "forward", "forward", "forward", "cast", "dispatch", "wgrad"])
    fmt = rng.choice(["f32", "f32", "e8m0"])
    align = rng.choice([16, 128, 128])
    routing = rng.choice(["iid", "iid", "zipf"])
    if kind == "cast":
        transpose = rng.random() < 0.5
        rows = _log(rng, 1, 32768)
        if transpose:
            rows = -(-rows // 128) * 128
        return {"kind": "cast", "rows": rows, "cols": 128 * _log(rng, 1, 56), "scale_fmt": fmt, "transpose": transpose}
    E = _log(rng, 4, 64)
    k = rng.randint(1, min(8, E))
    step = 512 if fmt == "e8m0" else 128  # the layer's widths with byte scales are multiples of 512
    H, I = step * _log(rng, 1, 7168 // step), step * _log(rng, 1, 2048 // step)
    if kind == "dispatch":
        return {"kind": kind, "T": _log(rng, 1, 16384), "H": H, "E": E, "k": k, "align": align, "scale_fmt": fmt,
                "routing": routing}
    if kind == "wgrad":
        return {"kind": kind, "T": _log(rng, 64, 16384), "E": E, "k": k, "N": 2 * I, "K": H, "align": align,
                "scale_fmt": fmt, "routing": routing}
    E = min(E, 32) if H * I > 7168 * 1024 else E  # no more weights than the largest listed layer holds
    k = min(k, E)
    return _layer(kind, _log(rng, 1, 16384), H, E, k, I, align=align, scale_fmt=fmt, routing=routing,
                  fp8_checkpoint=rng.random() < 0.3, router_grad=kind == "step" and rng.random() < 0.3)


# ---- inputs ----

def _randn(shape, std, seed):
    """N(0, std^2) in bf16."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(torch.bfloat16)


def _routing(c, seed):
    """Top-k experts of random logits (skewed: expert popularity ~ rank^-1.2) and their softmax weights."""
    g = torch.Generator()
    g.manual_seed(seed)
    logits = torch.randn((c["T"], c["E"]), generator=g)
    if c["routing"] == "zipf":
        p = (torch.randperm(c["E"], generator=g).float() + 1.0) ** -1.2
        logits = torch.log(p / p.sum()) + 0.4 * logits
    idx = torch.topk(logits, c["k"], dim=1).indices
    probs = torch.gather(torch.softmax(logits, dim=1), 1, idx)
    return idx.to(torch.int32).contiguous().cuda(), probs.contiguous().cuda()


def _layer_inputs(c, seed):
    T, H, E, I = c["T"], c["H"], c["E"], c["I"]
    idx, probs = _routing(c, 10 * seed + 1)
    x = _randn((T, H), 1.0, 10 * seed + 2)
    w1 = _randn((E, 2 * I, H), 0.02, 10 * seed + 3)
    w2 = _randn((E, H, I), 0.02, 10 * seed + 4)
    dy = _randn((T, H), 1.0, 10 * seed + 5) if c["kind"] == "step" else None
    return x, idx, probs, w1, w2, dy


def _activation(c, seed):
    """N(0, 1) with one entry in a thousand a hundred times larger."""
    shape = (c["rows"], c["cols"])
    x = _randn(shape, 1.0, 10 * seed + 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(10 * seed + 2)
    return torch.where(torch.rand(shape, generator=g, device="cuda") < 1e-3, x * 100.0, x)


def _sdt(c):
    return torch.uint8 if c["scale_fmt"] == "e8m0" else torch.float32


def _m_cap(c):
    return ff8.ff8_rows_bound_aligned(c["T"], c["k"], c["E"], c["align"])


def _maps(c):
    """Routing maps of one batch and the permute's workspace."""
    T, k, E = c["T"], c["k"], c["E"]
    return {"row_map": torch.empty((T, k), dtype=torch.int32, device="cuda"),
            "offsets": torch.empty((E + 1,), dtype=torch.int32, device="cuda"),
            "src_row": torch.empty((_m_cap(c),), dtype=torch.int32, device="cuda"),
            "ws": torch.empty((max(1, ff8.ff8_permute_workspace_bytes(T, k, E)),), dtype=torch.uint8, device="cuda")}


def _permute(c, x, idx, m, q, s):
    ff8.ff8_permute_quant(x, None, c["k"], c["E"], idx, False, m["row_map"], m["offsets"], m["src_row"], q, s, m["ws"],
                          align=None if c["align"] == 128 else c["align"])


def _row_pair(rows, cols, sdt):
    return (torch.zeros((rows, cols), dtype=torch.uint8, device="cuda"),
            torch.full((rows, cols // 128), 1, dtype=sdt, device="cuda"))


def _col_pair(rows, cols, sdt):
    return (torch.zeros((rows // 128, cols, 128), dtype=torch.uint8, device="cuda"),
            torch.full((rows // 128, cols), 1, dtype=sdt, device="cuda"))


def prepare(case, seed):
    c = case
    kind = c["kind"]
    if kind in ("step", "forward"):
        x, idx, probs, w1, w2, dy = _layer_inputs(c, seed)
        layer = ExpertLayerFP8(c["T"], c["H"], c["E"], c["k"], c["I"], fp8_checkpoint=c["fp8_checkpoint"],
                               router_grad=c["router_grad"], align=c["align"], scale_fmt=c["scale_fmt"])
        state = {"case": c, "layer": layer, "x": x, "idx": idx, "probs": probs}
        if kind == "step":
            state.update(w1=w1, w2=w2, dy=dy)
        else:
            layer.quantize_weights(w1, w2)
        return state
    if kind == "cast":
        state = {"case": c, "x": _activation(c, seed), "row": _row_pair(c["rows"], c["cols"], _sdt(c))}
        if c["transpose"]:
            state["col"] = _col_pair(c["rows"], c["cols"], _sdt(c))
        return state
    M = _m_cap(c)
    idx, probs = _routing(c, 10 * seed + 1)
    m = _maps(c)
    if kind == "dispatch":
        return {"case": c, "x": _randn((c["T"], c["H"]), 1.0, 10 * seed + 2), "idx": idx, "probs": probs, "maps": m,
                "row": _row_pair(M, c["H"], _sdt(c)), "out": _randn((M, c["H"]), 1.0, 10 * seed + 3),
                "y": torch.empty((c["T"], c["H"]), dtype=torch.bfloat16, device="cuda")}
    # wgrad: gradient [M, N] and activation [M, K] rows of the groups, quantized and transposed
    cols = {}
    for name, width, sub in (("g", c["N"], 2), ("x", c["K"], 3)):
        q, s = _row_pair(M, width, _sdt(c))
        _permute(c, _randn((c["T"], width), 1.0, 10 * seed + sub), idx, m, q, s)
        cols[name] = _col_pair(M, width, _sdt(c))
        ff8.ff8_scaling_aware_transpose(q, s, *cols[name], m["offsets"], c["E"])
    return {"case": c, "offsets": m["offsets"], "g": cols["g"], "x": cols["x"],
            "dw": torch.empty((c["E"], c["N"], c["K"]), dtype=torch.float32, device="cuda")}


# ---- the measured pass ----

def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "step":
        layer = state["layer"]
        dx, dw1, dw2 = layer.step(state["x"], state["idx"], state["probs"], state["dy"], state["w1"], state["w2"])
        out = {"y": layer.own["y"], "dx": dx, "dw1": dw1, "dw2": dw2}
        if c["router_grad"]:
            out["dprobs"] = layer.own["dprobs"]
        return out
    if kind == "forward":
        return {"y": state["layer"].forward(state["x"], state["idx"], state["probs"])}
    if kind == "cast":
        q, s = state["row"]
        ff8.ff8_quant_rowwise(state["x"], q, s)
        if not c["transpose"]:
            return {"q": q, "s": s}
        qT, sT = state["col"]
        ff8.ff8_scaling_aware_transpose(q, s, qT, sT)
        return {"q": q, "s": s, "qT": qT, "sT": sT}
    if kind == "dispatch":
        m = state["maps"]
        q, s = state["row"]
        _permute(c, state["x"], state["idx"], m, q, s)
        ff8.ff8_unpermute(state["out"], m["row_map"], state["probs"], state["y"])
        return {"y": state["y"], "q": q, "s": s, "row_map": m["row_map"], "offsets": m["offsets"]}
    ff8.ff8_grouped_gemm_wgrad(*state["g"], *state["x"], state["offsets"], state["dw"])
    return {"dw": state["dw"]}


def work(case):
    c = case
    kind = c["kind"]
    sb = 1 if c["scale_fmt"] == "e8m0" else 4
    if kind == "cast":
        n = c["rows"] * c["cols"]
        outs = 2 if c["transpose"] else 1
        return {"bytes": 2 * n + outs * (n + sb * n // 128), "flops": 0}
    T, E, k = c["T"], c["E"], c["k"]
    M = T * k
    if kind == "dispatch":
        H = c["H"]
        return {"bytes": 2 * T * H + M * H + sb * M * H // 128 + 2 * M * H + 2 * T * H + 12 * M, "flops": 2 * M * H}
    if kind == "wgrad":
        N, K = c["N"], c["K"]
        return {"bytes": M * (N + K) + sb * M * (N + K) // 128 + 4 * E * N * K, "flops": 2 * M * N * K}
    H, I = c["H"], c["I"]
    if kind == "forward":
        hit = min(E, E * (1 - (1 - k / E) ** T))  # experts that get a token, for even routing
        w = hit * 3 * H * I
        return {"bytes": int(w + w * sb / 16384) + 4 * T * H + 8 * M, "flops": 6 * M * H * I}
    return {"bytes": 8 * T * H + E * 3 * H * I * (2 + 4) + 8 * M + (4 * M if c["router_grad"] else 0),
            "flops": 18 * M * H * I}


def tolerance(case):
    kind = case["kind"]
    if kind == "cast":
        return "exact"
    if kind == "dispatch":
        # bytes and maps are the same; y is a float32 sum of at most 8 terms, rounded once to bf16
        # (1.7e-3 from float64)
        return {"rel": 7e-3}
    if kind == "wgrad":
        # float32 accumulation on the matrix core: 1.5e-5 from float64
        return {"rel": 1e-4}
    # bf16 outputs and FP8 codes that another rounding of the bf16 stage before them moves: 2.6e-3
    # from float64; with a handful of tokens one moved code weighs more (4.7e-3)
    return {"rel": 1e-2 if case["T"] >= 256 else 2e-2}


# ---- float64 restatement ----

def _pow2(t):
    return torch.ldexp(torch.ones((), dtype=torch.float64, device=t.device), t)


def _e4m3(v):
    """Nearest-even e4m3 codes of float64 values in [-448, 448]."""
    return v.to(torch.float32).to(torch.float8_e4m3fn)


def _quant(x, block=False):
    """x [rows, cols] float64 -> (codes, exponents T) of 1x128 tiles or 128x128 blocks."""
    rows, cols = x.shape
    r = 128 if block else 1
    t = x.view(rows // r, r, cols // 128, 128)
    amax = t.abs().amax(dim=(1, 3))
    m, e = torch.frexp(amax)  # 448 = 0.875 * 2^9
    T = torch.where(m <= 0.875, e - 9, e - 8).to(torch.int32)
    T = torch.where(amax > 0, T.clamp(min=-126), torch.full_like(T, -126))
    q = _e4m3(t * _pow2(-T)[:, None, :, None])
    return q.view(rows, cols), T


def _dequant(q, T, block=False):
    rows, cols = q.shape
    r = 128 if block else 1
    return (q.to(torch.float64).view(rows // r, r, cols // 128, 128) * _pow2(T)[:, None, :, None]).view(rows, cols)


def _cast(x):
    return _dequant(*_quant(x))


def _bf16(x):
    return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _stored(T, c):
    return (T + 127).to(torch.uint8) if c["scale_fmt"] == "e8m0" else _pow2(T)


def _groups(c, idx):
    """Padded groups: offsets, and per expert its tokens and slots in ascending token order."""
    tok, slot, off = [], [], [0]
    for e in range(c["E"]):
        t, j = torch.nonzero(idx == e, as_tuple=True)
        tok.append(t)
        slot.append(j)
        off.append(off[-1] + -(-t.numel() // c["align"]) * c["align"])
    return tok, slot, off


def _grouped(parts, off, width):
    """Per-expert (codes, exponents) laid out with their padding (zero codes at 2^-126)."""
    rows = -(-off[-1] // 128) * 128
    q = torch.zeros((rows, width), dtype=torch.float8_e4m3fn, device="cuda")
    T = torch.full((rows, width // 128), -126, dtype=torch.int32, device="cuda")
    for e, (pq, pT) in enumerate(parts):
        q.view(torch.uint8)[off[e]:off[e] + pq.shape[0]] = pq.view(torch.uint8)
        T[off[e]:off[e] + pT.shape[0]] = pT
    return q, T


class _Columns:
    """Scaling-aware transpose of a grouped tensor, read back by rows: codes at their block's largest scale."""

    def __init__(self, parts, off, width):
        self.q, self.T = _grouped(parts, off, width)
        self.Tmax = self.T.view(-1, 128, width // 128).amax(dim=1)

    def rows(self, r0, r1):
        Tm = self.Tmax[torch.arange(r0, r1, device="cuda") // 128]
        v = self.q[r0:r1].to(torch.float64).view(r1 - r0, -1, 128)
        v = _e4m3(v * _pow2(self.T[r0:r1] - Tm)[:, :, None]).to(torch.float64) * _pow2(Tm)[:, :, None]
        return v.view(r1 - r0, -1)


def _wgrad(g, x, off, E, N, K):
    dw = torch.zeros((E, N, K), dtype=torch.float64, device="cuda")
    for e in range(E):
        if off[e + 1] > off[e]:
            dw[e] = g.rows(off[e], off[e + 1]).t().contiguous() @ x.rows(off[e], off[e + 1])
    return dw


def _exact_layer(c, seed):
    x, idx, probs, w1, w2, dy = _layer_inputs(c, seed)
    T, H, E, I = c["T"], c["H"], c["E"], c["I"]
    f64 = torch.float64
    tok, slot, off = _groups(c, idx)
    y = torch.zeros((T, H), dtype=f64, device="cuda")
    dx, dprobs = torch.zeros_like(y), torch.zeros((T, c["k"]), dtype=f64, device="cuda")
    px, ph, pdy, pda = [], [], [], []
    for e in range(E):
        t, j = tok[e], slot[e]
        W1 = _dequant(*_quant(w1[e].to(f64), True), True)
        W2 = _dequant(*_quant(w2[e].to(f64), True), True)
        p = probs[t, j][:, None]
        xq = _quant(x[t].to(f64))
        a = _bf16(_dequant(*xq) @ W1.t().contiguous())
        g, u = a[:, :I], a[:, I:]
        hq = _quant(g * torch.sigmoid(g) * u)
        yp = _bf16(_dequant(*hq) @ W2.t().contiguous())
        y.index_add_(0, t, p.to(f64) * yp)
        if dy is None:
            continue
        dprobs[t, j] = (dy[t].to(f64) * yp).sum(dim=1)
        dyq = _quant((p * dy[t].to(torch.float32)).to(f64))
        dh = _bf16(_dequant(*dyq) @ W2)
        if c["fp8_checkpoint"]:
            a = _cast(a.contiguous())
            g, u = a[:, :I], a[:, I:]
        sg = torch.sigmoid(g)
        daq = _quant(torch.cat([dh * u * sg * (1 + g * (1 - sg)), dh * g * sg], dim=1))
        dx.index_add_(0, t, _bf16(_dequant(*daq) @ W1))
        px.append(xq)
        ph.append(hq)
        pdy.append(dyq)
        pda.append(daq)
    if dy is None:
        return {"y": y}
    out = {"y": y, "dx": dx,
           "dw1": _wgrad(_Columns(pda, off, 2 * I), _Columns(px, off, H), off, E, 2 * I, H),
           "dw2": _wgrad(_Columns(pdy, off, H), _Columns(ph, off, I), off, E, H, I)}
    if c["router_grad"]:
        out["dprobs"] = dprobs
    return out


def exact(case, seed):
    c = case
    if c["kind"] in ("step", "forward"):
        return _exact_layer(c, seed)
    if c["kind"] == "cast":
        q, T = _quant(_activation(c, seed).to(torch.float64))
        out = {"q": q.view(torch.uint8), "s": _stored(T, c)}
        if c["transpose"]:
            cols = _Columns([(q, T)], [0, c["rows"]], c["cols"])
            v = torch.cat([_e4m3(cols.q[r:r + 128].to(torch.float64).view(128, -1, 128)
                                 * _pow2(cols.T[r:r + 128] - cols.Tmax[r // 128])[:, :, None]).view(torch.uint8)
                           .view(128, -1).t()[None] for r in range(0, c["rows"], 128)])
            out["qT"] = v
            out["sT"] = _stored(cols.Tmax.repeat_interleave(128, dim=1), c)
        return out
    idx, probs = _routing(c, 10 * seed + 1)
    tok, slot, off = _groups(c, idx)
    if c["kind"] == "wgrad":
        cols = []
        for width, sub in ((c["N"], 2), (c["K"], 3)):
            v = _randn((c["T"], width), 1.0, 10 * seed + sub).to(torch.float64)
            cols.append(_Columns([_quant(v[t]) for t in tok], off, width))
        return {"dw": _wgrad(*cols, off, c["E"], c["N"], c["K"])}
    # dispatch: the rows past the last group keep what the buffers held (zero codes, a stored 1)
    H, M = c["H"], _m_cap(c)
    x = _randn((c["T"], H), 1.0, 10 * seed + 2).to(torch.float64)
    q, T = _grouped([_quant(x[t]) for t in tok], off, H)
    qm, sm = _row_pair(M, H, torch.uint8 if c["scale_fmt"] == "e8m0" else torch.float64)
    qm[:off[-1]] = q.view(torch.uint8)[:off[-1]]
    sm[:off[-1]] = _stored(T, c)[:off[-1]]
    row_map = torch.full((c["T"], c["k"]), -1, dtype=torch.int32, device="cuda")
    for e in range(c["E"]):
        row_map[tok[e], slot[e]] = off[e] + torch.arange(tok[e].numel(), dtype=torch.int32, device="cuda")
    rows = _randn((M, H), 1.0, 10 * seed + 3)
    y = torch.zeros((c["T"], H), dtype=torch.float64, device="cuda")
    for j in range(c["k"]):
        y += probs[:, j, None].to(torch.float64) * rows[row_map[:, j].long()].to(torch.float64)
    return {"y": y, "q": qm, "s": sm, "row_map": row_map, "offsets": torch.tensor(off, dtype=torch.int32, device="cuda")}
