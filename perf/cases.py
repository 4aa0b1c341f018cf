"""Performance cases: what a DFP16 training program has this library do.

Four kinds of work, all through the public binding:

* ``layer``   one convolution layer of a training step: quantise x, w and dy,
  forward, down-convert y, backward-data, down-convert dx, backward-weights
  (``passes``: "train" all of it, "first" without backward-data as in a
  network's first layer, "forward" the forward half alone);
* ``fc``      the same step of a fully connected layer through the GEMM, or
  with ``block`` > 0 its Blocked-DFP forward product;
* ``bn``      batch normalisation + residual + ReLU, forward and backward;
* ``sgd``     the FP32 weight update and Q_w.

Inputs are drawn on the GPU with the distributions of
``paper_1802_00930_amd.workloads``: ReLU(N(0,1)) activations, He-normal
weights, N(0,1)*1e-3 gradients.
"""
from __future__ import annotations

import math

import torch

from paper_1802_00930_amd import dfp

DEV = "cuda"


def _layer(name, n, c, hw, k, r, stride=1, pad=0, L=64, bits=15, rounding="nearest", passes="train", dfp32=False):
    return {"name": name, "kind": "layer", "n": n, "c": c, "hw": hw, "k": k, "r": r, "stride": stride, "pad": pad,
            "L": L, "bits": bits, "rounding": rounding, "passes": passes, "dfp32": dfp32}


def listed():
    return [
        # the smallest layer of the benchmark: every launch is latency
        _layer("layer16x32", 2, 16, 14, 32, 3, 1, 1, L=16),
        # the paper's ResNet-50 conv2_x 3x3 layer, the benchmark's headline
        _layer("res2_3x3", 32, 64, 56, 64, 3, 1, 1, rounding="stochastic"),
        # the same layer with the short accumulation chain of the chunk sweep
        _layer("res2_3x3_L16", 32, 64, 56, 64, 3, 1, 1, L=16, rounding="stochastic"),
        # ResNet-50 conv4_x bottleneck 1x1 layer
        _layer("res4_1x1", 64, 1024, 14, 256, 1, rounding="biased"),
        # ResNet-50 conv5_x 3x3: long reduction over small, odd 7x7 images
        _layer("res5_3x3", 64, 512, 7, 512, 3, 1, 1),
        # VGG-16 conv1_2: the largest activations of the benchmark
        _layer("vgg_conv1_2", 32, 64, 224, 64, 3, 1, 1, rounding="stochastic"),
        # ResNet-50 stem as a network's first layer: 3 channels, 7x7, stride 2
        _layer("stem_first", 64, 3, 224, 64, 7, 2, 3, passes="first"),
        # full-width 16-bit integers; the products carry two more bits, so the chain is a quarter as long
        _layer("res4_3x3_p16", 32, 256, 14, 256, 3, 1, 1, L=16, bits=16),
        # ResNet-50's fully connected layer
        {"name": "fc", "kind": "fc", "m": 64, "fin": 2048, "fout": 1000, "L": 64, "block": 0, "rounding": "nearest"},
        # its forward product with one exponent per 128 input features
        {"name": "fc_blocked", "kind": "fc", "m": 64, "fin": 2048, "fout": 1000, "L": 64, "block": 128,
         "rounding": "nearest"},
        # the normalisation that ends a ResNet-50 conv2_x bottleneck
        {"name": "bn_res2", "kind": "bn", "n": 64, "c": 256, "hw": 3136, "rounding": "nearest"},
        # update of a conv5_x 3x3 filter
        {"name": "sgd_res5", "kind": "sgd", "n": 512 * 512 * 9, "rounding": "nearest"},
    ]


_MOST_MACS = 32 * 64 * 64 * 9 * 224 * 224
_MOST_VALUES = 32 * 64 * 224 * 224


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_layer(rng):
    while True:
        family = rng.choice(("3x3", "3x3", "3x3", "1x1", "1x1", "1x1s2", "stem"))
        n = _log(rng, 1, 64)
        if family == "stem":
            c, k, r, stride, pad = rng.choice((1, 3, 4)), 8 * _log(rng, 2, 12), 7, 2, 3
            hw = _log(rng, 63, 224)
        else:
            top = 2048 if family != "3x3" else 512
            c, k = (8 * _log(rng, 2, top // 8) for _ in range(2))
            if rng.random() < 0.2:
                k += rng.randrange(1, 8)
            r, pad = (3, 1) if family == "3x3" else (1, 0)
            stride = 2 if family == "1x1s2" else 1
            hw = rng.choice((7, 14, 28, 56, 112)) if rng.random() < 0.6 else _log(rng, 7, 112)
        bits = 16 if rng.random() < 0.125 else 15
        L = 16 if bits == 16 else rng.choice((64, 64, 64, 64, 32, 16, 8))
        p = (hw + 2 * pad - r) // stride + 1
        macs, values = n * k * c * r * r * p * p, n * max(c * hw * hw, k * p * p)
        if macs > (2e9 if bits == 16 else _MOST_MACS / 2) or values > _MOST_VALUES / 2:
            continue
        passes = "first" if family == "stem" else rng.choice(("train", "train", "train", "forward"))
        return _layer(None, n, c, hw, k, r, stride, pad, L, bits, rng.choice(("nearest", "stochastic", "biased", "down")),
                      passes, dfp32=bits == 15 and rng.random() < 0.125)


def draw(rng):
    kind = rng.choice(("layer",) * 8 + ("fc", "fc_blocked", "bn", "sgd"))
    rounding = rng.choice(("nearest", "stochastic", "biased", "down"))
    if kind == "layer":
        case = _draw_layer(rng)
        del case["name"]
        return case
    if kind in ("fc", "fc_blocked"):
        fin = _log(rng, 64, 4096) if rng.random() < 0.5 else 64 * _log(rng, 1, 64)
        return {"kind": "fc", "m": _log(rng, 1, 256), "fin": fin, "fout": _log(rng, 10, 4096),
                "L": rng.choice((64, 64, 32)), "block": 128 if kind == "fc_blocked" else 0, "rounding": rounding}
    if kind == "bn":
        while True:
            n, c, side = _log(rng, 1, 64), 8 * _log(rng, 2, 256), _log(rng, 7, 112)
            if n * c * side * side <= 64 * 256 * 3136:
                return {"kind": "bn", "n": n, "c": c, "hw": side * side, "rounding": rounding}
    return {"kind": "sgd", "n": _log(rng, 1000, 20_000_000), "rounding": rounding}


# ------------------------------------------------------------------ inputs
def _p(case):
    return (case["hw"] + 2 * case["pad"] - case["r"]) // case["stride"] + 1


def _normal(gen, shape, scale=1.0, relu=False):
    t = torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)
    if relu:
        t.clamp_(min=0)
    return t if scale == 1.0 else t.mul_(scale)


def _fp32_inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    if case["kind"] == "layer":
        n, c, hw, k, r, p = case["n"], case["c"], case["hw"], case["k"], case["r"], _p(case)
        return (_normal(gen, (n, c, hw, hw), relu=True), _normal(gen, (k, c, r, r), math.sqrt(2.0 / (c * r * r))),
                _normal(gen, (n, k, p, p), 1e-3))
    if case["kind"] == "fc":
        m, fin, fout = case["m"], case["fin"], case["fout"]
        return (_normal(gen, (m, fin), relu=True), _normal(gen, (fout, fin), math.sqrt(1.0 / fin)),
                _normal(gen, (m, fout), 1e-3))
    if case["kind"] == "bn":
        shape = (case["n"], case["c"], case["hw"])
        y = (_normal(gen, shape) * 3000).round_().clamp_(-16384, 16384).to(torch.int16)
        dz = (_normal(gen, shape) * 3000).round_().clamp_(-16384, 16384).to(torch.int16)
        gamma = _normal(gen, (case["c"],), 0.2) + 1
        return y, dz, _normal(gen, shape), gamma, _normal(gen, (case["c"],), 0.2)
    n = case["n"]
    return _normal(gen, (n,), 0.02), _normal(gen, (n,), 1e-3), _normal(gen, (n,), 1e-3)


_BN_EXP = {"y": -11, "dz": -22}  # exponents that a down-converted y and dz have
_SGD = (0.1, 0.9, 1e-4)          # learning rate, momentum, weight decay
_SEED = 1                        # Philox key of the stochastic mode


def _scales(*names):
    return {n: dfp.new_scale(DEV) for n in names}


def _int16(t):
    return torch.empty_like(t, dtype=torch.int16)


def prepare(case, seed):
    st = {"case": dict(case)}
    inputs = _fp32_inputs(case, seed)
    if case["kind"] == "layer":
        c, k, r, hw = case["c"], case["k"], case["r"], case["hw"]
        x, w, dy = inputs

        def desc(L):
            return dfp.make_desc(case["n"], c, hw, hw, k, r, r, case["stride"], case["pad"], chunk_len=L,
                                 bits=case["bits"], rounding=case["rounding"], seed=_SEED)
        full = case["dfp32"]  # one chunk over the whole reduction, INT32 outputs
        st["desc"] = {"fwd": desc(c * r * r if full else case["L"]), "bwd": desc(k * r * r if full else case["L"]),
                      "wt": desc(case["L"])}
        st["ws"] = {n: dfp.alloc_workspace(st["desc"][n], d, DEV)
                    for n, d in (("fwd", dfp.FWD), ("bwd", dfp.BWD_DATA), ("wt", dfp.BWD_WT))}
        out = torch.int32 if full else torch.float32
        st.update(x=x, w=w, dy=dy, qx=_int16(x), qw=_int16(w), qdy=_int16(dy), y=torch.empty_like(dy, dtype=out),
                  qy=_int16(dy), dx=torch.empty_like(x, dtype=out), qdx=_int16(x), dw=torch.empty_like(w))
        st["s"] = _scales("x", "w", "dy", "y", "dx", "qy", "qdx")
    elif case["kind"] == "fc":
        m, fin, fout, L = case["m"], case["fin"], case["fout"], case["L"]
        x, w, dy = inputs
        st.update(x=x, w=w, dy=dy, qx=_int16(x), qw=_int16(w), y=torch.empty_like(dy), qy=_int16(dy))
        fwd = dfp.make_gemm_desc(m, fout, fin, False, True, L)
        if case["block"]:
            nb = -(-fin // case["block"])
            st.update(desc=fwd, ex=torch.empty(nb, m, dtype=torch.int8, device=DEV),
                      ew=torch.empty(nb, fout, dtype=torch.int8, device=DEV),
                      ws=dfp.alloc_gemm_blocked_workspace(fwd, case["block"], DEV))
        else:
            st["desc"] = (fwd, dfp.make_gemm_desc(m, fin, fout, False, False, L),
                          dfp.make_gemm_desc(fout, fin, m, True, False, L))
            st["ws"] = [dfp.alloc_gemm_workspace(d, DEV) for d in st["desc"]]
            st.update(qdy=_int16(dy), dx=torch.empty_like(x), qdx=_int16(x), dw=torch.empty_like(w))
        st["s"] = _scales("x", "w", "dy", "y", "dx")
    elif case["kind"] == "bn":
        y, dz, res, gamma, beta = inputs
        d = dfp.make_bn_desc(case["n"], case["c"], case["hw"], rounding=case["rounding"], seed=_SEED)
        st.update(desc=d, y=y, dz=dz, res=res, gamma=gamma, beta=beta, z=torch.empty_like(res), zq=_int16(res),
                  dyq=_int16(res), dres=torch.empty_like(res), ws=dfp.alloc_bn_workspace(d, DEV),
                  **{n: torch.empty_like(gamma) for n in ("mean", "inv_std", "dgamma", "dbeta")})
        st["s"] = _scales("y", "dz", "z", "dy")
        for n, e in _BN_EXP.items():
            st["s"][n][1] = e
    else:
        w, v, dw = inputs
        st.update(w=w, v=v, dw=dw, wq=_int16(w), s=_scales("w"))
    return st


# --------------------------------------------------------------------- run
def _run_layer(st):
    case, d, ws, s = st["case"], st["desc"], st["ws"], st["s"]
    full, passes = case["dfp32"], case["passes"]
    out = {}
    dfp.dfp_quantize(d["fwd"], dfp.ROLE_X, st["x"], st["qx"], s["x"])
    dfp.dfp_quantize(d["fwd"], dfp.ROLE_W, st["w"], st["qw"], s["w"])
    if full:
        dfp.dfp_conv_fwd_i32(d["fwd"], st["qx"], s["x"], st["qw"], s["w"], st["y"], s["y"], ws["fwd"])
        dfp.dfp_downconvert_i32(d["fwd"], dfp.ROLE_Y, st["y"], s["y"], st["qy"], s["qy"], amax_ready=True)
        out["sqy"] = s["qy"]
    else:
        dfp.dfp_conv_fwd(d["fwd"], st["qx"], s["x"], st["qw"], s["w"], st["y"], s["y"], ws["fwd"])
        dfp.dfp_downconvert(d["fwd"], dfp.ROLE_Y, st["y"], st["qy"], s["y"], amax_ready=True)
    out.update(qx=st["qx"], sx=s["x"], qw=st["qw"], sw=s["w"], y=st["y"], sy=s["y"], qy=st["qy"])
    if passes == "forward":
        return out
    dfp.dfp_quantize(d["wt"], dfp.ROLE_DY, st["dy"], st["qdy"], s["dy"])
    out.update(qdy=st["qdy"], sdy=s["dy"])
    if passes == "train":
        if full:
            dfp.dfp_conv_bwd_data_i32(d["bwd"], st["qdy"], s["dy"], st["qw"], s["w"], st["dx"], s["dx"], ws["bwd"])
            dfp.dfp_downconvert_i32(d["bwd"], dfp.ROLE_DX, st["dx"], s["dx"], st["qdx"], s["qdx"], amax_ready=True)
            out["sqdx"] = s["qdx"]
        else:
            dfp.dfp_conv_bwd_data(d["bwd"], st["qdy"], s["dy"], st["qw"], s["w"], st["dx"], s["dx"], ws["bwd"])
            dfp.dfp_downconvert(d["bwd"], dfp.ROLE_DX, st["dx"], st["qdx"], s["dx"], amax_ready=True)
        out.update(dx=st["dx"], sdx=s["dx"], qdx=st["qdx"])
    dfp.dfp_conv_bwd_weights(d["wt"], st["qx"], s["x"], st["qdy"], s["dy"], st["dw"], ws["wt"])
    out["dw"] = st["dw"]
    return out


def _run_fc(st):
    case, d, s = st["case"], st["desc"], st["s"]
    rnd = case["rounding"]
    if case["block"]:
        b = case["block"]
        dfp.dfp_quantize_blocked(b, 15, rnd, _SEED, dfp.ROLE_X, st["x"], st["qx"], st["ex"], s["x"])
        dfp.dfp_quantize_blocked(b, 15, rnd, _SEED, dfp.ROLE_W, st["w"], st["qw"], st["ew"], s["w"])
        dfp.dfp_gemm_blocked(d, b, st["qx"], st["ex"], st["qw"], st["ew"], st["y"], s["y"], st["ws"])
        dfp.dfp_downconvert_tensor(15, rnd, _SEED, dfp.ROLE_Y, st["y"], st["qy"], s["y"], amax_ready=True)
        return {n: st[n] for n in ("qx", "ex", "qw", "ew", "y", "qy")} | {"sy": s["y"]}
    dfp.dfp_quantize_tensor(15, rnd, _SEED, dfp.ROLE_X, st["x"], st["qx"], s["x"])
    dfp.dfp_quantize_tensor(15, rnd, _SEED, dfp.ROLE_W, st["w"], st["qw"], s["w"])
    dfp.dfp_quantize_tensor(15, rnd, _SEED, dfp.ROLE_DY, st["dy"], st["qdy"], s["dy"])
    dfp.dfp_gemm(d[0], st["qx"], s["x"], st["qw"], s["w"], st["y"], s["y"], st["ws"][0])
    dfp.dfp_downconvert_tensor(15, rnd, _SEED, dfp.ROLE_Y, st["y"], st["qy"], s["y"], amax_ready=True)
    dfp.dfp_gemm(d[1], st["qdy"], s["dy"], st["qw"], s["w"], st["dx"], s["dx"], st["ws"][1])
    dfp.dfp_downconvert_tensor(15, rnd, _SEED, dfp.ROLE_DX, st["dx"], st["qdx"], s["dx"], amax_ready=True)
    dfp.dfp_gemm(d[2], st["qdy"], s["dy"], st["qx"], s["x"], st["dw"], None, st["ws"][2])
    return {n: st[n] for n in ("qx", "qw", "qdy", "y", "qy", "dx", "qdx", "dw")} | {"s" + n: t for n, t in s.items()}


def run(st):
    kind = st["case"]["kind"]
    if kind == "layer":
        return _run_layer(st)
    if kind == "fc":
        return _run_fc(st)
    s = st["s"]
    if kind == "bn":
        dfp.dfp_bn_relu_fwd(st["desc"], st["y"], s["y"], st["gamma"], st["beta"], st["zq"], s["z"], st["mean"],
                            st["inv_std"], res=st["res"], z=st["z"], workspace=st["ws"])
        dfp.dfp_bn_relu_bwd(st["desc"], st["dz"], s["dz"], st["y"], s["y"], st["gamma"], st["beta"], st["mean"],
                            st["inv_std"], st["dyq"], s["dy"], st["dgamma"], st["dbeta"], res=st["res"],
                            dres=st["dres"], workspace=st["ws"])
        return {n: st[n] for n in ("zq", "z", "mean", "inv_std", "dyq", "dgamma", "dbeta", "dres")} | {
            "sz": s["z"], "sdy": s["dy"]}
    dfp.dfp_sgd_quantize(*_SGD, 15, st["case"]["rounding"], _SEED, st["w"], st["v"], st["dw"], st["wq"], s["w"])
    return {"w": st["w"], "v": st["v"], "wq": st["wq"], "sw": s["w"]}


# -------------------------------------------------------------------- work
def work(case):
    """Inputs read once, outputs written once; a multiply-accumulate is two operations."""
    if case["kind"] == "layer":
        n, c, k, r = case["n"], case["c"], case["k"], case["r"]
        x, w, y = n * c * case["hw"] ** 2, k * c * r * r, n * k * _p(case) ** 2
        convs = {"train": 3, "first": 2, "forward": 1}[case["passes"]]
        size = {"train": 12 * x + 10 * w + 12 * y, "first": 6 * x + 10 * w + 12 * y, "forward": 6 * (x + w + y)}
        return {"bytes": size[case["passes"]], "flops": 2 * convs * y * c * r * r}
    if case["kind"] == "fc":
        m, fin, fout = case["m"], case["fin"], case["fout"]
        x, w, y = m * fin, fin * fout, m * fout
        if case["block"]:
            return {"bytes": 6 * (x + w + y), "flops": 2 * m * fin * fout}
        return {"bytes": 12 * x + 10 * w + 12 * y, "flops": 6 * m * fin * fout}
    if case["kind"] == "bn":  # y, res -> zq, z; dz, y, res -> dyq, dres
        return {"bytes": 26 * case["n"] * case["c"] * case["hw"], "flops": 20 * case["n"] * case["c"] * case["hw"]}
    return {"bytes": 22 * case["n"], "flops": 6 * case["n"]}


def tolerance(case):
    """The interface fixes every rounding and the order of every FP32 sum, and a repeated run gives the same bits."""
    return "exact"


# ------------------------------------------------------- 64-bit references
def _philox(idx, role, seed):
    """Word idx mod 4 of Philox4x32-10 block idx div 4 (key seed, counter (block, 0, role, 0)), in int64."""
    low = 0xFFFFFFFF

    def mul(a, c):
        hi = (a * (c >> 16) + ((a * (c & 0xFFFF)) >> 16)) >> 16
        return hi & low, (a * c) & low

    q = idx[::4] >> 2
    c = [q & low, q >> 32, torch.full_like(q, role), torch.zeros_like(q)]
    k0, k1 = seed & low, seed >> 32
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return torch.stack(c, 1).reshape(-1)[: idx.numel()]


def _quantized(f, bits, rounding, role):
    """The DFP value i * 2^E of every element, as float64 integers i and the exponent E."""
    top = float(f.abs().max())
    if top == 0.0:
        return f.double(), 0
    e = math.frexp(top)[1] - 1 - (bits - 2)
    x = f.double() * 2.0 ** -e
    if rounding == "nearest":
        i = torch.round(x)
    elif rounding == "biased":
        i = torch.floor(x + 0.5)
    else:
        i = torch.floor(x)
        if rounding == "stochastic":
            for a in range(0, f.numel(), 1 << 24):  # a multiple of four elements at a time
                xs, part = x.view(-1)[a: a + (1 << 24)], i.view(-1)[a: a + (1 << 24)]
                u = _philox(torch.arange(a, a + xs.numel(), device=f.device), role, _SEED)
                part += (u < torch.floor((xs - part) * 2.0 ** 32)).double()
    if bits == 16:
        i.clamp_(-32767, 32767)
    return i, e


def _conv64(case, x, w, dy, scale_y, scale_dx, scale_dw, want_dx):
    """Forward, backward-data and backward-weights in float64, one image at a time."""
    n, k, r, p, hw = case["n"], case["k"], case["r"], _p(case), case["hw"]
    opt = {"kernel_size": r, "stride": case["stride"], "padding": case["pad"]}
    wm = w.reshape(k, -1)
    y = torch.empty(n, k, p, p, dtype=torch.float64, device=x.device)
    dx = torch.empty_like(x) if want_dx else None
    dw = torch.zeros_like(wm)
    for i in range(n):
        cols = torch.nn.functional.unfold(x[i: i + 1], **opt)[0]
        y[i] = (wm @ cols).view(k, p, p) * scale_y
        if dy is not None:
            g = dy[i].reshape(k, -1)
            dw += g @ cols.t()
            if want_dx:
                dx[i] = torch.nn.functional.fold((wm.t() @ g)[None], (hw, hw), **opt)[0] * scale_dx
    return y, dx, (dw * scale_dw).view_as(w)


def exact(case, seed):
    inputs = _fp32_inputs(case, seed)
    kind = case["kind"]
    if kind == "layer":
        b, rnd = case["bits"], case["rounding"]
        x, ex = _quantized(inputs[0], b, rnd, dfp.ROLE_X)
        w, ew = _quantized(inputs[1], b, rnd, dfp.ROLE_W)
        dy, ed = _quantized(inputs[2], b, rnd, dfp.ROLE_DY) if case["passes"] != "forward" else (None, 0)
        y, dx, dw = _conv64(case, x, w, dy, 2.0 ** (ex + ew), 2.0 ** (ed + ew), 2.0 ** (ex + ed),
                            case["passes"] == "train")
        full = case["dfp32"]
        out = dict.fromkeys(("qx", "sx", "qw", "sw", "sy", "qy")) | {"y": None if full else y}
        if full:
            out["sqy"] = None
        if case["passes"] == "forward":
            return None if full else out
        out.update(qdy=None, sdy=None, dw=dw)
        if case["passes"] == "train":
            out.update(dx=None if full else dx, sdx=None, qdx=None)
            if full:
                out["sqdx"] = None
        return out
    if kind == "fc":
        rnd, bk = case["rounding"], case["block"]
        if bk:
            return None if rnd == "stochastic" else {
                **dict.fromkeys(("qx", "ex", "qw", "ew", "qy", "sy")),
                "y": _blocked64(inputs[0], bk, rnd) @ _blocked64(inputs[1], bk, rnd).t()}
        (x, ex), (w, ew), (dy, ed) = (_quantized(t, 15, rnd, role) for t, role in
                                      zip(inputs, (dfp.ROLE_X, dfp.ROLE_W, dfp.ROLE_DY)))
        return {**dict.fromkeys(("qx", "qw", "qdy", "qy", "qdx", "sx", "sw", "sdy", "sy", "sdx")),
                "y": x @ w.t() * 2.0 ** (ex + ew), "dx": dy @ w * 2.0 ** (ed + ew), "dw": dy.t() @ x * 2.0 ** (ex + ed)}
    if kind == "bn":
        return _bn64(case, *inputs)
    w, v, dw = (t.double() for t in inputs)
    lr, mu, wd = _SGD
    v = mu * v + (wd * w + dw)
    return {"w": w - lr * v, "v": v, "wq": None, "sw": None}


def _blocked64(f, block, rounding):
    """Every element's DFP value with one exponent per block of a row."""
    parts = []
    for a in range(0, f.shape[1], block):
        x = f[:, a: a + block].double()
        top = x.abs().amax(1, keepdim=True)
        e = torch.where(top > 0, torch.frexp(top)[1].double() - 14, torch.zeros_like(top))
        x = x * torch.exp2(-e)
        x = {"nearest": torch.round, "biased": lambda t: torch.floor(t + 0.5), "down": torch.floor}[rounding](x)
        parts.append(x * torch.exp2(e))
    return torch.cat(parts, 1)


def _bn64(case, y, dz, res, gamma, beta):
    cnt = case["n"] * case["hw"]
    yv, g = y.double() * 2.0 ** _BN_EXP["y"], dz.double() * 2.0 ** _BN_EXP["dz"]
    ga, be = gamma.double()[None, :, None], beta.double()[None, :, None]
    mean = yv.mean((0, 2))
    inv = 1.0 / torch.sqrt((yv * yv).mean((0, 2)) - mean * mean + 1e-5)
    xhat = (yv - mean[None, :, None]) * inv[None, :, None]
    pre = xhat * ga + be + res.double()
    g = torch.where(pre > 0, g, torch.zeros_like(g))
    return {"zq": None, "z": pre.clamp(min=0), "mean": mean, "inv_std": inv, "dyq": None,
            "dgamma": (g * xhat).sum((0, 2)), "dbeta": g.sum((0, 2)), "dres": g, "sz": None, "sdy": None}
