"""The measured work of this library: what programs that run small convolutional networks on it have it do.

Single layers on the blocked layout, in fp32 and on uint8 codes, the layout change at the network's boundary, and
whole networks; sizes are those of the layer sweep, the paper's layer study and the stand-in networks of `workloads/`,
and ragged ones between them. `listed()` names the cases, `draw(rng)` gives further ones of the same ranges.
"""
import math

import numpy as np
import torch

import paper_2303_04769_amd as S
import workloads as WL

DEV = "cuda:0"
NETS = {"residual_cnn": WL.residual_cnn, "dsep_cnn": WL.dsep_cnn, "audio_cnn": WL.audio_cnn, "dense_autoencoder": WL.dense_autoencoder}


def listed():
    return [
        # ---- whole networks
        # Batch inference of images as they arrive (plain NCHW in, logits out): the benchmark's step.
        {"name": "residual_cnn_b256", "kind": "net", "net": "residual_cnn", "N": 256},
        # One image at a time, as an on-line service or a device loop does: latency is what counts.
        {"name": "dsep_cnn_b1", "kind": "net", "net": "dsep_cnn", "N": 1},
        # A quantized keyword-spotting model on a mid-sized batch of clips.
        {"name": "audio_cnn_u8_b100", "kind": "net_u8", "net": "audio_cnn", "N": 100},
        # ---- fp32 layers
        # The first row of the layer sweep at the benchmark's batch: the layer a convolutional network spends its time
        # in. The largest case.
        {"name": "conv3x3_64x56_b256", "kind": "conv", "N": 256, "Ci": 64, "Co": 64, "H": 56, "W": 56, "k": 3, "stride": 1},
        # A down-sampling layer on ragged sizes (odd image, channel counts that are no power of two), padded by one on
        # every side.
        {"name": "conv3x3s2_48to96_45x37_b50", "kind": "conv", "N": 50, "Ci": 48, "Co": 96, "H": 45, "W": 37, "k": 3, "stride": 2},
        # The small size of the paper's layer study (6 x 6 x 512) on a single image: few pixels, a long reduction.
        {"name": "conv3x3_512x6_b1", "kind": "conv", "N": 1, "Ci": 512, "Co": 512, "H": 6, "W": 6, "k": 3, "stride": 1},
        # A strided depthwise layer of a depthwise-separable network on an odd image.
        {"name": "dw3x3s2_96x57x43_b64", "kind": "dw", "N": 64, "Ci": 96, "H": 57, "W": 43, "k": 3, "stride": 2},
        # The pooling row of the layer sweep: memory traffic and little else.
        {"name": "maxpool3s2_256x56_b64", "kind": "pool", "N": 64, "Ci": 256, "H": 56, "W": 56, "k": 3, "stride": 2, "mode": "max"},
        # ---- quantized layers
        # The second row of the layer sweep on codes.
        {"name": "conv3x3_u8_128x28_b64", "kind": "conv_u8", "N": 64, "Ci": 128, "Co": 128, "H": 28, "W": 28, "k": 3, "stride": 1,
         "zx": 121, "zw": 135},
        # A pointwise layer of a depthwise-separable network, ragged sizes, symmetric filter codes.
        {"name": "conv1x1_u8_96to160_19x23_b133", "kind": "conv_u8", "N": 133, "Ci": 96, "Co": 160, "H": 19, "W": 23, "k": 1, "stride": 1,
         "zx": 0, "zw": 128},
        # The audio network's depthwise layer at its large batch.
        {"name": "dw3x3_u8_64x25x5_b1024", "kind": "dw_u8", "N": 1024, "Ci": 64, "H": 25, "W": 5, "k": 3, "stride": 1, "zx": 128, "zw": 131},
        # ---- the boundary
        # Quantized feature maps handed out of the library as a plain NCHW tensor.
        {"name": "unpack_u8_128x28_b64", "kind": "layout", "dtype": "u8", "dir": "unpack", "N": 64, "Ci": 128, "H": 28, "W": 28},
    ]


# ---------------------------------------------------------------------------------------------------- drawn cases

MAX_FLOPS = 7.0e9     # of a drawn layer; the largest listed one has 59e9
MAX_ELEMS = 24e6      # values of a drawn layer's larger tensor; the largest listed one has 51e6


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    return 16 * max(1, _log_int(rng, lo, hi) // 16)


def draw(rng):
    kind = rng.choice(["net", "net_u8", "conv", "conv", "dw", "pool", "conv_u8", "conv_u8", "dw_u8", "layout"])
    if kind == "net":
        return {"kind": kind, "net": rng.choice(sorted(NETS)), "N": _log_int(rng, 1, 256)}
    if kind == "net_u8":
        return {"kind": kind, "net": rng.choice(["residual_cnn", "dsep_cnn", "audio_cnn"]), "N": _log_int(rng, 1, 256)}
    while True:
        c = {"kind": kind, "N": _log_int(rng, 1, 1024), "Ci": _channels(rng, 16, 512), "H": _log_int(rng, 5, 112)}
        c["W"] = c["H"] if rng.random() < 0.4 else _log_int(rng, 5, 112)
        elems = c["N"] * c["Ci"] * c["H"] * c["W"]
        if kind in ("conv", "conv_u8"):
            c["Co"] = c["Ci"] if rng.random() < 0.5 else _channels(rng, 16, 512)
            c["k"] = rng.choice([1, 3, 3, 5] if kind == "conv" else [1, 3, 3])
            c["stride"] = rng.choice([1, 1, 2])
        elif kind in ("dw", "dw_u8"):
            c["k"], c["stride"] = 3, rng.choice([1, 1, 2])
        elif kind == "pool":
            c["k"], c["stride"], c["mode"] = rng.choice([(2, 2, "max"), (3, 2, "max"), (2, 2, "avg"), (3, 1, "max")])
        else:
            c["dtype"], c["dir"] = rng.choice(["f32", "u8"]), rng.choice(["pack", "unpack"])
        if kind.endswith("_u8"):
            c["zx"], c["zw"] = rng.choice([0, 128, rng.randrange(256)]), rng.choice([128, rng.randrange(256)])
        w = work(c)
        if w["flops"] <= MAX_FLOPS and max(elems, w["bytes"] / 8) <= MAX_ELEMS and elems >= 50000:
            return c


# ---------------------------------------------------------------------------------------------------- inputs

def _pad(c):
    p = 0 if c["kind"] == "pool" and not (c["k"] == 3 and c["stride"] == 1) else c["k"] // 2
    return (p, p, p, p)


def _out_hw(c):
    p = _pad(c)[0]
    return (c["H"] + 2 * p - c["k"]) // c["stride"] + 1, (c["W"] + 2 * p - c["k"]) // c["stride"] + 1


def _net_tensors(c, seed):
    net = NETS[c["net"]]()
    if c["kind"] == "net":
        x, ws = WL.network_tensors(net, c["N"], seed)
        return net, x, ws, None
    x, ws, qs = WL.quantized_network_tensors(net, c["N"], seed)
    return net, x, ws, qs


def _layer_tensors(c, seed):
    """Plain (NCHW / OIHW) input and filter: activations N(0, 1) with He-normal filters, codes uniform over 0..255."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    u8 = c["kind"].endswith("_u8") or c.get("dtype") == "u8"

    def make(shape, fan_in):
        if u8:
            return torch.randint(0, 256, shape, generator=g, device=DEV, dtype=torch.uint8)
        return torch.randn(shape, generator=g, device=DEV) * math.sqrt(2.0 / fan_in if fan_in else 1.0)

    x = make((c["N"], c["Ci"], c["H"], c["W"]), 0)
    w = None
    if c["kind"].startswith("conv"):
        w = make((c["Co"], c["Ci"], c["k"], c["k"]), c["Ci"] * c["k"] ** 2)
    elif c["kind"].startswith("dw"):
        w = make((c["Ci"], 1, c["k"], c["k"]), c["k"] ** 2)
    return x, w


def _quant(c):
    K = c["k"] ** 2 * (c["Ci"] if c["kind"] == "conv_u8" else 1)
    # a uniform code has a root mean square distance of 74 from the middle and more from another zero point
    mult, shift = WL.u8_multiplier(K, x_rms=math.hypot(74.0, c["zx"] - 128) * math.hypot(74.0, c["zw"] - 128) / 74.0)
    return {"zx": c["zx"], "zw": c["zw"], "zy": 128, "mult": mult, "shift": shift, "lo": 0, "hi": 255}


def prepare(case, seed):
    c = case
    if c["kind"] in ("net", "net_u8"):
        net, x, ws, qs = _net_tensors(c, seed)
        x_d = torch.from_numpy(x).to(DEV)
        last = net.layers[-1]
        if c["kind"] == "net":
            pn = S.PackedNetwork(net, ws, DEV)
            out = torch.empty(pn.out_elems(c["N"]), dtype=torch.float32, device=DEV)
        else:
            pn = S.PackedNetworkU8(net, ws, qs, DEV)
            out = torch.empty(pn.out_elems(c["N"]), dtype=torch.uint8, device=DEV)
        pn.workspace(c["N"])
        st = {"case": c, "pn": pn, "x": x_d, "out": out}
        # The plain input goes straight into the first layer where the library takes it there, else it is packed by a call.
        st["plain"] = False
        if c["kind"] == "net":
            try:
                pn.run_plain(x_d, out, c["N"])
                st["plain"] = True
            except S.SmallError as e:
                if e.code != 7:
                    raise
        if not st["plain"]:
            st["xb"] = torch.empty_like(x_d).reshape(-1)
        assert (last.Ho, last.Wo) == (1, 1)
        return st
    x, w = _layer_tensors(c, seed)
    u8 = x.dtype == torch.uint8
    pack = S.small_pack_u8 if u8 else S.small_pack
    N, Ci, H, W = x.shape
    xb = torch.empty(x.numel(), dtype=x.dtype, device=DEV)
    pack(x, xb, N, Ci, H, W, 16)
    if c["kind"] == "layout":
        src = x.reshape(-1) if c["dir"] == "pack" else xb
        return {"case": c, "x": src, "out": torch.empty_like(src)}
    Ho, Wo = _out_hw(c)
    Co = c.get("Co", Ci)
    st = {"case": c, "x": xb, "out": torch.empty(N * Co * Ho * Wo, dtype=x.dtype, device=DEV)}
    if w is not None:
        wb = torch.empty(w.numel(), dtype=w.dtype, device=DEV)
        if c["kind"] == "conv":
            S.small_pack_filter(w, wb, Co, Ci, c["k"], c["k"], 16, 16)
        elif c["kind"] == "dw":
            S.small_pack_dw_filter(w, wb, Ci, c["k"], c["k"], 16)
        elif c["kind"] == "conv_u8":
            S.small_pack_filter_u8(w, wb, Co, Ci, c["k"], c["k"], 16, 16)
            st["sums"] = torch.empty(Co, dtype=torch.int32, device=DEV)
            S.small_filter_sums_u8(wb, st["sums"], Co, Ci, c["k"], c["k"], 16, 16)
        else:
            wb = w.reshape(Ci // 16, 16, c["k"], c["k"]).permute(0, 2, 3, 1).contiguous().reshape(-1)
        st["w"] = wb
    if c["kind"].endswith("_u8"):
        st["q"] = S.small_quant(**_quant(c))
    return st


def run(state):
    c, out = state["case"], state["out"]
    kind, N = c["kind"], c["N"]
    if kind == "net":
        pn = state["pn"]
        if state["plain"]:
            pn.run_plain(state["x"], out, N)
        else:
            net = pn.net
            S.small_pack(state["x"], state["xb"], N, net.C0, net.H0, net.W0, net.layers[0].Cib)
            pn.run(state["xb"], out, N)
        return out
    if kind == "net_u8":
        pn = state["pn"]
        net = pn.net
        S.small_pack_u8(state["x"], state["xb"], N, net.C0, net.H0, net.W0, net.layers[0].Cib)
        pn.run(state["xb"], out, N)
        return out
    Ci, H, W, k, s = c["Ci"], c["H"], c["W"], c.get("k"), c.get("stride")
    if kind == "conv":
        S.small_conv2d(state["x"], state["w"], out, N, Ci, c["Co"], H, W, k, k, s, _pad(c), 16, 16)
    elif kind == "conv_u8":
        S.small_conv2d_u8(state["x"], state["w"], out, N, Ci, c["Co"], H, W, k, k, s, _pad(c), 16, 16, state["q"], state["sums"])
    elif kind == "dw":
        S.small_dwconv2d(state["x"], state["w"], out, N, Ci, H, W, k, k, s, _pad(c), 16)
    elif kind == "dw_u8":
        S.small_dwconv2d_u8(state["x"], state["w"], out, N, Ci, H, W, k, k, s, _pad(c), 16, state["q"])
    elif kind == "pool":
        S.small_pool2d(state["x"], out, N, Ci, H, W, k, k, s, _pad(c), 16, S.POOL_MAX if c["mode"] == "max" else S.POOL_AVG)
    else:
        move = {("f32", "pack"): S.small_pack, ("f32", "unpack"): S.small_unpack,
                ("u8", "pack"): S.small_pack_u8, ("u8", "unpack"): S.small_unpack_u8}[c["dtype"], c["dir"]]
        move(state["x"], out, N, Ci, H, W, 16)
    return out


def work(case):
    c = case
    if c["kind"] in ("net", "net_u8"):
        net = NETS[c["net"]]()
        size = 4 if c["kind"] == "net" else 1
        n = c["N"] * (net.C0 * net.H0 * net.W0 + net.n_out) + net.n_weights
        return {"bytes": float(size * n), "flops": 2.0 * c["N"] * net.macs_per_image()}
    size = 1 if c["kind"].endswith("_u8") or c.get("dtype") == "u8" else 4
    n_in = c["N"] * c["Ci"] * c["H"] * c["W"]
    if c["kind"] == "layout":
        return {"bytes": 2.0 * size * n_in, "flops": 0.0}
    Ho, Wo = _out_hw(c)
    if c["kind"].startswith("conv"):
        n_out, n_w = c["N"] * c["Co"] * Ho * Wo, c["Co"] * c["Ci"] * c["k"] ** 2
        return {"bytes": float(size * (n_in + n_out + n_w)), "flops": 2.0 * n_out * c["Ci"] * c["k"] ** 2}
    n_out = c["N"] * c["Ci"] * Ho * Wo
    n_w = c["Ci"] * c["k"] ** 2 if c["kind"].startswith("dw") else 0
    return {"bytes": float(size * (n_in + n_out + n_w)), "flops": (2.0 if n_w else 1.0) * n_out * c["k"] ** 2}


def tolerance(case):
    c = case
    if c["kind"] in ("conv_u8", "dw_u8", "net_u8", "layout") or (c["kind"] == "pool" and c["mode"] == "max"):
        return "exact"            # codes, copies and maxima
    if c["kind"] == "net":
        return NET_TOL
    # fp32 sums of K products: 1.6e-8 to 1.8e-8 sqrt(K) against 64 bits seen (4.3e-7 at K = 576, 1.1e-6 at K = 4608;
    # 5.7e-8 on depthwise layers), and about four times that stated; the largest single difference lies some five
    # times above the mean one.
    rel = max(4e-7, 7.2e-8 * math.sqrt(c["k"] ** 2 * (c["Ci"] if c["kind"] == "conv" else 1)))
    return {"rel": rel, "max": 10 * rel}


# About four times the largest error against 64-bit results seen (1.1e-7 residual CNN, 5.4e-7 depthwise-separable CNN).
NET_TOL = {"rel": 2e-6, "max": 2e-5}


# ---------------------------------------------------------------------------------------------------- 64-bit results

def _blocked(t, cb=16):
    """[N][C][H][W] -> the blocked layout, flat."""
    N, C, H, W = t.shape
    cb = min(cb, C)
    return t.reshape(N, C // cb, cb, H, W).permute(0, 1, 3, 4, 2).contiguous().reshape(-1)


def _windows(x, kh, kw, stride, pad, fill):
    """For every tap (y, x) the strided view of the padded input that it reads."""
    t, b, l, r = pad
    xp = torch.nn.functional.pad(x, (l, r, t, b), value=fill)
    Ho, Wo = (x.shape[2] + t + b - kh) // stride + 1, (x.shape[3] + l + r - kw) // stride + 1
    for y in range(kh):
        for z in range(kw):
            yield y, z, xp[:, :, y:y + (Ho - 1) * stride + 1:stride, z:z + (Wo - 1) * stride + 1:stride]


def _conv64(x, w, stride, pad):
    out = None
    for y, z, v in _windows(x, w.shape[2], w.shape[3], stride, pad, 0.0):
        N, C, Ho, Wo = v.shape
        term = w[:, :, y, z].contiguous() @ v.permute(1, 0, 2, 3).reshape(C, -1)
        out = term if out is None else out.add_(term)
    return out.reshape(w.shape[0], N, Ho, Wo).permute(1, 0, 2, 3)


def _dw64(x, w, stride, pad):
    return sum(v * w[:, 0, y, z].reshape(1, -1, 1, 1) for y, z, v in _windows(x, w.shape[2], w.shape[3], stride, pad, 0.0))


def _pool64(x, kh, kw, stride, pad, mode):
    if mode == "max":
        out = None
        for _, _, v in _windows(x, kh, kw, stride, pad, -math.inf):
            out = v if out is None else torch.maximum(out, v)
        return out
    total = sum(v for _, _, v in _windows(x, kh, kw, stride, pad, 0.0))
    count = sum(v for _, _, v in _windows(torch.ones_like(x[:1, :1]), kh, kw, stride, pad, 0.0))
    return total, count


def _requant64(acc, q):
    """acc: whole numbers in float64 (exact); the multiplication by the fixed-point scale in int64."""
    v = acc.round().to(torch.int64) * q["mult"]
    if q["shift"]:
        v = (v + (1 << (q["shift"] - 1))) >> q["shift"]
    return (v + q["zy"]).clamp(q["lo"], q["hi"])


def _net64(c, seed):
    net, x, ws, qs = _net_tensors(c, seed)
    u8 = qs is not None
    bufs = {WL.nets.IN: torch.from_numpy(x).to(DEV).double()}
    ws = [torch.from_numpy(w).to(DEV).double() for w in ws]
    for i, L in enumerate(net.layers):
        v, q = bufs[L.src], qs[i] if u8 else None
        if L.op in ("conv", "dense", "dw"):
            w = ws[L.w]
            if u8:
                v, w = v - q["zx"], w - q["zw"]
            y = (_dw64 if L.op == "dw" else _conv64)(v, w.reshape(w.shape[0], -1, L.kh, L.kw), L.stride, L.pad)
            y = _requant64(y, q).double() if u8 else y
        elif L.op == "relu":
            y = v.clamp(min=float(q["z"]) if u8 else 0.0)
        elif L.op == "add":
            b = bufs[L.src2]
            if u8:
                acc = (v - q["za"]).to(torch.int64) * q["mult_a"] + (b - q["zb"]).to(torch.int64) * q["mult_b"]
                y = (((acc + (1 << (q["shift"] - 1))) >> q["shift"]) + q["zy"]).clamp(q["lo"], q["hi"]).double()
            else:
                y = v + b
        else:
            total, n = _pool64(v, L.kh, L.kw, L.stride, L.pad, "avg")
            y = torch.div(total + torch.div(n, 2, rounding_mode="floor"), n, rounding_mode="floor") if u8 else total / n
        bufs[L.dst] = y
    out = _blocked(bufs[WL.nets.OUT])
    return out.to(torch.uint8) if u8 else out


def exact(case, seed):
    c = case
    if c["kind"] in ("net", "net_u8"):
        return _net64(c, seed)
    x, w = _layer_tensors(c, seed)
    if c["kind"] == "layout":
        return _blocked(x) if c["dir"] == "pack" else x.reshape(-1)
    if c["kind"] == "pool":
        if c["mode"] == "max":
            return _blocked(_pool64(x.double(), c["k"], c["k"], c["stride"], _pad(c), "max"))
        total, n = _pool64(x.double(), c["k"], c["k"], c["stride"], _pad(c), "avg")
        return _blocked(total / n)
    layer = _conv64 if c["kind"].startswith("conv") else _dw64
    if not c["kind"].endswith("_u8"):
        return _blocked(layer(x.double(), w.double(), c["stride"], _pad(c)))
    q = _quant(c)
    return _blocked(_requant64(layer(x.double() - q["zx"], w.double() - q["zw"], c["stride"], _pad(c)), q).to(torch.uint8))
