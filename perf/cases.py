"""The performance cases of the two operators, through the package's public calls.

Four kinds of pass, each as a user's program makes it:

  vt_forward   ``sample_vt``: inference with the fused Sampling-VT operator
  vt_train     ``sample_vt_autograd`` and its backward: a training step's share of
               the view transformation (output and feature gradient)
  sca_forward  ``sca_forward``: inference with FlashSCA
  sca_train    ``sca_autograd`` and its backward: output and the gradients of the
               value maps, the sampling offsets and the attention logits

The listed sizes are those of the repository's workloads (``synth``): a small
grid, the 200 x 200 x 8 setting, the half-precision batch, the long-range grid,
the height sweep's largest point, BEVFormer-base and its small relative, and
one ragged size.  ``draw`` spreads sizes over the same ranges.

Inputs are seeded: a ring of cameras looking outwards (focal length 0.75 image
widths, a small jitter of every pose), standard-normal feature maps, and for
FlashSCA the initial offset pattern of BEVFormer's offset predictor plus unit
noise.  They are made on the GPU, where a program has them.

``exact`` evaluates both operators and their gradients in plain torch with
float64 sums.  The sampling coordinates follow the operators' documented
float32 recipe (every product and sum rounded on its own), since masks and
floors are decided by those float32 values; each float32 step is computed in
float64 and rounded once, which gives the correctly rounded float32 result.
"""
import math

import numpy as np
import torch

import paper_2607_10071_amd as fb

_DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def _vt(name, op, B, N, img_h, img_w, H, W, C, dtype, X, Y, half, z_lo, z_hi, Z, reduce="mean"):
    return {"name": name, "op": op, "B": B, "N": N, "img_h": img_h, "img_w": img_w, "H": H, "W": W,
            "C": C, "dtype": dtype, "X": X, "Y": Y, "half": half, "z_lo": z_lo, "z_hi": z_hi,
            "Z": Z, "reduce": reduce}


def _sca(name, op, B, N, img_h, img_w, H, W, L, C, heads, P, dtype, X, Y, half, Z, reduce="mean"):
    return {"name": name, "op": op, "B": B, "N": N, "img_h": img_h, "img_w": img_w, "H": H, "W": W,
            "L": L, "C": C, "heads": heads, "P": P, "dtype": dtype, "X": X, "Y": Y, "half": half,
            "z_lo": -5.0, "z_hi": 3.0, "Z": Z, "reduce": reduce}


def listed():
    return [
        # a small grid around the vehicle: latency of one call
        _vt("vt_forward_small", "vt_forward", 1, 6, 256, 704, 16, 44, 32, "f32", 50, 50, 25.0,
            -5.0, 3.0, 4),
        # the 200 x 200 x 8 setting of the headline figure
        _vt("vt_forward_200x200x8", "vt_forward", 1, 6, 256, 704, 32, 88, 80, "f32", 200, 200,
            50.0, -5.0, 3.0, 8),
        # highway range, large images, half precision
        _vt("vt_forward_long_range", "vt_forward", 1, 6, 900, 1600, 112, 200, 64, "f16", 400, 400,
            100.0, -5.0, 3.0, 16),
        # many heights on a fine grid, eight cameras, a batch: the largest forward
        _vt("vt_forward_64_heights", "vt_forward", 2, 8, 256, 704, 32, 88, 64, "bf16", 512, 512,
            64.0, -5.0, 3.0, 64),
        # sizes that fit no tile, a rectangular grid, the plain sum over cameras
        _vt("vt_forward_ragged", "vt_forward", 3, 5, 270, 610, 34, 77, 99, "f32", 173, 211, 45.0,
            -4.0, 4.0, 7, "sum"),
        # one training step of the view transformation at the 200 x 200 x 8 setting
        _vt("vt_train_200x200x8", "vt_train", 1, 6, 256, 704, 32, 88, 80, "f32", 200, 200, 50.0,
            -5.0, 3.0, 8),
        # the same in mixed precision over a batch, wider features
        _vt("vt_train_batch_bf16", "vt_train", 4, 6, 256, 704, 32, 88, 128, "bf16", 200, 200, 50.0,
            -5.0, 3.0, 8),
        # a small cross-attention: latency of one call
        _sca("sca_forward_small", "sca_forward", 1, 6, 256, 704, 16, 44, 2, 32, 4, 4, "f32", 23, 23,
             25.0, 2),
        # BEVFormer-base inference, 8 points per head and level
        _sca("sca_forward_base", "sca_forward", 1, 6, 900, 1600, 116, 200, 4, 256, 8, 8, "f32", 200,
             200, 51.2, 4),
        # BEVFormer-base inference in half precision, two samples
        _sca("sca_forward_base_bf16", "sca_forward", 2, 6, 900, 1600, 116, 200, 4, 256, 8, 8, "bf16",
             200, 200, 51.2, 4),
        # one training step of the cross-attention at BEVFormer-base
        _sca("sca_train_base", "sca_train", 1, 6, 900, 1600, 116, 200, 4, 256, 8, 8, "f32", 200, 200,
             51.2, 4),
        # the same with 16 points in mixed precision
        _sca("sca_train_base_p16_bf16", "sca_train", 1, 6, 900, 1600, 116, 200, 4, 256, 8, 16, "bf16",
             200, 200, 51.2, 4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = {}
    for c in listed():
        most[c["op"]] = max(most.get(c["op"], 0.0), _cost(c))
    op = rng.choice(["vt_forward", "vt_train", "sca_forward", "sca_train"])
    while True:
        # all sizes anew until the case costs no more than the largest of its kind
        img_h, img_w = rng.choice([(256, 704), (448, 800), (900, 1600), (270, 610)])
        dtype = rng.choice(["f32", "f32", "f16", "bf16"])
        reduce = rng.choice(["mean", "mean", "mean", "sum"])
        N = rng.choice([4, 5, 6, 6, 6, 8])
        B = rng.choice([1, 1, 2, 3, 4])
        if op.startswith("vt"):
            stride = rng.choice([8, 8, 16])
            C = 8 * _log_int(rng, 4, 32) if rng.random() < 0.75 else _log_int(rng, 32, 256)
            half = rng.uniform(25.0, 100.0)
            case = _vt("", op, B, N, img_h, img_w, -(-img_h // stride), -(-img_w // stride), C,
                       dtype, _log_int(rng, 50, 512), _log_int(rng, 50, 512), half, -5.0, 3.0,
                       _log_int(rng, 4, 64 if op == "vt_forward" else 16), reduce)
        else:
            stride = rng.choice([8, 16])
            Z = rng.choice([2, 4, 4])
            case = _sca("", op, B, N, img_h, img_w, -(-img_h // stride), -(-img_w // stride),
                        rng.randint(1, 4), 0, rng.choice([4, 8, 8]), Z * rng.choice([1, 2, 3, 4, 8]),
                        dtype, _log_int(rng, 23, 200), _log_int(rng, 23, 200),
                        rng.uniform(25.0, 55.0), Z, reduce)
            case["C"] = case["heads"] * rng.choice([8, 16, 24, 32, 32, 64])
        if _cost(case) <= most[op]:
            del case["name"]
            return case


# ---- inputs ----------------------------------------------------------------------------------


def _rotation(axis, t):
    c, s = math.cos(t), math.sin(t)
    if axis == "x":
        return np.array([[1, 0, 0], [0, c, -s], [0, s, c]])
    if axis == "y":
        return np.array([[c, 0, s], [0, 1, 0], [-s, 0, c]])
    return np.array([[c, -s, 0], [s, c, 0], [0, 0, 1]])


def _rig(case, seed):
    """lidar2img [B, N, 4, 4] float32 of a ring of cameras, jittered per batch element."""
    rng = np.random.default_rng([int(seed), 11])
    B, N, w, h = case["B"], case["N"], case["img_w"], case["img_h"]
    K = np.array([[0.75 * w, 0, 0.5 * w], [0, 0.75 * w, 0.5 * h], [0, 0, 1.0]])
    out = np.zeros((B, N, 4, 4), dtype=np.float32)
    for b in range(B):
        for n in range(N):
            yaw = 2.0 * math.pi * n / N
            roll, pitch, turn = rng.uniform(-2.0, 2.0, 3) * math.pi / 180.0
            pos = np.array([math.cos(yaw), math.sin(yaw), 1.5]) + rng.uniform(-0.05, 0.05, 3)
            axes = np.array([[math.sin(yaw), -math.cos(yaw), 0.0], [0.0, 0.0, -1.0],
                             [math.cos(yaw), math.sin(yaw), 0.0]])   # right, down, forward
            R = _rotation("z", roll) @ _rotation("x", pitch) @ _rotation("y", turn) @ axes
            out[b, n, :3, :3] = K @ R
            out[b, n, :3, 3] = -(K @ R @ pos)
            out[b, n, 3, 3] = 1.0
    return out


def _levels(case):
    h, w, out = case["H"], case["W"], []
    for _ in range(case["L"]):
        out.append((h, w))
        h, w = -(-h // 2), -(-w // 2)
    return tuple(out)


def _heights(case):
    Z, lo, hi = case["Z"], case["z_lo"], case["z_hi"]
    if case["op"].startswith("vt"):   # centres of Z equal bins
        z = lo + (np.arange(Z) + 0.5) * (hi - lo) / Z
    else:                             # pillar anchors, half a metre inside the ends
        z = lo + 0.5 + np.arange(Z) * ((hi - lo) - 1.0) / max(1, Z - 1)
    return z.astype(np.float32)


def _grid(case):
    half = case["half"]
    return fb.BevGrid(-half, 2.0 * half / case["X"], case["X"], -half, 2.0 * half / case["Y"],
                      case["Y"])


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    dt = _DTYPES[case["dtype"]]
    B, N, C, X, Y = case["B"], case["N"], case["C"], case["X"], case["Y"]
    train = case["op"].endswith("train")

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev)

    st = {"op": case["op"], "reduce": case["reduce"], "grid": _grid(case), "z": _heights(case),
          "img_hw": (case["img_h"], case["img_w"]),
          "lidar2img": torch.from_numpy(_rig(case, seed)).to(dev)}
    if case["op"].startswith("vt"):
        st["features"] = normal(B, N, case["H"], case["W"], C).to(dt).requires_grad_(train)
        if train:
            st["grad_out"] = normal(B, C, X, Y)
        return st
    heads, L, P, Q = case["heads"], case["L"], case["P"], X * Y
    levels = _levels(case)
    st["levels"], st["heads"] = levels, heads
    S = sum(h * w for h, w in levels)
    st["value"] = normal(B, N, S, C).to(dt).requires_grad_(train)
    # head m's points lie along angle 2 pi m / heads, point k at k + 1 pixels
    th = 2.0 * math.pi * torch.arange(heads, device=dev) / heads
    d = torch.stack([th.cos(), th.sin()], -1)
    d = d / d.abs().amax(-1, keepdim=True)
    k = torch.arange(P, device=dev) + 1.0
    base = d[:, None, None, :] * k[None, None, :, None]
    st["offsets"] = (base + normal(B, Q, heads, L, P, 2)).requires_grad_(train)
    st["logits"] = normal(B, Q, heads, L, P).requires_grad_(train)
    if train:
        st["grad_out"] = normal(B, Q, C)
    return st


def run(st):
    op = st["op"]
    if op == "vt_forward":
        return fb.sample_vt(st["features"], st["lidar2img"], st["z"], st["grid"], st["img_hw"],
                            reduce=st["reduce"])
    if op == "vt_train":
        out = fb.sample_vt_autograd(st["features"], st["lidar2img"], st["z"], st["grid"],
                                    st["img_hw"], reduce=st["reduce"])
        (g,) = torch.autograd.grad(out, [st["features"]], st["grad_out"])
        return {"out": out.detach(), "grad_features": g}
    if op == "sca_forward":
        return fb.sca_forward(st["value"], st["lidar2img"], st["z"], st["grid"], st["img_hw"],
                              st["levels"], st["heads"], st["offsets"], st["logits"],
                              reduce=st["reduce"])
    out = fb.sca_autograd(st["value"], st["lidar2img"], st["z"], st["grid"], st["img_hw"],
                          st["levels"], st["heads"], st["offsets"], st["logits"],
                          reduce=st["reduce"])
    gv, go, gl = torch.autograd.grad(out, [st["value"], st["offsets"], st["logits"]],
                                     st["grad_out"])
    return {"out": out.detach(), "grad_value": gv, "grad_offsets": go, "grad_logits": gl}


# ---- what a pass cannot do without -----------------------------------------------------------

# Shares that the ring rig gives: samples inside an image per (voxel, camera)
# and cameras per query.
_VALID = 0.17
_HITS = 1.1


def work(case):
    B, N, C, X, Y, Z = (case[k] for k in ("B", "N", "C", "X", "Y", "Z"))
    es = _BYTES[case["dtype"]]
    train = case["op"].endswith("train")
    if case["op"].startswith("vt"):
        feat, out = B * N * case["H"] * case["W"] * C, B * C * X * Y
        nbytes = feat * es + 64 * B * N + out * 4
        # a projection per (voxel, camera), four multiply-adds per channel and valid sample
        flops = B * X * Y * Z * N * (30 + _VALID * 8 * C)
        if train:
            nbytes += out * 4 + feat * es
            flops += B * X * Y * Z * N * _VALID * 8 * C
        return {"bytes": nbytes, "flops": flops}
    S = sum(h * w for h, w in _levels(case))
    val, out = B * N * S * C, B * X * Y * C
    pts = B * X * Y * case["heads"] * case["L"] * case["P"]
    nbytes = val * es + 64 * B * N + pts * 12 + out * 4
    flops = pts * _HITS * 8 * (C // case["heads"])
    if train:   # the value gradient, and the dot products of every tap with the output gradient
        nbytes += out * 4 + val * es + pts * 12
        flops *= 3
    return {"bytes": nbytes, "flops": flops}


def _cost(case):
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / 2e13


def tolerance(case):
    """Measured against ``exact``: float32 outputs are 1e-7 to 5e-7 off (the sums
    of many heights most), at most 8e-6 of a value; four times that and more."""
    if case["op"].endswith("train") and case["dtype"] != "f32":
        # the feature or value gradient is rounded once to the features' type:
        # 1.7e-3 (bfloat16) and 2.1e-4 (half) off
        return {"rel": 7e-3, "max": 1.6e-2} if case["dtype"] == "bf16" else {"rel": 9e-4, "max": 2e-3}
    return {"rel": 2e-6, "max": 5e-5}


# ---- the same results in 64 bits -------------------------------------------------------------


def _r(t):
    """Round float64 values to float32 (kept as float64)."""
    return t.float().double()


def _f32(v):
    return float(np.float32(v))


def _centres(case, dev):
    g = _grid(case)
    i = torch.arange(case["X"], device=dev, dtype=torch.float64) + 0.5
    j = torch.arange(case["Y"], device=dev, dtype=torch.float64) + 0.5
    x = _r(_f32(g.x_min) + _r(i * _f32(g.dx)))
    y = _r(_f32(g.y_min) + _r(j * _f32(g.dy)))
    return (x[:, None].expand(case["X"], case["Y"]).reshape(-1),
            y[None, :].expand(case["X"], case["Y"]).reshape(-1))


def _project(m, x, y, z):
    """Rows 0..2 of one matrix times (x, y, z, 1), every step rounded to float32."""
    return [_r(_r(_r(_r(m[k][0] * x) + _r(m[k][1] * y)) + _f32(_f32(m[k][2]) * z)) + m[k][3])
            for k in range(3)]


def _taps(xf, yf, W, H):
    """The four bilinear corners: (column, row, weight, d weight/dx, d weight/dy, in range)."""
    x0, y0 = xf.floor(), yf.floor()
    ax, ay = xf - x0, yf - y0
    for ty in (0, 1):
        for tx in (0, 1):
            c, r = x0.long() + tx, y0.long() + ty
            wx, wy = (ax if tx else 1.0 - ax), (ay if ty else 1.0 - ay)
            ok = (c >= 0) & (c < W) & (r >= 0) & (r < H)
            yield c, r, wx * wy, (wy if tx else -wy), (wx if ty else -wx), ok


_ROWS = 1 << 20   # gathered rows held in float64 at a time


def _exact_vt(case, st):
    dev = st["features"].device
    B, N, C, H, W = (case[k] for k in ("B", "N", "C", "H", "W"))
    X, Y, Z = case["X"], case["Y"], case["Z"]
    ih, iw = case["img_h"], case["img_w"]
    sx, sy = _f32(np.float32(W) / np.float32(iw)), _f32(np.float32(H) / np.float32(ih))
    eps = _f32(st["grid"].depth_eps)
    x, y = _centres(case, dev)
    mats = st["lidar2img"].double().cpu().tolist()
    feats = st["features"].detach()
    out = torch.zeros(B, X * Y, C, dtype=torch.float64, device=dev)
    train = case["op"] == "vt_train"
    if train:
        grad = torch.zeros(B, N, H * W, C, dtype=torch.float64, device=dev)
        gout = st["grad_out"].reshape(B, C, X * Y).transpose(1, 2).double().contiguous()
    for b in range(B):
        for z in st["z"].tolist():
            seen = []
            den = torch.zeros(X * Y, dtype=torch.float64, device=dev)
            for n in range(N):
                up, vp, d = _project(mats[b][n], x, y, z)
                u, v = _r(up / d), _r(vp / d)
                idx = torch.nonzero((d > eps) & (u >= 0) & (u < iw) & (v >= 0) & (v < ih))[:, 0]
                den[idx] += 1.0
                seen.append((n, idx, _r(_r(u[idx] * sx) - 0.5), _r(_r(v[idx] * sy) - 0.5)))
            mean = 1.0 / den.clamp(min=1.0) if case["reduce"] == "mean" else torch.ones_like(den)
            for n, idx, xf, yf in seen:
                fm = feats[b, n].reshape(H * W, C)
                for c, r, w, _, _, ok in _taps(xf, yf, W, H):
                    at = torch.nonzero(ok)[:, 0]
                    for k in range(0, at.numel(), _ROWS):
                        a = at[k:k + _ROWS]
                        cell, pix = idx[a], (r * W + c)[a]
                        f = (w[a] * mean[cell])[:, None]
                        out[b, cell] += f * fm[pix].double()   # each cell once
                        if train:
                            grad[b, n].index_add_(0, pix, f * gout[b][cell])
    out = out.transpose(1, 2).reshape(B, C, X, Y)
    if not train:
        return out
    return {"out": out, "grad_features": grad.reshape(B, N, H, W, C)}


def _exact_sca(case, st):
    dev = st["value"].device
    B, N, C, X, Y, Z = (case[k] for k in ("B", "N", "C", "X", "Y", "Z"))
    heads, L, P, Q = case["heads"], case["L"], case["P"], X * Y
    D, iw, ih = C // heads, float(case["img_w"]), float(case["img_h"])
    eps = _f32(st["grid"].depth_eps)
    x, y = _centres(case, dev)
    mats = st["lidar2img"].double().cpu().tolist()
    value = st["value"].detach()
    offsets = st["offsets"].detach()
    att = torch.softmax(st["logits"].detach().double().reshape(B, Q, heads, L * P), -1)
    att = att.reshape(B, Q, heads, L, P)
    out = torch.zeros(B, Q, heads, D, dtype=torch.float64, device=dev)
    train = case["op"] == "sca_train"
    if train:
        S = value.shape[2]
        gval = torch.zeros(B, N, S * heads, D, dtype=torch.float64, device=dev)
        goff = torch.zeros(B, Q, heads, L, P, 2, dtype=torch.float64, device=dev)
        gatt = torch.zeros(B, Q, heads, L, P, dtype=torch.float64, device=dev)
        gout = st["grad_out"].double().reshape(B, Q, heads, D)
    hm = torch.arange(heads, device=dev)
    for b in range(B):
        ref, hit = {}, {}
        for n in range(N):
            hit[n] = torch.zeros(Q, dtype=torch.bool, device=dev)
            for k, z in enumerate(st["z"].tolist()):
                up, vp, d = _project(mats[b][n], x, y, z)
                front = d > eps
                dd = torch.where(front, d, torch.full_like(d, eps))
                un, vn = _r(_r(up / dd) / iw), _r(_r(vp / dd) / ih)
                ref[n, k] = (un, vn)
                hit[n] |= front & (un > 0) & (un < 1) & (vn > 0) & (vn < 1)
        count = sum(h.double() for h in hit.values())
        mean = 1.0 / count.clamp(min=1.0) if case["reduce"] == "mean" else torch.ones_like(count)
        for n in range(N):
            q = torch.nonzero(hit[n])[:, 0]
            vm = value[b, n].reshape(-1, D)   # row = pixel * heads + head
            start = 0
            for lv, (Hl, Wl) in enumerate(_levels(case)):
                for k in range(P):
                    un, vn = ref[n, k % Z]
                    o = offsets[b, q, :, lv, k, :].double()   # [q, heads, 2]
                    xf = _r(_r(_r(un[q] * Wl)[:, None] + o[..., 0]) - 0.5)
                    yf = _r(_r(_r(vn[q] * Hl)[:, None] + o[..., 1]) - 0.5)
                    inside = (xf > -1) & (xf < Wl) & (yf > -1) & (yf < Hl)
                    xf, yf = torch.where(inside, xf, -2.0), torch.where(inside, yf, -2.0)
                    a = att[b, q, :, lv, k] * mean[q][:, None]
                    for c, r, w, wdx, wdy, ok in _taps(xf, yf, Wl, Hl):
                        row = ((start + r * Wl + c) * heads + hm).clamp(min=0)
                        row = torch.where(ok, row, torch.zeros_like(row))
                        v = vm[row].double()                  # [q, heads, D]
                        okf = ok.double()
                        out[b, q] += (a * w * okf)[..., None] * v
                        if train:
                            G = gout[b, q]
                            gval[b, n].index_add_(0, row.reshape(-1),
                                                  ((a * w * okf)[..., None] * G).reshape(-1, D))
                            dot = (v * G).sum(-1) * okf
                            gatt[b, q, :, lv, k] += mean[q][:, None] * w * dot
                            goff[b, q, :, lv, k, 0] += a * wdx * dot
                            goff[b, q, :, lv, k, 1] += a * wdy * dot
                start += Hl * Wl
    out = out.reshape(B, Q, C)
    if not train:
        return out
    s = (att * gatt).sum((-1, -2), keepdim=True)
    return {"out": out, "grad_value": gval.reshape(B, N, -1, C), "grad_offsets": goff,
            "grad_logits": att * (gatt - s)}


def exact(case, seed):
    st = prepare(case, seed)
    with torch.no_grad():
        return _exact_vt(case, st) if case["op"].startswith("vt") else _exact_sca(case, st)
