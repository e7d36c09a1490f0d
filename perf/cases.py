"""Performance cases: what users of this library run, through its public entry points.

The listed cases are the library's own workloads (the single-image call, the convolution sweep, the
unsigned char setting, corner detection, the uneven batch, the filter bank's training step, the volume)
at their configured sizes, beside odd sizes, half storage, both boundaries and a small training step.
``draw`` spreads sizes, radii, types and boundaries over the ranges between them.  Calls are made
as a program makes them that has not searched for variants first: the library's own choice runs.

A case is a dict of plain values; ``prepare`` builds its inputs on the GPU from a seed, ``run`` makes one
pass, ``work`` counts the bytes and operations that the result cannot do without, ``exact`` gives the same
outputs in 64 bits from plain torch.
"""
import numpy as np
import torch
import torch.nn.functional as nnf

from paper_1605_06399_amd import synth
from paper_1605_06399_amd import torch_api as T

_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_SIZE = {"f32": 4, "f16": 2, "bf16": 2}
HARRIS_K, NMS_TAU = 0.04, 1e-3


def listed():
    return [
        # one small photo or thumbnail smoothed with a 5-tap Gaussian: launch and call latency
        {"name": "sep_512_r2_f32", "op": "sep", "w": 512, "h": 512, "r": 2, "dtype": "f32", "border": "clamp"},
        # the sweep's widest separable filter on its 4096 x 4096 image
        {"name": "sep_4096_r7_f32", "op": "sep", "w": 4096, "h": 4096, "r": 7, "dtype": "f32", "border": "clamp"},
        # half storage, odd width (rows not 4-pixel aligned), constant boundary
        {"name": "sep_3001x1999_r3_bf16", "op": "sep", "w": 3001, "h": 1999, "r": 3, "dtype": "bf16",
         "border": "constant"},
        # the sweep's widest 2-D filter: 225 taps per pixel
        {"name": "conv2d_4096_r7_f32", "op": "conv2d", "w": 4096, "h": 4096, "r": 7, "dtype": "f32",
         "border": "clamp"},
        # a video-sized frame in half storage, odd in both directions
        {"name": "conv2d_1921x1083_r3_f16", "op": "conv2d", "w": 1921, "h": 1083, "r": 3, "dtype": "f16",
         "border": "clamp"},
        # the 8-bit setting: 8192 x 8192 bytes, 5 x 5 integer taps
        {"name": "u8_8192_r2", "op": "u8", "w": 8192, "h": 8192, "r": 2, "border": "clamp"},
        # corner detection of a large image, mask only
        {"name": "corners_8192", "op": "corners", "w": 8192, "h": 8192, "r": 2},
        # corner detection of an odd frame as two calls, where the response is wanted too
        {"name": "harris_nms_1919x1081", "op": "harris_nms", "w": 1919, "h": 1081, "r": 2},
        # 256 uneven images in one captured launch
        {"name": "batch_256_f16", "op": "batch", "count": 256, "side_lo": 64, "side_hi": 2048, "dtype": "f16",
         "graph": True},
        # training step of the filter bank (forward with the loss, both gradients) at its configured size
        {"name": "bank_step_32x16x1024_r4", "op": "bank_step", "n": 32, "f": 16, "h": 1024, "w": 1024, "r": 4},
        # a small bank used as a layer: forward, then both gradients from an upstream gradient
        {"name": "bank_layer_4x8x201_r2", "op": "bank_layer", "n": 4, "f": 8, "h": 201, "w": 200, "r": 2},
        # a volume, separable in three directions
        {"name": "conv3d_256_r2_f32", "op": "conv3d", "w": 256, "h": 256, "d": 256, "r": 2, "dtype": "f32",
         "border": "clamp"},
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    op = rng.choice(["sep", "conv2d", "u8", "corners", "harris_nms", "batch", "bank_step", "bank_layer", "conv3d"])
    if op in ("sep", "conv2d"):
        return {"op": op, "w": _log(rng, 256, 4096), "h": _log(rng, 256, 4096), "r": rng.randint(1, 7),
                "dtype": rng.choice(["f32", "f32", "f16", "bf16"]), "border": rng.choice(["clamp", "constant"])}
    if op == "u8":
        return {"op": op, "w": _log(rng, 512, 8192), "h": _log(rng, 512, 8192), "r": rng.randint(1, 5),
                "border": rng.choice(["clamp", "constant"])}
    if op in ("corners", "harris_nms"):
        return {"op": op, "w": _log(rng, 512, 8192), "h": _log(rng, 512, 8192), "r": rng.randint(1, 3)}
    if op == "batch":
        return {"op": op, "count": _log(rng, 8, 256), "side_lo": 64, "side_hi": _log(rng, 256, 2048),
                "dtype": rng.choice(["f16", "bf16"]), "graph": rng.random() < 0.5}
    if op == "conv3d":
        return {"op": op, "w": _log(rng, 64, 256), "h": _log(rng, 64, 256), "d": _log(rng, 64, 256),
                "r": rng.randint(1, 3), "dtype": rng.choice(["f32", "f32", "f16", "bf16"]),
                "border": rng.choice(["clamp", "constant"])}
    if op == "bank_step":
        return {"op": op, "n": _log(rng, 2, 32), "f": rng.randint(4, 16), "h": _log(rng, 128, 1024),
                "w": _log(rng, 128, 1024), "r": rng.randint(2, 4)}
    return {"op": op, "n": _log(rng, 1, 16), "f": rng.randint(2, 16), "h": _log(rng, 64, 512),
            "w": _log(rng, 64, 512), "r": rng.randint(1, 4)}


# ----------------------------------------------------------------------------- inputs

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 16 + stream) % (1 << 62))
    return g


def _uniform(seed, stream, shape, dtype=torch.float32):
    return torch.rand(shape, generator=_gen(seed, stream), device="cuda").to(dtype)


def _taps(seed, stream, count):
    return torch.from_numpy(synth.normal_taps_normalised(seed, count, stream=stream)).cuda()


def _rectangles(seed, h, w):
    """U[0,1) noise with up to 64 brighter rectangles (the corner workload's image)."""
    x = _uniform(seed, 0, (h, w))
    inside = torch.zeros((h, w), dtype=torch.bool, device="cuda")
    u = np.random.RandomState(seed % (1 << 32)).rand(64, 4)
    for a, b, c, d in u:
        x0, y0 = int(a * w), int(b * h)
        inside[y0:y0 + 16 + int(d * 497), x0:x0 + 16 + int(c * 497)] = True
    return x + inside.to(torch.float32)


def _batch_items(case):
    """(width, height, radius, row pitch in pixels) of each image of the batch: a case's images keep their
    sizes, its seeds change their pixels."""
    rs = np.random.RandomState(case["count"] * 4099 + case["side_hi"])
    items = []
    for _ in range(case["count"]):
        w, h = (int(v) for v in rs.randint(case["side_lo"], case["side_hi"] + 1, 2))
        items.append((w, h, int(rs.randint(1, 8)), (w + 127) // 128 * 128))
    return items


def prepare(case, seed):
    op = case["op"]
    if op in ("sep", "conv2d"):
        r, n = case["r"], 2 * case["r"] + 1
        x = _uniform(seed, 0, (case["h"], case["w"]), _DT[case["dtype"]])
        s = {"op": op, "x": x, "out": torch.empty_like(x), "border": case["border"],
             "constant": 0.0 if case["border"] == "clamp" else 0.25}
        if op == "sep" and case["w"] * case["h"] <= 1 << 18:   # a small image: the smoothing Gaussian
            g = torch.from_numpy(synth.gaussian_taps(r, max(1.0, r / 2.0))).cuda()
            s["taps"] = (g, g)
        elif op == "sep":
            s["taps"] = (_taps(seed, 1, n), _taps(seed, 2, n))
        else:
            s["taps"] = _taps(seed, 1, n * n).reshape(n, n)
        return s
    if op == "u8":
        x = torch.randint(0, 256, (case["h"], case["w"]), generator=_gen(seed, 0), device="cuda", dtype=torch.uint8)
        return {"op": op, "x": x, "out": torch.empty_like(x), "border": case["border"],
                "constant": 0 if case["border"] == "clamp" else 64,
                "taps": torch.from_numpy(synth.u8_taps(seed, case["r"], synth.U8_SHIFT)).cuda()}
    if op in ("corners", "harris_nms"):
        x = _rectangles(seed, case["h"], case["w"])
        s = {"op": op, "x": x, "mask": torch.empty(x.shape, dtype=torch.uint8, device="cuda"),
             "taps": torch.from_numpy(synth.gaussian_taps(case["r"], max(1.0, case["r"] / 2.0))).cuda()}
        if op == "harris_nms":
            s["resp"] = torch.empty_like(x)
        return s
    if op == "batch":
        items = _batch_items(case)
        total = sum(h * p for _, h, _, p in items)
        src = _uniform(seed, 0, (total,), _DT[case["dtype"]])
        dst = torch.zeros(total, dtype=_DT[case["dtype"]], device="cuda")
        taps = {r: torch.from_numpy(synth.gaussian_taps(r, r / 2.0)).cuda() for r in range(1, 8)}
        images, outputs, per, at = [], [], [], 0
        for w, h, r, p in items:
            images.append(src[at:at + h * p].view(h, p)[:, :w])
            outputs.append(dst[at:at + h * p].view(h, p)[:, :w])
            per.append(taps[r])
            at += h * p
        plan = T.BatchPlan(images, outputs, per)
        if case["graph"]:
            plan.graph()
        return {"op": op, "plan": plan, "src": src, "dst": dst, "graph": case["graph"]}
    if op in ("bank_step", "bank_layer"):
        n, f, h, w, k = case["n"], case["f"], case["h"], case["w"], 2 * case["r"] + 1
        s = {"op": op, "x": _uniform(seed, 0, (n, 1, h, w)).requires_grad_(True),
             "w": (0.1 * torch.randn((f, k, k), generator=_gen(seed, 1), device="cuda")).requires_grad_(True)}
        if op == "bank_step":
            s["t"] = _uniform(seed, 2, (n, f, h, w))
        else:
            s["gy"] = torch.randn((n, f, h, w), generator=_gen(seed, 2), device="cuda")
        return s
    r, n = case["r"], 2 * case["r"] + 1
    x = _uniform(seed, 0, (case["d"], case["h"], case["w"]), _DT[case["dtype"]])
    g = torch.from_numpy(synth.gaussian_taps(r, max(1.0, r / 2.0))).cuda()
    return {"op": op, "x": x, "out": torch.empty_like(x), "taps": g, "border": case["border"],
            "constant": 0.0 if case["border"] == "clamp" else 0.25}


# ----------------------------------------------------------------------------- one pass

def run(state):
    op = state["op"]
    if op == "sep":
        return T.conv_sep(state["x"], *state["taps"], out=state["out"], border=state["border"],
                          constant=state["constant"])
    if op == "conv2d":
        return T.conv2d(state["x"], state["taps"], out=state["out"], border=state["border"],
                        constant=state["constant"])
    if op == "u8":
        return T.conv2d_u8(state["x"], state["taps"], synth.U8_SHIFT, out=state["out"], border=state["border"],
                           constant=state["constant"])
    if op == "corners":
        return T.corners(state["x"], state["taps"], k=HARRIS_K, threshold=NMS_TAU, out=state["mask"])
    if op == "harris_nms":
        resp = T.harris(state["x"], state["taps"], k=HARRIS_K, out=state["resp"])
        return resp, T.nms(resp, NMS_TAU, out=state["mask"])
    if op == "batch":
        if state["graph"]:
            state["plan"].replay()
        else:
            state["plan"].launch()
        return state["dst"]
    if op == "bank_step":
        loss = T.filter_bank_loss(state["x"], state["w"], state["t"])
        gx, gw = torch.autograd.grad(loss, (state["x"], state["w"]))
        return loss.detach(), gx, gw
    if op == "bank_layer":
        y = T.filter_bank(state["x"], state["w"])
        gx, gw = torch.autograd.grad(y, (state["x"], state["w"]), state["gy"])
        return y.detach(), gx, gw
    return T.conv3d_sep(state["x"], state["taps"], state["taps"], state["taps"], out=state["out"],
                        border=state["border"], constant=state["constant"])


# ----------------------------------------------------------------------------- what a pass cannot do without

def work(case):
    op = case["op"]
    if op == "batch":
        items = _batch_items(case)
        return {"bytes": sum(2 * _SIZE[case["dtype"]] * w * h for w, h, _, _ in items),
                "flops": sum(4 * (2 * r + 1) * w * h for w, h, r, _ in items)}
    r, n = case["r"], 2 * case["r"] + 1
    if op in ("bank_step", "bank_layer"):
        px, taps = case["n"] * case["h"] * case["w"], case["f"] * n * n
        big = px * case["f"]
        # step: x, w and the target in, both gradients out; layer: x, w and the upstream gradient in,
        # the output and both gradients out
        return {"bytes": 4 * (2 * px + 2 * taps + (big if op == "bank_step" else 2 * big)), "flops": 3 * 2 * px * taps}
    px = case["w"] * case["h"]
    if op == "sep":
        return {"bytes": 2 * _SIZE[case["dtype"]] * px, "flops": px * 4 * n}
    if op == "conv2d":
        return {"bytes": 2 * _SIZE[case["dtype"]] * px, "flops": px * 2 * n * n}
    if op == "u8":
        return {"bytes": 2 * px, "flops": px * 2 * n * n}
    if op in ("corners", "harris_nms"):
        # Sobel, three products, a separable window of each, the response, the comparisons
        return {"bytes": (5 if op == "corners" else 9) * px, "flops": px * (18 + 3 + 3 * 4 * n + 8 + 9)}
    px *= case["d"]
    return {"bytes": 2 * _SIZE[case["dtype"]] * px, "flops": px * 6 * n}


# ----------------------------------------------------------------------------- the same in 64 bits

def _pad(x, pads, border, constant):
    """x (float64, 2-D or 3-D) extended by its boundary condition; pads: the last dimension's pair first."""
    if border == "constant":
        return nnf.pad(x, pads, value=constant)
    return nnf.pad(x[None, None], pads, mode="replicate")[0, 0]


def _window(p, taps, dim, size):
    """sum_i taps[i] * p shifted by i along dim, `size` results."""
    return sum(float(c) * p.narrow(dim, i, size) for i, c in enumerate(taps.tolist()))


def _sep64(x, tx, ty, r, border, constant):
    h, w = x.shape
    p = _pad(x.double(), (r, r, r, r), border, constant)
    return _window(_window(p, tx, 1, w), ty, 0, h)


def _harris64(x, g, r):
    h, w = x.shape
    p = _pad(x.double(), (1, 1, 1, 1), "clamp", 0.0)
    s, d = torch.tensor([1.0, 2.0, 1.0]), torch.tensor([-1.0, 0.0, 1.0])
    ix, iy = _window(_window(p, d, 1, w), s, 0, h), _window(_window(p, s, 1, w), d, 0, h)
    sxx, syy, sxy = (_sep64(v, g, g, r, "clamp", 0.0) for v in (ix * ix, iy * iy, ix * iy))
    return sxx * syy - sxy * sxy - float(np.float32(HARRIS_K)) * (sxx + syy) ** 2


def _fold(z, dim, r):
    """Adds the r padded positions beyond each end of dim onto its first and last element."""
    size = z.shape[dim] - 2 * r
    z.narrow(dim, r, 1).add_(z.narrow(dim, 0, r).sum(dim, keepdim=True))
    z.narrow(dim, r + size - 1, 1).add_(z.narrow(dim, r + size, r).sum(dim, keepdim=True))
    return z.narrow(dim, r, size)


def _bank64(s, case):
    """(y or loss, gx, gw): one image at a time, taps as matrix products."""
    n, f, h, w, r = case["n"], case["f"], case["h"], case["w"], case["r"]
    k = 2 * r + 1
    x, wt = s["x"].detach(), s["w"].detach().double().reshape(f, k * k)
    gw = torch.zeros((f, k * k), dtype=torch.float64, device="cuda")
    gx = torch.empty((n, 1, h, w), dtype=torch.float64, device="cuda")
    y_all, loss = [], torch.zeros((), dtype=torch.float64, device="cuda")
    for i in range(n):
        p = _pad(x[i, 0].double(), (r, r, r, r), "clamp", 0.0)
        col = torch.stack([p[j:j + h, m:m + w] for j in range(k) for m in range(k)]).reshape(k * k, h * w)
        y = wt @ col
        if case["op"] == "bank_step":
            diff = y - s["t"][i].double().reshape(f, h * w)
            loss += (diff * diff).sum()
            gy = 2.0 * diff
        else:
            y_all.append(y.reshape(f, h, w))
            gy = s["gy"][i].double().reshape(f, h * w)
        gw += gy @ col.t().contiguous()
        back = (wt.t().contiguous() @ gy).reshape(k, k, h, w)
        z = torch.zeros_like(p)
        for j in range(k):
            for m in range(k):
                z[j:j + h, m:m + w] += back[j, m]
        gx[i, 0] = _fold(_fold(z, 0, r), 1, r)
    first = loss if case["op"] == "bank_step" else torch.stack(y_all)
    return first, gx, gw.reshape(f, k, k)


def exact(case, seed):
    op = case["op"]
    if op in ("u8", "corners"):
        return None
    s = prepare(case, seed)
    if op == "sep":
        return _sep64(s["x"], *s["taps"], case["r"], s["border"], s["constant"])
    if op == "conv2d":
        r = case["r"]
        p = _pad(s["x"].double(), (r, r, r, r), s["border"], s["constant"])
        return sum(_window(p.narrow(0, j, case["h"]), s["taps"][j], 1, case["w"]) for j in range(2 * r + 1))
    if op == "harris_nms":
        return _harris64(s["x"], s["taps"], case["r"]), None
    if op == "batch":
        out, at = torch.zeros(s["src"].shape, dtype=torch.float64, device="cuda"), 0
        for w, h, r, p in _batch_items(case):
            g = torch.from_numpy(synth.gaussian_taps(r, r / 2.0))
            out[at:at + h * p].view(h, p)[:, :w] = _sep64(s["src"][at:at + h * p].view(h, p)[:, :w], g, g, r,
                                                          "clamp", 0.0)
            at += h * p
        return out
    if op in ("bank_step", "bank_layer"):
        return _bank64(s, case)
    r, (d, h, w) = case["r"], s["x"].shape
    p = _pad(s["x"].double(), (r,) * 6, s["border"], s["constant"])
    g = s["taps"]
    return _window(_window(_window(p, g, 2, w), g, 1, h), g, 0, d)
