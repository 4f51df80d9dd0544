"""Workloads of the median filter whose speed is followed.

Every case goes through the public entry points of
``paper_2507_19926_amd.ops`` the way a program calls them: inputs resident on
the GPU, one call per pass. ``listed`` holds the fixed cases, ``draw`` makes
further ones of the same ranges, ``prepare`` the inputs of a case, ``run`` one
pass, ``work`` the traffic a pass cannot do without and ``exact`` the result
by plain torch (selection, so the values are exact in any precision).

Integer images are uniform noise, except ``rgb`` images (smooth gradients with
5 % salt-and-pepper, in place of photographs); float images are N(0.5, 0.2)
with 2 % outliers at +-10.
"""
from __future__ import annotations

import math

import torch

from paper_2507_19926_amd import ops

_DTYPES = {"u8": torch.uint8, "u16": torch.uint16, "u32": torch.uint32, "f32": torch.float32}
_SIZE = {"u8": 1, "u16": 2, "u32": 4, "f32": 4}


def listed():
    return [
        # one small image: launch latency
        {"name": "u8_512_k3", "kind": "plane", "data": "noise", "dtype": "u8", "planes": 1, "h": 512, "w": 512,
         "kw": 3, "kh": 3},
        # an ordinary image of odd size at a denoising radius
        {"name": "u8_765x1021_k25", "kind": "plane", "data": "rgb", "dtype": "u8", "planes": 1, "h": 765,
         "w": 1021, "kw": 25, "kh": 25},
        # 30-megapixel photographs, three 8-bit planes: salt-and-pepper removal,
        # denoising, and the largest window (background estimation)
        {"name": "u8_rgb30_k3", "kind": "plane", "data": "rgb", "dtype": "u8", "planes": 3, "h": 4480, "w": 6720,
         "kw": 3, "kh": 3},
        {"name": "u8_rgb30_k17", "kind": "plane", "data": "rgb", "dtype": "u8", "planes": 3, "h": 4480, "w": 6720,
         "kw": 17, "kh": 17},
        {"name": "u8_rgb30_k75", "kind": "plane", "data": "rgb", "dtype": "u8", "planes": 3, "h": 4480, "w": 6720,
         "kw": 75, "kh": 75},
        # a 16-bit detector or microscope frame, background window
        {"name": "u16_4096_k35", "kind": "plane", "data": "noise", "dtype": "u16", "planes": 1, "h": 4096,
         "w": 4096, "kw": 35, "kh": 35},
        # float data: a small window on a large frame, a larger one on a ragged frame
        {"name": "f32_4096_k7", "kind": "plane", "data": "noise", "dtype": "f32", "planes": 1, "h": 4096,
         "w": 4096, "kw": 7, "kh": 7},
        {"name": "f32_1531x2049_k25", "kind": "plane", "data": "noise", "dtype": "f32", "planes": 1, "h": 1531,
         "w": 2049, "kw": 25, "kh": 25},
        # a rectangular window (stripe removal) on the photograph
        {"name": "u8_rgb30_21x13", "kind": "plane", "data": "rgb", "dtype": "u8", "planes": 3, "h": 4480,
         "w": 6720, "kw": 21, "kh": 13},
        # a volume (tomography), 3-D box
        {"name": "volume_u8_256_k5", "kind": "volume", "dtype": "u8", "d": 256, "h": 256, "w": 256, "k": 5},
        # serving: 256 images of mixed sizes, windows and types in one plan
        {"name": "batch_256_mixed", "kind": "batch", "n": 256, "lo": 64, "hi": 2048, "kmax": 25},
        # a differentiable layer: forward and backward of a batch of float images
        {"name": "autograd_32x3x512_k7", "kind": "autograd", "n": 32, "c": 3, "h": 512, "w": 512, "k": 7},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("plane",) * 6 + ("rect",) * 2 + ("volume", "batch", "autograd", "autograd"))
    if kind == "volume":
        return {"kind": kind, "dtype": rng.choice(("u8", "u8", "u16", "f32")), "d": rng.randint(24, 256),
                "h": rng.randint(32, 256), "w": rng.randint(32, 256), "k": rng.choice((3, 5, 7))}
    if kind == "batch":
        return {"kind": kind, "n": rng.randint(8, 256), "lo": 64, "hi": _log(rng, 256, 2048),
                "kmax": rng.randrange(5, 27, 2)}
    if kind == "autograd":
        return {"kind": kind, "n": rng.randint(1, 32), "c": rng.choice((1, 3)), "h": _log(rng, 33, 512),
                "w": _log(rng, 33, 512), "k": rng.randrange(3, 17, 2)}
    dtype = rng.choice(("u8", "u8", "u8", "u16", "f32", "f32", "u32"))
    hi_h, hi_w = (4480, 6720) if dtype == "u8" else (3072, 3072)
    case = {"kind": "plane", "data": rng.choice(("noise", "rgb")) if dtype == "u8" else "noise", "dtype": dtype,
            "planes": rng.choice((1, 1, 3)) if dtype == "u8" else 1, "h": _log(rng, 96, hi_h),
            "w": _log(rng, 96, hi_w)}
    if kind == "rect":
        kw = rng.randrange(1, 33, 2)
        case["kw"], case["kh"] = kw, rng.choice([s for s in range(1, 33, 2) if s != kw])
    else:
        case["kw"] = case["kh"] = rng.randrange(3, 77, 2)
    return case


def _plane(gen, data, dtype, planes, h, w):
    """(planes, h, w) on the GPU ((h, w) for one plane)."""
    if data == "rgb":
        y = torch.arange(h, device="cuda", dtype=torch.float32)[:, None] / max(h - 1, 1)
        x = torch.arange(w, device="cuda", dtype=torch.float32)[None, :] / max(w - 1, 1)
        ramps = (x.expand(h, w), y.expand(h, w), (x * w + y * h) / (h + w))
        t = torch.stack([(255.0 * ramps[c % 3]).round().to(torch.uint8) for c in range(planes)])
        u = torch.rand(t.shape, generator=gen, device="cuda")
        t = torch.where(u < 0.025, torch.zeros_like(t), torch.where(u > 0.975, torch.full_like(t, 255), t))
    else:
        shape = (planes, h, w)
        if dtype == "f32":
            t = 0.5 + 0.2 * torch.randn(shape, generator=gen, device="cuda")
            u = torch.rand(shape, generator=gen, device="cuda")
            t = torch.where(u < 0.01, torch.full_like(t, -10.0), torch.where(u > 0.99, torch.full_like(t, 10.0), t))
        elif dtype == "u8":
            t = torch.randint(0, 256, shape, generator=gen, device="cuda", dtype=torch.uint8)
        elif dtype == "u16":
            t = torch.randint(-(1 << 15), 1 << 15, shape, generator=gen, device="cuda",
                              dtype=torch.int16).view(torch.uint16)
        else:
            t = torch.randint(-(1 << 31), 1 << 31, shape, generator=gen, device="cuda",
                              dtype=torch.int64).to(torch.int32).view(torch.uint32)
    return t[0] if planes == 1 else t


def _batch_shapes(case):
    """Sizes, windows and types of a batch, the same for every seed (a plan is
    built for its shapes)."""
    g = torch.Generator().manual_seed(case["n"] * 1009 + case["hi"])
    u = torch.rand((case["n"], 4), generator=g).tolist()
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    out = []
    for a, b, c, d in u:
        k = 3 + 2 * min(int(c * ((case["kmax"] - 1) // 2)), (case["kmax"] - 3) // 2)
        out.append((int(round(math.exp(lo + a * (hi - lo)))), int(round(math.exp(lo + b * (hi - lo)))), k,
                    "u8" if d < 0.5 else "u16"))
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    kind = case["kind"]
    if kind == "plane":
        x = _plane(gen, case["data"], case["dtype"], case["planes"], case["h"], case["w"])
        return {"kind": kind, "x": x, "kw": case["kw"], "kh": case["kh"]}
    if kind == "volume":
        return {"kind": kind, "x": _plane(gen, "noise", case["dtype"], case["d"], case["h"], case["w"]),
                "k": case["k"]}
    if kind == "batch":
        shapes = _batch_shapes(case)
        xs = [_plane(gen, "noise", dt, 1, h, w) for h, w, _, dt in shapes]
        # the results lie in one buffer per type, image after image
        flat = {dt: torch.empty(sum(h * w for h, w, _, t in shapes if t == dt), dtype=_DTYPES[dt], device="cuda")
                for dt in sorted({t for _, _, _, t in shapes})}
        used = dict.fromkeys(flat, 0)
        outs = []
        for h, w, _, dt in shapes:
            outs.append(flat[dt][used[dt]:used[dt] + h * w].view(h, w))
            used[dt] += h * w
        plan = ops.BatchedPlan(xs, outs, [k for _, _, k, _ in shapes])
        return {"kind": kind, "plan": plan, "outs": [_bits(f) for f in flat.values()]}
    shape = (case["n"], case["c"], case["h"], case["w"])
    x = torch.rand(shape, generator=gen, device="cuda").requires_grad_(True)
    g = torch.randn(shape, generator=gen, device="cuda")
    return {"kind": kind, "x": x, "g": g, "k": case["k"]}


def _bits(y):
    """y, unsigned 16- and 32-bit tensors seen as signed ones (torch indexes
    and reduces few unsigned types)."""
    return y.view({torch.uint16: torch.int16, torch.uint32: torch.int32}.get(y.dtype, y.dtype))


def run(state):
    kind = state["kind"]
    if kind == "plane":
        if state["kw"] == state["kh"]:
            return _bits(ops.median_filter(state["x"], state["kw"]))
        return _bits(ops.median_filter_rect(state["x"], state["kw"], state["kh"]))
    if kind == "volume":
        return _bits(ops.median_filter_3d(state["x"], state["k"]))
    if kind == "batch":
        state["plan"].launch()
        return state["outs"]
    y = ops.MedianFilterFn.apply(state["x"], state["k"])
    (gx,) = torch.autograd.grad(y, state["x"], state["g"])
    return {"y": y.detach(), "gx": gx}


def work(case):
    kind = case["kind"]
    if kind == "plane":
        b = 2 * _SIZE[case["dtype"]] * case["planes"] * case["h"] * case["w"]
    elif kind == "volume":
        b = 2 * _SIZE[case["dtype"]] * case["d"] * case["h"] * case["w"]
    elif kind == "batch":
        b = sum(2 * _SIZE[dt] * h * w for h, w, _, dt in _batch_shapes(case))
    else:
        # image and upstream gradient in, median and gradient out, and the
        # position each median was taken from written once and read once
        b = 24 * case["n"] * case["c"] * case["h"] * case["w"]
    return {"bytes": b, "flops": 0}


_EXACT_LIMIT = 2.2e9     # window values sorted


def _windows(x, r0, r1, kw, kh):
    """The kh*kw clamped window values, in row-major order, of output rows
    [r0, r1) of the planes x (p, h, w): (p, r1-r0, w, kh*kw)."""
    rx, ry = (kw - 1) // 2, (kh - 1) // 2
    h, w = x.shape[-2:]
    ys = (torch.arange(r0 - ry, r1 + ry, device=x.device)).clamp(0, h - 1)
    xs = (torch.arange(-rx, w + rx, device=x.device)).clamp(0, w - 1)
    u = x[:, ys][:, :, xs].unfold(1, kh, 1).unfold(2, kw, 1)
    return u.reshape(x.shape[0], r1 - r0, w, kh * kw)


def exact(case, seed):
    """Float outputs only: integer results are compared as they are."""
    kind = case["kind"]
    if kind == "plane" and case["dtype"] == "f32":
        n = case["kw"] * case["kh"]
        if case["planes"] * case["h"] * case["w"] * n > _EXACT_LIMIT:
            return None
        x = prepare(case, seed)["x"]
        p = x if x.dim() == 3 else x[None]
        y = torch.empty_like(p)
        rows = max(1, int(1e8 // (n * p.shape[0] * p.shape[2])))
        for r0 in range(0, p.shape[1], rows):
            r1 = min(p.shape[1], r0 + rows)
            y[:, r0:r1] = _windows(p, r0, r1, case["kw"], case["kh"]).sort(dim=-1).values[..., (n - 1) // 2]
        return y.reshape(x.shape).double()
    if kind == "autograd":
        k, h, w = case["k"], case["h"], case["w"]
        n = k * k
        if case["n"] * case["c"] * h * w * n > _EXACT_LIMIT:
            return None
        st = prepare(case, seed)
        x = st["x"].detach().reshape(-1, h, w)
        g = st["g"].reshape(-1, h, w).double()
        y = torch.empty_like(x)
        gx = torch.zeros(x.numel(), device=x.device, dtype=torch.float64)
        r = (k - 1) // 2
        px = torch.arange(w, device=x.device)
        rows = max(1, int(1e8 // (n * x.shape[0] * w)))
        for r0 in range(0, h, rows):
            r1 = min(h, r0 + rows)
            u = _windows(x, r0, r1, k, k)
            m = u.sort(dim=-1).values[..., (n - 1) // 2]
            y[:, r0:r1] = m
            first = (u == m[..., None]).to(torch.uint8).argmax(dim=-1)
            py = torch.arange(r0, r1, device=x.device)[:, None]
            qy = (py - r + first // k).clamp(0, h - 1)
            qx = (px - r + first % k).clamp(0, w - 1)
            plane = torch.arange(x.shape[0], device=x.device)[:, None, None]
            gx.index_add_(0, ((plane * h + qy) * w + qx).reshape(-1), g[:, r0:r1].reshape(-1))
        shape = st["x"].shape
        return {"y": y.double().reshape(shape), "gx": gx.reshape(shape)}
    return None
