"""Performance cases: the calls that programs make of this package, by size.

Every case goes through the package's public entry points.  Frames are seeded
gratings plus noise (8-bit) or noise on [0, 1) (float); fixations are drawn
per seed.  ``exact`` is the method written out in 64-bit torch operations.

Kinds of case:

* ``frame``: ``forward`` on one tensor of n frames, into a buffer that the
  program keeps (a viewer's frame loop, a model's input transform);
* ``batch``: ``forward_batch`` on a list of frames of mixed resolution;
* ``step``: ``foveate`` and its backward pass through autograd;
* ``adjoint``: ``backward`` alone, into a kept gradient buffer;
* ``serve``: a burst of frames through a ``Server``, waited for;
* ``host``: frames in pinned host memory through a ``HostPipeline``.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2012_08655_amd as fov

DT = {"u8": torch.uint8, "f32": torch.float32, "f64": torch.float64}
BYTES = {"u8": 1, "f32": 4, "f64": 8}
# The frame sizes of viewers and servers, lowest to highest.
RESOLUTIONS = ((480, 640), (720, 1280), (1080, 1920), (2160, 3840))


def _case(name, kind, n, c, h, w, layout, din, dout, block, e0, slope, cap, gaze="half", shift=False, sigma_map=False):
    d = {"kind": kind, "n": n, "c": c, "h": h, "w": w, "layout": layout, "in": din, "out": dout, "block": block,
         "e0": e0, "slope": slope, "cap": cap, "gaze": gaze, "shift": shift, "map": sigma_map}
    return {"name": name, **d} if name else d


def listed():
    return [
        # The smallest calls: one small frame per call, where launches and latency count.
        _case("f32_gray_256", "frame", 1, 1, 256, 256, "CHW", "f32", "f32", 32, 32.0, 0.05, 8.0),
        _case("u8_gray_480p", "frame", 1, 1, 480, 640, "HW", "u8", "u8", 32, 64.0, 0.02, 16.0),
        # The headline: a viewer's 1080p RGB frame loop.
        _case("u8_rgb_1080p", "frame", 1, 3, 1080, 1920, "HWC", "u8", "u8", 32, 64.0, 0.02, 16.0),
        # The largest single frame, with the tiling centred on the gaze (fragment shift).
        _case("u8_rgb_2160p_shift", "frame", 1, 3, 2160, 3840, "HWC", "u8", "u8", 32, 64.0, 0.02, 16.0, shift=True),
        # Offline processing of a mixed set of frames in one launch; the largest call.
        _case("u8_batch_64_mixed", "batch", 64, 3, 0, 0, "HWC", "u8", "u8", 32, 64.0, 0.0, 16.0),
        # 8-bit images of an odd size into a model's float input, blur from a per-fragment map
        # (saliency) instead of the ramp, small fragments.
        _case("u8_f32_map_odd", "frame", 8, 3, 317, 451, "NCHW", "u8", "f32", 16, 0.0, 0.0, 9.0, sigma_map=True),
        # A model's input transform at the training resolutions: forward alone,
        _case("f32_fwd_512", "frame", 4, 3, 512, 512, "NCHW", "f32", "f32", 32, 32.0, 0.03, 12.0, gaze="any"),
        # a whole differentiable step,
        _case("f32_step_224", "step", 32, 3, 224, 224, "NCHW", "f32", "f32", 32, 32.0, 0.03, 12.0, gaze="any"),
        # and the backward pass alone.
        _case("f32_bwd_512", "adjoint", 4, 3, 512, 512, "NCHW", "f32", "f32", 32, 32.0, 0.03, 12.0, gaze="any"),
        # Gradient checks and reference runs in double precision.
        _case("f64_step_160", "step", 2, 3, 160, 160, "NCHW", "f64", "f64", 16, 0.0, 0.03, 12.0, gaze="any"),
        # A server's burst of viewers' frames (all resolutions in turn), batched on several streams.
        _case("u8_serve_16", "serve", 16, 3, 0, 0, "HWC", "u8", "u8", 32, 64.0, 0.0, 16.0),
        # Frames in host memory there and back (transfers included).
        _case("u8_host_1080p", "host", 8, 3, 1080, 1920, "HWC", "u8", "u8", 32, 64.0, 0.02, 16.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("frame8", "frame8", "frame8", "to_f32", "fwd", "step", "adjoint", "f64", "batch", "serve"))
    if kind == "frame8":  # viewer frames, any size up to 4K, gray or RGB, tiled from the corner or centred
        h = _log(rng, 200, 2160)
        w = int(h * rng.uniform(1.0, 1.8))
        c = rng.choice((1, 3, 3))
        return _case(None, "frame", 1, c, h, w, "HWC", "u8", "u8", rng.choice((16, 32, 32, 32, 64)),
                     rng.choice((32.0, 64.0)), rng.uniform(0.01, 0.04), rng.choice((8.0, 16.0, 16.0)),
                     shift=rng.random() < 0.4)
    if kind == "to_f32":
        h, n = _log(rng, 64, 512), rng.choice((1, 3, 8, 16))
        return _case(None, "frame", n, 3, h, int(h * rng.uniform(0.8, 1.5)), "NCHW", "u8", "f32",
                     rng.choice((16, 32)), 32.0, rng.uniform(0.01, 0.05), 12.0, gaze="any", sigma_map=rng.random() < 0.5)
    if kind in ("fwd", "step", "adjoint"):  # training batches
        h = _log(rng, 64, 512)
        n = _log(rng, 1, 32)
        return _case(None, {"fwd": "frame"}.get(kind, kind), n, rng.choice((1, 3, 3)), h, int(h * rng.uniform(0.9, 1.4)),
                     "NCHW", "f32", "f32", rng.choice((16, 32, 32)), rng.choice((0.0, 32.0)), rng.uniform(0.02, 0.05),
                     12.0, gaze="any", shift=rng.random() < 0.3)
    if kind == "f64":
        h = _log(rng, 40, 200)
        return _case(None, rng.choice(("step", "frame")), rng.choice((1, 2)), 3, h, int(h * rng.uniform(0.8, 1.4)), "NCHW",
                     "f64", "f64", rng.choice((16, 32)), 0.0, rng.uniform(0.02, 0.06), rng.choice((6.0, 12.0)), gaze="any")
    if kind == "batch":
        return _case(None, "batch", _log(rng, 4, 48), 3, 0, 0, "HWC", "u8", "u8", 32, 64.0, 0.0, rng.choice((8.0, 16.0)))
    return _case(None, "serve", _log(rng, 2, 16), 3, 0, 0, "HWC", "u8", "u8", 32, 64.0, 0.0, rng.choice((8.0, 16.0)))


# ---- inputs -----------------------------------------------------------------------------------------
def _sizes(case):
    """(h, w) of every frame of a case: mixed cases take the resolutions in turn."""
    if case["h"]:
        return [(case["h"], case["w"])] * case["n"]
    return [RESOLUTIONS[(i * 7 + i // 4) % 4] for i in range(case["n"])]


def _params(case, rng):
    """One dict of parameters per frame: gaze in the central half of the frame or anywhere in it."""
    out = []
    for h, w in _sizes(case):
        lo, hi = (0.25, 0.75) if case["gaze"] == "half" else (0.0, 1.0)
        p = {"fix_x": float(rng.uniform(lo * (w - 1), hi * (w - 1))), "fix_y": float(rng.uniform(lo * (h - 1), hi * (h - 1))),
             "e0": case["e0"], "slope": case["slope"] or float(rng.uniform(0.01, 0.04)), "cap": case["cap"],
             "block": case["block"], "origin_x": 0, "origin_y": 0}
        out.append(fov.fragment_shift(p) if case["shift"] else p)
    return out


def _sigma_map(case, p, rng):
    """Blur strengths of the fragments from a smooth map of values, some of them 0 (kept sharp)."""
    h, w, B = case["h"], case["w"], case["block"]
    nby, nbx = -(-(h - p["origin_y"]) // B), -(-(w - p["origin_x"]) // B)
    y, x = np.mgrid[0:nby, 0:nbx].astype(np.float64)
    f = rng.uniform(0.1, 0.5, 4)
    m = np.sin(f[0] * x + f[1] * y + rng.uniform(0, 6)) + np.sin(f[2] * x - f[3] * y + rng.uniform(0, 6))
    return np.clip((m + 1.0) / 3.0 * case["cap"], 0.0, None).astype(np.float32)


def _gratings(h, w, c, gen):
    """u8 [h, w, c] frame on the GPU: eight cosine gratings per channel plus noise."""
    dev = gen.device
    u = torch.rand((c, 8, 3), generator=gen, device=dev)
    ys = torch.arange(h, device=dev, dtype=torch.float32)
    xs = torch.arange(w, device=dev, dtype=torch.float32)
    out = torch.empty((h, w, c), dtype=torch.uint8, device=dev)
    for ch in range(c):
        period = 4.0 * 64.0 ** u[ch, :, 0]
        theta = math.pi * u[ch, :, 1]
        ax = (2 * math.pi * torch.cos(theta) / period)[:, None] * xs + (2 * math.pi * u[ch, :, 2])[:, None]
        by = (2 * math.pi * torch.sin(theta) / period)[:, None] * ys
        acc = torch.cos(by).t() @ torch.cos(ax) - torch.sin(by).t() @ torch.sin(ax)
        acc = 127.5 + 107.5 / 8.0 * acc + 40.0 * torch.rand((h, w), generator=gen, device=dev) - 20.0
        out[:, :, ch] = acc.round().clamp(0, 255).to(torch.uint8)
    return out


def _tensor(case, gen):
    """The frames of a case of one size, in its layout."""
    n, c, h, w = case["n"], case["c"], case["h"], case["w"]
    if case["in"] != "u8":
        shape = {"NCHW": (n, c, h, w), "CHW": (c, h, w)}[case["layout"]]
        return torch.rand(shape, generator=gen, device=gen.device, dtype=DT[case["in"]])
    fr = torch.stack([_gratings(h, w, c, gen) for _ in range(n)])
    return {"NCHW": lambda: fr.permute(0, 3, 1, 2).contiguous(), "HWC": lambda: fr[0], "HW": lambda: fr[0, :, :, 0].contiguous()}[
        case["layout"]]()


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    rng = np.random.default_rng(int(seed))
    kind, s = case["kind"], {"case": case}
    s["params"] = _params(case, rng)
    if kind in ("batch", "serve"):
        s["x"] = [_gratings(h, w, case["c"], gen) for h, w in _sizes(case)]
        s["out"] = [torch.empty_like(t) for t in s["x"]]
        if kind == "serve":
            s["server"] = fov.Server(hbm_budget_bytes=256 << 20, max_batch_frames=16, max_inflight_batches=4,
                                     max_fragments=16 * 8160, max_block=case["block"], max_sigma=case["cap"])
    elif kind == "host":
        s["x"] = [_gratings(h, w, case["c"], gen).cpu().pin_memory() for h, w in _sizes(case)]
        s["out"] = [torch.empty(t.shape, dtype=t.dtype, pin_memory=True) for t in s["x"]]
        s["pipeline"] = fov.HostPipeline(case["h"] * case["w"] * case["c"], depth=4)
    else:
        if case["map"]:
            for p in s["params"]:
                p["sigma_map"] = torch.from_numpy(_sigma_map(case, p, rng).reshape(-1)).to(dev)
        s["x"] = _tensor(case, gen)
        if kind in ("step", "adjoint"):
            s["g"] = torch.randn(s["x"].shape, generator=gen, device=dev, dtype=s["x"].dtype)
        if kind == "step":
            s["x"].requires_grad_(True)
        else:
            s["out"] = torch.empty_like(s["x"], dtype=DT[case["out"]])
        s["params"] = s["params"][0] if case["n"] == 1 else s["params"]
    return s


# ---- the calls --------------------------------------------------------------------------------------
def run(state):
    case, params, x = state["case"], state["params"], state["x"]
    kind, layout = case["kind"], case["layout"]
    if kind == "frame":
        return fov.forward(x, params, out=state["out"], layout=layout)
    if kind == "batch":
        return fov.forward_batch(x, params, outs=state["out"], layout=layout)
    if kind == "step":
        y = fov.foveate(x, params, layout)
        (gx,) = torch.autograd.grad(y, x, state["g"])
        return [y.detach(), gx]
    if kind == "adjoint":
        return fov.backward(state["g"], params, grad_in=state["out"], layout=layout)
    if kind == "serve":
        tickets = [state["server"].submit(f, o, p, layout=layout) for f, o, p in zip(x, state["out"], params)]
        state["server"].drain()
        for t in tickets:
            state["server"].poll(t)
        return state["out"]
    tickets = []  # host: at most four frames in flight
    for i, (f, o, p) in enumerate(zip(x, state["out"], params)):
        if i >= 4:
            state["pipeline"].wait(tickets[i - 4])
        tickets.append(state["pipeline"].submit(f, p, out=o, layout=layout))
    for t in tickets[-4:]:
        state["pipeline"].wait(t)
    return state["out"]


# ---- what a pass cannot do without ------------------------------------------------------------------
def _sigmas(h, w, p, smap=None):
    """Blur strength of every fragment [nby, nbx]."""
    B = p["block"]
    nby, nbx = -(-(h - p["origin_y"]) // B), -(-(w - p["origin_x"]) // B)
    if smap is not None:
        return np.clip(np.asarray(smap, np.float64).reshape(nby, nbx), 0.0, p["cap"])
    cx = p["origin_x"] + np.arange(nbx, dtype=np.float64) * B + (B - 1) / 2.0
    cy = p["origin_y"] + np.arange(nby, dtype=np.float64) * B + (B - 1) / 2.0
    e = np.sqrt((cx[None, :] - p["fix_x"]) ** 2 + (cy[:, None] - p["fix_y"]) ** 2)
    return np.where(e < p["e0"], 0.0, np.clip(p["slope"] * (e - p["e0"]), 0.0, p["cap"]))


def work(case):
    """Frames read once and written once, and the multiply-adds of the two separable passes over each
    fragment (the first one over its halo rows too), for gazes of one fixed seed."""
    rng = np.random.default_rng(0)
    fmas = px = 0
    for (h, w), p in zip(_sizes(case), _params(case, rng)):
        B = p["block"]
        s = _sigmas(h, w, p, _sigma_map(case, p, rng) if case["map"] else None)
        n = 2 * np.ceil(3.0 * s) + 1
        by, bx = np.indices(s.shape)
        bh = np.minimum(p["origin_y"] + (by + 1) * B, h) - np.maximum(p["origin_y"] + by * B, 0)
        bw = np.minimum(p["origin_x"] + (bx + 1) * B, w) - np.maximum(p["origin_x"] + bx * B, 0)
        fmas += float((np.where(s > 0, n * bw * (2 * bh + n - 1), 0.0)).sum()) * case["c"]
        px += h * w * case["c"]
    passes = 2 if case["kind"] == "step" else 1
    return {"bytes": float(passes * px * (BYTES[case["in"]] + BYTES[case["out"]])), "flops": 2.0 * passes * fmas}


# ---- the method in 64 bits --------------------------------------------------------------------------
def _exact_frame(x, p, sigma):
    """x [c, h, w] float64 on the GPU; sigma [nby, nbx].  Each fragment is its clamped window between two
    banded matrices of its taps."""
    c, h, w = x.shape
    B, dev = p["block"], x.device
    nby, nbx = sigma.shape
    r = np.ceil(3.0 * sigma).astype(np.int64).reshape(-1)
    R = int(r.max())
    sg = torch.from_numpy(sigma.reshape(-1)).to(dev)
    rr = torch.from_numpy(r).to(dev)
    k = torch.arange(-R, R + 1, device=dev, dtype=torch.float64)
    e = torch.exp(-k[None] ** 2 / (2.0 * torch.where(sg > 0, sg, 1.0)[:, None] ** 2))
    e = torch.where(k[None].abs() <= rr[:, None], e, 0.0)
    taps = e / e.sum(1, keepdim=True)
    i, o = torch.arange(B + 2 * R, device=dev), torch.arange(B, device=dev)
    off = i[:, None] - o[None, :]  # window row - output row: tap index
    live = (off >= 0) & (off <= 2 * R)
    fr = torch.arange(nby * nbx, device=dev)
    Y0, X0 = p["origin_y"] + (fr // nbx) * B, p["origin_x"] + (fr % nbx) * B
    pieces, step = [], max(1, (1 << 27) // (c * (B + 2 * R) ** 2))
    for f in range(0, nby * nbx, step):
        t = taps[f:f + step]
        T = torch.where(live, t[:, off.clamp(0, 2 * R)], 0.0)  # [b, window, B]
        ys = (Y0[f:f + step, None] - R + i).clamp(0, h - 1)
        xs = (X0[f:f + step, None] - R + i).clamp(0, w - 1)
        win = x[:, ys[:, :, None], xs[:, None, :]]  # [c, b, window, window]
        pieces.append(torch.matmul(T.transpose(1, 2).contiguous()[None], torch.matmul(win, T[None])))
    out = torch.cat(pieces, 1).reshape(c, nby, nbx, B, B).permute(0, 1, 3, 2, 4).reshape(c, nby * B, nbx * B)
    oy, ox = -p["origin_y"], -p["origin_x"]
    return out[:, oy:oy + h, ox:ox + w]


def exact(case, seed):
    if case["out"] == "u8":
        return None  # whole numbers
    s = prepare(case, seed)
    plist = s["params"] if isinstance(s["params"], list) else [s["params"]]
    x = s["x"].detach().double().reshape(case["n"], case["c"], case["h"], case["w"])
    y, gx = torch.empty_like(x), torch.empty_like(x)
    for i, p in enumerate(plist):
        smap = p["sigma_map"].double().cpu().numpy() if case["map"] else None
        sigma = _sigmas(case["h"], case["w"], p, smap)
        if case["kind"] == "frame":
            y[i] = _exact_frame(x[i], p, sigma)
            continue
        xi = x[i].clone().requires_grad_(True)
        yi = _exact_frame(xi, p, sigma)
        g = s["g"].double().reshape(x.shape)[i]
        (gx[i],) = torch.autograd.grad(yi, xi, g)
        y[i] = yi.detach()
    y, gx = y.reshape(s["x"].shape), gx.reshape(s["x"].shape)
    return y if case["kind"] == "frame" else gx if case["kind"] == "adjoint" else [y, gx]
