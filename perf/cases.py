"""Representative calls of the 2-D wavelet transform, for timing and for comparing builds.

Each case is one call (or one pair of calls) a user's program makes through
the package's entry points: `fwd`, `inv`, `dwt2` (with its gradient) and
`BatchedForward`.  Sizes come from the tests and the benchmark (8192^2, 1024^2,
stacks of 8192^2 planes, uneven batches of 64 pixels and more, 256^2 planes) or
are generic (video frames, scans of odd size).

    listed()            the cases with a name
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs and handles on the GPU, from the seed alone
    run(state)          one pass; returns every output whole
    work(case)          bytes and operations a pass cannot do without
    exact(case, seed)   the outputs in 64 bits, from plain torch
"""
from __future__ import annotations

import math
import random

import torch

import paper_1704_08657_amd as pkg

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "i32": torch.int32}


def _case(op, wavelet, dtype, planes, height, width, levels, name=None):
    c = {"op": op, "wavelet": wavelet, "dtype": dtype, "planes": planes, "height": height, "width": width,
         "levels": levels}
    if name:
        c["name"] = name
    return c


def _batch(dtype, count, lo, hi, levels, shapes, name=None):
    c = {"op": "batched", "wavelet": "cdf97", "dtype": dtype, "count": count, "lo": lo, "hi": hi, "levels": levels,
         "shapes": shapes}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one thumbnail: the smallest call, bound by launches and latency
        _case("fwd", "cdf97", "f32", 1, 192, 256, 3, "thumbnail fwd f32"),
        # one medium image at the full depth: every level is a small launch
        _case("fwd", "cdf97", "f32", 1, 1024, 1024, 5, "image fwd f32"),
        # the benchmark's headline call: one large image, one level
        _case("fwd", "cdf97", "f32", 1, 8192, 8192, 1, "large fwd f32"),
        # reconstruction of a large image from its whole pyramid
        _case("inv", "cdf97", "f32", 1, 8192, 8192, 5, "large inv f32"),
        # a scan of odd height and width: no row is aligned
        _case("fwd", "cdf97", "f32", 1, 3469, 5197, 3, "odd scan fwd f32"),
        # a stack of large planes with 16-bit storage (the largest case)
        _case("fwd", "cdf97", "bf16", 3, 8192, 8192, 5, "large planes fwd bf16"),
        # decoding a colour video frame kept in 16 bits
        _case("inv", "cdf97", "f16", 3, 2160, 3840, 4, "frame inv f16"),
        # lossless coding of a colour frame of odd size: both directions
        _case("lossless", "cdf53", "i32", 3, 1081, 1921, 5, "odd frame lossless i32"),
        # the longer four-tap wavelet, analysis of an image ...
        _case("fwd", "dd137", "f32", 1, 4096, 4096, 3, "dd137 fwd f32"),
        # ... and synthesis of a frame of odd size with 16-bit storage
        _case("inv", "dd137", "bf16", 3, 2161, 3841, 2, "dd137 odd frame inv bf16"),
        # a training step's transform and its gradient: a batch of colour crops
        _case("grad", "cdf97", "f32", 192, 256, 256, 3, "training crops grad f32"),
        # a collection of images of uneven sizes in one call
        _batch("f32", 60, 64, 2048, 5, 1, "uneven batch fwd f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _levels(h, w):
    n = 0
    while h >= 2 and w >= 2 and n < 5:
        n, h, w = n + 1, (h + 1) // 2, (w + 1) // 2
    return n


def draw(rng):
    op = rng.choice(["fwd", "fwd", "fwd", "inv", "inv", "grad", "lossless", "batched"])
    if op == "batched":
        hi = _log(rng, 128, 2048)
        count = min(_log(rng, 4, 60), max(4, (48 << 20) // (hi * hi // 3)))
        return _batch(rng.choice(["f32", "f32", "bf16", "f16"]), count, 64, hi, rng.randint(1, 5),
                      rng.randrange(1 << 20))
    if op == "lossless":
        wavelet, dtype = "cdf53", "i32"
    elif op == "grad":
        wavelet, dtype = "cdf97", "f32"
    else:
        wavelet = rng.choice(["cdf97", "cdf97", "cdf97", "cdf53f", "dd137"])
        dtype = rng.choice(["f32", "f32", "bf16", "f16"])
    # pixels of the whole call: the long wavelet and the two-way calls draw smaller ones
    most = (16 << 20) if wavelet == "dd137" or op in ("grad", "lossless") else (64 << 20)
    side, aspect = _log(rng, 64, 8192), math.exp(rng.uniform(-1, 1))
    h, w = (max(48, int(side * math.sqrt(a))) for a in (aspect, 1 / aspect))
    kind = rng.randrange(3)                 # sides: any, even, multiples of 64
    if kind == 1:
        h, w = h // 2 * 2, w // 2 * 2
    elif kind == 2:
        h, w = max(64, h // 64 * 64), max(64, w // 64 * 64)
    while h * w > most:
        h = max(48, h // 2)
        w = max(48, w // 2)
    planes = rng.choice([1, 1, 3, _log(rng, 1, 256)])
    planes = max(1, min(planes, most // (h * w)))
    return _case(op, wavelet, dtype, planes, h, w, rng.randint(1, _levels(h, w)))


# ---- inputs -----------------------------------------------------------------

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _images(planes, h, w, gen):
    """Smooth ramps plus noise in about [0, 1]: what natural images look like to the transform."""
    dev = gen.device
    x = torch.randn((planes, h, w), generator=gen, device=dev).mul_(0.05)
    a = torch.rand((planes, 1, 1), generator=gen, device=dev)
    x += a * torch.linspace(0, 1, h, device=dev).view(1, h, 1)
    x += (1 - a) * torch.linspace(0, 1, w, device=dev).view(1, 1, w)
    return x


def _pyramids(planes, h, w, levels, gen):
    """Mallat pyramids: an image-like LL band, small details around it."""
    y = torch.randn((planes, h, w), generator=gen, device=gen.device).mul_(0.06)
    hl, wl = h, w
    for _ in range(levels):
        hl, wl = (hl + 1) // 2, (wl + 1) // 2
    y[:, :hl, :wl] = _images(planes, hl, wl, gen) * float(2 ** levels)
    return y


def _shapes(case):
    r = random.Random(case["shapes"])
    return [(r.randint(case["lo"], case["hi"]), r.randint(case["lo"], case["hi"])) for _ in range(case["count"])]


def _inputs(case, seed):
    gen = torch.Generator(device=_device())
    gen.manual_seed(seed)
    dt, op = DTYPES[case["dtype"]], case["op"]
    if op == "batched":
        return [_images(1, h, w, gen)[0].to(dt) for h, w in _shapes(case)]
    p, h, w = case["planes"], case["height"], case["width"]
    if op == "inv":
        x = _pyramids(p, h, w, case["levels"], gen).to(dt)
    elif op == "lossless":
        x = _images(p, h, w, gen).mul_(255).round_().clamp_(0, 255).to(dt)
    else:
        x = _images(p, h, w, gen).to(dt)
    if p == 1:
        x = x[0]                            # a single image is a [H, W] tensor
    if op == "grad":
        # the cotangent a loss on the coefficients sends back
        return x, torch.randn(x.shape, generator=gen, device=gen.device).mul_(0.1)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    if case["op"] == "batched":
        x = pkg.BatchedForward(x, case["levels"])      # the handle such a program keeps
    elif case["op"] == "grad":
        x[0].requires_grad_(True)
    return {"case": case, "x": x}


def run(state):
    c, x = state["case"], state["x"]
    op, wavelet, levels = c["op"], c["wavelet"], c["levels"]
    if op == "fwd":
        return pkg.fwd(x, wavelet, levels)
    if op == "inv":
        return pkg.inv(x, wavelet, levels)
    if op == "lossless":
        y = pkg.fwd(x, wavelet, levels)
        return y, pkg.inv(y, wavelet, levels)
    if op == "batched":
        return x.run()
    x, g = x
    y = pkg.dwt2(x, levels)
    (gx,) = torch.autograd.grad(y, x, g)
    return y.detach(), gx


# ---- work and exact values --------------------------------------------------

def work(case):
    if case["op"] == "batched":
        n = sum(h * w for h, w in _shapes(case))
    else:
        n = case["planes"] * case["height"] * case["width"]
    ways = 2 if case["op"] in ("grad", "lossless") else 1
    size = torch.empty(0, dtype=DTYPES[case["dtype"]]).element_size()
    # per sample and axis: 1.5 operations for each two-tap step, 4 for each
    # four-tap one; the levels after the first add a third
    per = {"cdf97": 2 * 4 * 1.5 + 0.5, "cdf53": 2 * 2 * 2, "cdf53f": 2 * 2 * 1.5 + 0.5, "dd137": 2 * 2 * 4 + 0.5}
    deeper = sum(0.25 ** l for l in range(case["levels"]))
    return {"bytes": 2 * n * size * ways, "flops": n * per[case["wavelet"]] * deeper * ways}


# (predict taps, update taps) per lifting pair, as {offset: coefficient}
_PAIRS = {
    "cdf97": [({0: -1.586134342059924, 1: -1.586134342059924}, {-1: -0.052980118572961, 0: -0.052980118572961}),
              ({0: 0.882911075530934, 1: 0.882911075530934}, {-1: 0.443506852043971, 0: 0.443506852043971})],
    "cdf53f": [({0: -0.5, 1: -0.5}, {-1: 0.25, 0: 0.25})],
    "dd137": [({-1: 1 / 16, 0: -9 / 16, 1: -9 / 16, 2: 1 / 16}, {-2: -1 / 32, -1: 9 / 32, 0: 9 / 32, 1: -1 / 32})],
}
_ZETA = {"cdf97": math.sqrt(2.0) / (1.0 - 2.0 * 0.052980118572961 * (1.0 - 2.0 * 1.586134342059924)),
         "cdf53f": math.sqrt(2.0), "dd137": math.sqrt(2.0)}


def _lift(src, dst, taps, n, parity, sign):
    """dst[m] + sign * sum taps[k] src[m + k] along the last axis, under whole-point symmetric extension."""
    m = torch.arange(dst.shape[-1], device=dst.device)
    for k, c in taps.items():
        p = torch.remainder(2 * (m + k) + parity, 2 * (n - 1))
        p = torch.where(p > n - 1, 2 * (n - 1) - p, p)
        dst = dst + (sign * c) * src[..., (p - parity) // 2]
    return dst


def _fwd_axis(x, wavelet):
    n, e, o = x.shape[-1], x[..., 0::2], x[..., 1::2]
    for P, U in _PAIRS[wavelet]:
        o = _lift(e, o, P, n, 0, 1)
        e = _lift(o, e, U, n, 1, 1)
    z = _ZETA[wavelet]
    return torch.cat([e * z, o / z], -1)


def _inv_axis(y, wavelet):
    n, z = y.shape[-1], _ZETA[wavelet]
    e, o = y[..., :(n + 1) // 2] / z, y[..., (n + 1) // 2:] * z
    for P, U in reversed(_PAIRS[wavelet]):
        e = _lift(o, e, U, n, 1, -1)
        o = _lift(e, o, P, n, 0, -1)
    x = torch.empty_like(y)
    x[..., 0::2], x[..., 1::2] = e, o
    return x


def _both(x, wavelet, axis):
    return axis(axis(x, wavelet).transpose(-1, -2), wavelet).transpose(-1, -2)


def _exact_fwd(x, wavelet, levels):
    h, w = x.shape[-2:]
    y = _both(x, wavelet, _fwd_axis)
    if levels == 1:
        return y
    hl, wl = (h + 1) // 2, (w + 1) // 2
    ll = _exact_fwd(y[..., :hl, :wl], wavelet, levels - 1)
    return torch.cat([torch.cat([ll, y[..., :hl, wl:]], -1), y[..., hl:, :]], -2)


def _exact_inv(y, wavelet, levels):
    y = y.clone()
    sizes = [tuple(y.shape[-2:])]
    for _ in range(levels - 1):
        sizes.append(((sizes[-1][0] + 1) // 2, (sizes[-1][1] + 1) // 2))
    for h, w in reversed(sizes):
        y[..., :h, :w] = _both(y[..., :h, :w], wavelet, _inv_axis)
    return y


def exact(case, seed):
    op, wavelet, levels = case["op"], case["wavelet"], case["levels"]
    if op == "lossless":
        return None                         # whole numbers: equal, or wrong
    x = _inputs(case, seed)
    if op == "batched":
        return [_exact_fwd(i.double(), wavelet, levels) for i in x]
    if op == "inv":
        return _planewise(x, lambda v: _exact_inv(v, wavelet, levels))
    if op == "fwd":
        return _planewise(x, lambda v: _exact_fwd(v, wavelet, levels))
    x, g = x[0].double().requires_grad_(True), x[1].double()
    y = _exact_fwd(x, wavelet, levels)
    (gx,) = torch.autograd.grad(y, x, g)
    return y.detach(), gx


def _planewise(x, f):
    """f on each plane in turn (64-bit copies of one plane at a time)."""
    if x.dim() == 2:
        return f(x.double())
    return torch.stack([f(v.double()) for v in x])
