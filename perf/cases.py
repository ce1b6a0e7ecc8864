"""The work that users of this library have it do, as a list of measured cases.

A case is one call through the torch-level entry points (``compress``,
``decompress``, ``compress_batch``, ``decompress_batch``) on fields resident
in device memory, with the buffers a program keeps between calls (stream,
workspace, reconstruction) made beforehand.

Fields follow the recipes of ``paper_2603_26968_amd.synth`` (power-law
turbulence with noise, a floored lognormal field, sinusoids with sharp
fronts, Gaussian bumps), made on the device from the seed.  Shapes are those
of the benchmark's workloads and of the paper's data sets (90x500x500,
310x128x128, 69x69x115), or drawn over the same ranges.
"""
import math
import random

import numpy as np
import torch

import paper_2603_26968_amd as P

DEV = "cuda:0"


# ------------------------------------------------------------------ cases
def _one(name, op, field, dtype, shape, eb, mode="noa"):
    return {"name": name, "op": op, "field": field, "dtype": dtype,
            "shape": "x".join(str(s) for s in shape), "eb": eb, "mode": mode}


def listed():
    return [
        # a large simulation output of doubles, heavy tailed, with exact ties:
        # the benchmark's headline field, written and read back
        _one("c3d-512-f64-lognormal", "compress", "lognormal", "f64", (512, 512, 512), 1e-3),
        _one("d3d-512-f64-lognormal", "decompress", "lognormal", "f64", (512, 512, 512), 1e-3),
        # an ordinary single-precision volume at an ordinary bound
        _one("c3d-256-f32-turb", "compress", "turb", "f32", (256, 256, 256), 1e-3),
        _one("d3d-256-f32-turb", "decompress", "turb", "f32", (256, 256, 256), 1e-3),
        # a flat, uneven volume at the coarse bound of the paper's tables:
        # many points share a bin, the order repair has the most to do
        _one("c3d-90x500x500-f32-coarse", "compress", "turb", "f32", (90, 500, 500), 1e-2),
        # doubles at the fine bound, given as an absolute bound
        _one("c3d-310x128x128-f64-abs", "compress", "turb", "f64", (310, 128, 128), 1e-4, "abs"),
        # a 2D map with smooth regions and sharp fronts
        _one("c2d-1800x3600-f32-fronts", "compress", "fronts", "f32", (1800, 3600), 1e-3),
        _one("d2d-1800x3600-f32-fronts", "decompress", "fronts", "f32", (1800, 3600), 1e-3),
        # the smallest calls: one image written, one small volume of odd sides
        # read; latency and launches
        _one("c2d-512-f32-bumps", "compress", "bumps", "f32", (512, 512), 1e-3),
        _one("d3d-69x69x115-f64-turb", "decompress", "turb", "f64", (69, 69, 115), 1e-4),
        # many uneven 2D and 3D fields in one call, as a service collects them
        {"name": "c-batch-48", "op": "compress_batch", "count": 48, "mix": 1, "dtypes": "f32"},
        {"name": "d-batch-48", "op": "decompress_batch", "count": 48, "mix": 1, "dtypes": "f32"},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_shape(rng, ndim, points):
    """Uneven sides around the cube (square) of that many points."""
    w = [_log_uniform(rng, 0.6, 1.7) for _ in range(ndim)]
    g = math.prod(w) ** (1.0 / ndim)
    return [max(3, round(points ** (1.0 / ndim) * v / g)) for v in w]


def draw(rng):
    if rng.random() < 0.2:
        return {"op": rng.choice(["compress_batch", "decompress_batch"]),
                "count": rng.randint(3, 56), "mix": rng.randint(2, 1 << 30),
                "dtypes": rng.choice(["f32", "f64", "f32 f64"])}
    field = rng.choice(["turb", "turb", "lognormal", "fronts", "bumps"])
    ndim = 2 if field == "fronts" or (field == "bumps" and rng.random() < 0.5) else 3
    eb = _log_uniform(rng, 1e-4, 1e-2)
    # sizes up to the largest listed case; coarse bounds and smooth 2D maps
    # (long runs of points in one bin) up to a cost below it
    top = (1 << 23) if ndim == 2 else (1 << 26) * min(1.0, 1e-3 / eb)
    shape = _draw_shape(rng, ndim, _log_uniform(rng, 1 << 14, top))
    case = _one("", rng.choice(["compress", "decompress"]), field, rng.choice(["f32", "f64"]),
                shape, eb, rng.choice(["noa", "noa", "abs"]))
    del case["name"]
    return case


# ------------------------------------------------------------------ fields
def _shape(text):
    return tuple(int(s) for s in text.split("x"))


def _torch_dtype(text):
    return torch.float32 if text == "f32" else torch.float64


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _grf(shape, slope, gen):
    """A Gaussian random field of power spectrum |k|^-slope, standardised: cut
    out of a periodic one whose sides are powers of two."""
    full = [1 << max(3, (s - 1).bit_length()) for s in shape]
    spec = torch.fft.rfftn(torch.randn(full, dtype=torch.float64, device=DEV, generator=gen))
    k2 = torch.zeros(spec.shape, dtype=torch.float64, device=DEV)
    for a, n in enumerate(full):
        f = torch.fft.rfftfreq(n) if a == len(full) - 1 else torch.fft.fftfreq(n)
        view = [1] * len(full)
        view[a] = -1
        k2 += f.to(DEV, torch.float64).square().reshape(view)
    k2[(0,) * len(full)] = 1.0
    spec *= k2.pow_(-slope / 4.0)
    spec[(0,) * len(full)] = 0.0
    del k2
    g = torch.fft.irfftn(spec, s=full)
    g = g[tuple(slice(0, s) for s in shape)].contiguous()
    g -= g.mean()
    return g.div_(g.std())


def _turb(shape, gen):
    g = _grf(shape, 3.0, gen)
    g += 0.01 * torch.randn(shape, dtype=torch.float64, device=DEV, generator=gen)
    g -= g.min()
    return g.div_(g.max())


def _lognormal(shape, gen):
    g = _grf(shape, 2.5, gen).mul_(2.0).exp_()
    part = g.flatten()[:: max(1, g.numel() >> 22)]
    return g.clamp_(min=part.kthvalue(max(1, part.numel() // 10)).values)


def _axes(shape):
    return torch.meshgrid(*[torch.arange(s, dtype=torch.float64, device=DEV) for s in shape],
                          indexing="ij")


def _fronts(shape, rng):
    i, j = (a / s for a, s in zip(_axes(shape), shape))
    out = torch.zeros(shape, dtype=torch.float64, device=DEV)

    def wave(top):
        a, b = rng.randint(1, top), rng.randint(1, top)
        return torch.sin(2 * math.pi * (a * i + b * j) + rng.uniform(0, 2 * math.pi))

    for _ in range(8):
        out += rng.uniform(0.2, 1.0) * wave(6)
    for _ in range(4):
        h = rng.uniform(40.0, 120.0) * wave(3) + rng.uniform(40.0, 120.0) * wave(3)
        out += rng.uniform(0.5, 1.5) * torch.tanh((h + rng.uniform(-20.0, 20.0))
                                                   / rng.uniform(1.0, 4.0))
    return out


def _bumps(shape, rng, gen):
    axes = _axes(shape)
    out = 1e-3 * torch.randn(shape, dtype=torch.float64, device=DEV, generator=gen)
    for _ in range(32):
        rot, _ = np.linalg.qr(np.array([[rng.gauss(0, 1) for _ in shape] for _ in shape]))
        form = rot @ np.diag([rng.uniform(8.0, 64.0) ** -2 for _ in shape]) @ rot.T
        d = [a - rng.uniform(0, s) for a, s in zip(axes, shape)]
        quad = sum(float(form[r, c]) * (1 if r == c else 2) * d[r] * d[c]
                   for r in range(len(d)) for c in range(r, len(d)))
        out += rng.uniform(-1.0, 1.0) * torch.exp(-0.5 * quad)
    return out


def _field(kind, shape, dtype, seed):
    gen, rng = _gen(seed), random.Random(seed)
    if kind == "turb":
        x = _turb(shape, gen)
    elif kind == "lognormal":
        x = _lognormal(shape, gen)
    elif kind == "fronts":
        x = _fronts(shape, rng)
    else:
        x = _bumps(shape, rng, gen)
    return x.to(_torch_dtype(dtype)).contiguous()


def _fields(case, seed):
    """(kind, dtype, shape, eb, mode, seed) of every field of a case."""
    if "field" in case:
        return [(case["field"], case["dtype"], _shape(case["shape"]), case["eb"], case["mode"],
                 seed)]
    rng = random.Random(case["mix"])
    out = []
    for i in range(case["count"]):
        ndim = rng.choice([2, 3])
        side = _log_uniform(rng, *((64, 1024) if ndim == 2 else (32, 160)))
        shape = tuple(max(3, round(side * rng.uniform(0.8, 1.25))) for _ in range(ndim))
        out.append((rng.choice(["bumps", "bumps", "turb"]) if ndim == 3 else "bumps",
                    rng.choice(case["dtypes"].split()), shape, _log_uniform(rng, 1e-4, 1e-2),
                    "noa", seed * 1000 + i))
    return out


def _bound(x, eb, mode):
    """The bound as the caller gives it: relative to the range, or absolute."""
    return eb if mode == "noa" else eb * float(x.max().double() - x.min().double())


# ------------------------------------------------------------------ calls
def _bytes(nbytes):
    # zeroed: what lies past a stream in its buffer is then the same each time
    return torch.zeros(nbytes, dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    fs = _fields(case, seed)
    xs = [_field(kind, shape, dtype, s) for kind, dtype, shape, _, _, s in fs]
    ebs = [_bound(x, f[3], f[4]) for x, f in zip(xs, fs)]
    modes = [f[4] for f in fs]
    ctx = P.context(0)
    st = {"op": case["op"]}
    if case["op"] == "compress":
        x = xs[0]
        out = _bytes(P.lopc_compress_bound(x.shape, x.dtype))
        # the part of the buffer that holds the stream: as long as the field
        st |= {"x": x, "eb": ebs[0], "mode": modes[0], "out": out,
               "head": out[:x.numel() * x.element_size()],
               "ws": _bytes(P.lopc_workspace_size(ctx, x.shape, x.dtype, 0))}
    elif case["op"] == "decompress":
        x = xs[0]
        s, hdr = P.compress(x, ebs[0], modes[0], header=True)
        st |= {"s": s.clone(), "hdr": hdr, "out": torch.empty_like(x),
               "ws": _bytes(P.lopc_workspace_size(ctx, x.shape, x.dtype, 1))}
    elif case["op"] == "compress_batch":
        room = sum((P.lopc_compress_bound(x.shape, x.dtype) + 255) // 256 * 256 for x in xs)
        st |= {"xs": xs, "ebs": ebs, "modes": modes, "out": _bytes(room)}
    else:
        streams, hdrs = P.compress_batch(xs, ebs, modes, headers=True)
        st |= {"ss": [s.clone() for s in streams], "hdrs": hdrs,
               "outs": [torch.empty_like(x) for x in xs]}
    return st


def run(st):
    # a stream's length depends on the values, so compressions give the buffer
    # that holds the streams, of one length for a shape, and their sizes
    if st["op"] == "compress":
        s = P.compress(st["x"], st["eb"], st["mode"], out=st["out"], workspace=st["ws"])
        return st["head"], s.numel()
    if st["op"] == "decompress":
        return P.decompress(st["s"], out=st["out"], workspace=st["ws"], header=st["hdr"])
    if st["op"] == "compress_batch":
        ss = P.compress_batch(st["xs"], st["ebs"], st["modes"], out=st["out"])
        return st["out"], np.array([s.numel() for s in ss])
    return P.decompress_batch(st["ss"], outs=st["outs"], headers=st["hdrs"])


def work(case):
    # the field once and the stream once; a stream is about an eighth of its
    # field on these inputs (it depends on the values)
    n = sum(math.prod(shape) * (4 if dtype == "f32" else 8)
            for _, dtype, shape, _, _, _ in _fields(case, 0))
    return {"bytes": n + n // 8, "flops": 0}


# ------------------------------------------------------------------ exact
_EDGES = [(z, y, x) for z in (0, 1) for y in (0, 1) for x in (0, 1) if z + y + x]


def _reconstruction(x, eb, mode):
    """What decompression gives for field x: the s-th representable value
    above the lowest value of the point's bin, s the least solution of
    s(p) = max(0, max over same-bin neighbours n below p of s(n) + [n > p])."""
    eps = eb * float(x.max().double() - x.min().double()) if mode == "noa" else eb
    bins = (x.double() / eps).round_()
    b3 = bins.reshape((1,) * (3 - x.dim()) + tuple(x.shape))
    x3 = x.reshape(b3.shape)
    s = torch.zeros(b3.shape, dtype=torch.int32, device=DEV)
    pairs = []  # (lower-index end, upper-index end, same bin and lower end below, ... above)
    for off in _EDGES:
        if any(o and n < 2 for o, n in zip(off, b3.shape)):
            continue
        a = tuple(slice(0, n - o) for o, n in zip(off, b3.shape))
        c = tuple(slice(o, n) for o, n in zip(off, b3.shape))
        same = b3[a] == b3[c]
        up = x3[a] <= x3[c]  # a tie: the lower index is the smaller point
        pairs.append((a, c, same & up, same & ~up))
    before = -1
    while True:  # every pass raises; the sum stops at the least solution
        for a, c, up, down in pairs:
            s[c] = torch.maximum(s[c], s[a] * up)
            s[a] = torch.maximum(s[a], (s[c] + 1) * down)
        now = int(s.sum(dtype=torch.int64))
        if now == before:
            break
        before = now
    del pairs
    lo = ((bins - 0.5) * eps).to(x.dtype)
    whole = torch.int32 if x.dtype == torch.float32 else torch.int64
    key = lo.view(whole)
    key = torch.where(key < 0, -(key & torch.iinfo(whole).max), key)
    # lo is the lowest value of the bin or a neighbour of it
    top = (bins - 0.5) * eps

    def value(k):
        low = torch.iinfo(whole).min
        return torch.where(k < 0, (-k) | low, k).view(x.dtype)

    key += (value(key).double() < top).to(whole)
    return value(key + s.reshape(x.shape).to(whole)).double()


def exact(case, seed):
    if not case["op"].startswith("decompress"):
        return None  # a stream of bytes
    res = []
    for kind, dtype, shape, eb, mode, s in _fields(case, seed):
        x = _field(kind, shape, dtype, s)
        res.append(_reconstruction(x, _bound(x, eb, mode), mode))
    return res if case["op"] == "decompress_batch" else res[0]
