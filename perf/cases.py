"""What this package is measured on: transforms as a program calls them.

Six kinds of call, each through the package's Python entry points:

* ``rows``   many independent 1-D transforms of 2^4 .. 2^14 points (the
             lengths of the paper's Table 1 that fit one workgroup);
* ``split``  1-D transforms of 2^15 .. 2^22 points (two global passes);
* ``cube``   one 1-D transform of 2^25 or 2^26 points (three global passes);
* ``image``  2-D transforms of one or several images;
* ``many``   transforms of uneven lengths packed back to back;
* ``grad``   the differentiable transform and its backward.

``dir`` is ``fwd``, ``inv`` or ``both`` (forward, then the inverse of its
result, as a filter in the frequency domain does).  ``keep``: the program
keeps its result buffer from call to call; otherwise each call returns a new
one.  ``plan`` (``many`` only): the program holds the plan and executes it.
"""
import math
import random

import torch

from paper_1707_07263_amd import api, capi

_DT = {"c64": torch.complex64, "f16": torch.float16, "bf16": torch.bfloat16}
_CDT = {"c64": capi.FFT_C64, "f16": capi.FFT_C16F, "bf16": capi.FFT_C16BF}
MAX_POINTS = 1 << 24  # of a drawn case other than a cube


def _lines(name, kind, n, batch, dtype="c64", dir="fwd", keep=False):
    return {"name": name, "kind": kind, "n": n, "batch": batch, "dtype": dtype, "dir": dir, "keep": keep}


def _many(name, count, lo, hi, sizes_seed, dtype="c64", dir="fwd", plan=False):
    return {"name": name, "kind": "many", "count": count, "lo": lo, "hi": hi, "sizes_seed": sizes_seed,
            "dtype": dtype, "dir": dir, "plan": plan}


def listed():
    return [
        # one short signal: the latency of a call (the paper's single transforms)
        _lines("line-1024", "rows", 1024, 1),
        # very many short signals, an odd number of them (range or Doppler
        # bins of a radar frame)
        _lines("rows-64", "rows", 64, 100003),
        # azimuth lines of a SAR scene ("tens of thousands" of points) taken back
        _lines("rows-16384", "rows", 16384, 1001, dir="inv"),
        # recorded 16-bit samples, range lines
        _lines("rows-2048-f16", "rows", 2048, 6007, dtype="f16"),
        # long signals forward and back: the benchmark's step
        _lines("step-1048576", "split", 1 << 20, 16, dir="both", keep=True),
        # long signals in bfloat16 storage, there and back, an odd batch
        _lines("split-262144-bf16", "split", 1 << 18, 37, dtype="bf16", dir="both"),
        # one signal too long for two passes
        _lines("cube-67108864", "cube", 1 << 26, 1),
        # the paper's remote-sensing image
        {"name": "image-4096", "kind": "image", "rows": 4096, "cols": 4096, "batch": 1, "dtype": "c64",
         "dir": "fwd", "keep": False},
        # a stack of oblong tiles brought back from the frequency domain
        {"name": "images-512x2048", "kind": "image", "rows": 512, "cols": 2048, "batch": 9, "dtype": "c64",
         "dir": "inv", "keep": False},
        # signals of uneven lengths collected into one call
        _many("many-512", 512, 8, 16, 3),
        # a server that holds its plan: many shorter uneven signals in fp16
        _many("many-1000-f16", 1000, 4, 13, 5, dtype="f16", plan=True),
        # a layer inside a trained model: forward and adjoint
        {"name": "grad-65536", "kind": "grad", "n": 1 << 16, "batch": 64},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batch(rng, n):
    return max(1, _log_uniform(rng, 1, max(1, MAX_POINTS // n)))


def draw(rng):
    kind = rng.choices(["rows", "split", "cube", "image", "many", "grad"], [30, 24, 4, 18, 14, 10])[0]
    dtype = rng.choices(["c64", "f16", "bf16"], [60, 20, 20])[0]
    dir = rng.choice(["fwd", "inv", "both"])
    keep = rng.random() < 0.5
    if kind == "rows":
        n = 1 << rng.randint(4, 14)
        return {"kind": kind, "n": n, "batch": _batch(rng, n), "dtype": dtype, "dir": dir, "keep": keep}
    if kind == "split":
        n = 1 << rng.randint(15, 22)
        return {"kind": kind, "n": n, "batch": _batch(rng, n), "dtype": dtype, "dir": dir, "keep": keep}
    if kind == "cube":
        return {"kind": kind, "n": 1 << rng.randint(25, 26), "batch": 1, "dtype": dtype,
                "dir": rng.choice(["fwd", "inv"]), "keep": keep}
    if kind == "image":
        r, c = 1 << rng.randint(5, 12), 1 << rng.randint(5, 12)
        return {"kind": kind, "rows": r, "cols": c, "batch": _batch(rng, r * c), "dtype": dtype, "dir": dir,
                "keep": keep}
    if kind == "many":
        lo = rng.randint(4, 10)
        hi = rng.randint(lo + 1, 16)
        mean = ((1 << (hi + 1)) - (1 << lo)) / (hi - lo + 1)
        count = _log_uniform(rng, 3, max(4, min(2000, MAX_POINTS / mean)))
        return {"kind": kind, "count": count, "lo": lo, "hi": hi, "sizes_seed": rng.randint(0, 1 << 20),
                "dtype": dtype, "dir": rng.choice(["fwd", "inv"]), "plan": rng.random() < 0.5}
    n = 1 << rng.randint(6, 18)
    return {"kind": "grad", "n": n, "batch": _batch(rng, n)}


def _sizes(case):
    r = random.Random(case["sizes_seed"])
    return [1 << r.randint(case["lo"], case["hi"]) for _ in range(case["count"])]


def _shape(case):
    if case["kind"] == "image":
        return (case["batch"], case["rows"], case["cols"])
    if case["kind"] == "many":
        return (sum(_sizes(case)),)
    return (case["batch"], case["n"])


def _normal(shape, dtype, g):
    """re, im ~ N(0, 1)."""
    x = torch.randn(tuple(shape) + (2,), generator=g, device="cuda", dtype=torch.float32)
    return torch.view_as_complex(x) if dtype == "c64" else x.to(_DT[dtype])


def _speckle(shape, dtype, g):
    """SAR-like: a smooth amplitude field times Exp(1) speckle, uniform phase."""
    b, r, c = shape
    u = torch.rand(4, b, 4, generator=g, device="cuda", dtype=torch.float32)
    y = torch.arange(r, device="cuda", dtype=torch.float32)[None, None, :] / r
    x = torch.arange(c, device="cuda", dtype=torch.float32)[None, None, :] / c
    width = 0.05 + 0.2 * u[2][..., None]
    fy = torch.exp(-((y - u[0][..., None]) / width) ** 2) * (0.5 + u[3][..., None])
    fx = torch.exp(-((x - u[1][..., None]) / width) ** 2)
    field = (fy[:, :, :, None] * fx[:, :, None, :]).sum(1) + 0.1
    amp = field * torch.empty_like(field).exponential_(1.0, generator=g)
    amp /= amp.square().mean().sqrt()
    phase = torch.rand(shape, generator=g, device="cuda", dtype=torch.float32) * (2 * math.pi)
    z = torch.stack([amp * torch.cos(phase), amp * torch.sin(phase)], dim=-1)
    return torch.view_as_complex(z) if dtype == "c64" else z.to(_DT[dtype])


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    if case["kind"] == "image":
        return _speckle(_shape(case), case["dtype"], g), None
    if case["kind"] == "grad":
        return _normal(_shape(case), "c64", g), _normal(_shape(case), "c64", g)
    return _normal(_shape(case), case["dtype"], g), None


def prepare(case, seed):
    x, up = _inputs(case, seed)
    s = {"case": dict(case), "x": x}
    kind = case["kind"]
    if kind == "grad":
        s["x"] = x.requires_grad_(True)
        s["up"] = up
    elif kind == "many":
        s["sizes"] = _sizes(case)
        s["inverse"] = case["dir"] == "inv"
        if case["plan"]:
            s["plan"] = api.get_many_plan(s["sizes"], _CDT[case["dtype"]],
                                          capi.FFT_INVERSE if s["inverse"] else capi.FFT_FORWARD)
            s["out"] = torch.empty_like(x)
    else:
        calls = 2 if case["dir"] == "both" else 1
        s["out"] = [torch.empty_like(x) if case["keep"] else None for _ in range(calls)]
        s["fft"] = api.fft2 if kind == "image" else api.fft
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "grad":
        y = api.fft_autograd(s["x"])
        (gx,) = torch.autograd.grad(y, s["x"], s["up"])
        return {"y": y.detach(), "grad": gx}
    if case["kind"] == "many":
        if case["plan"]:
            s["plan"].exec(s["x"], s["out"])
            return s["out"]
        return api.fft_many(s["x"], s["sizes"], inverse=s["inverse"])
    f, out = s["fft"], s["out"]
    if case["dir"] == "both":
        y = f(s["x"], out=out[0])
        return {"y": y, "z": f(y, inverse=True, out=out[1])}
    return f(s["x"], inverse=case["dir"] == "inv", out=out[0])


def work(case):
    """Each call reads every point once and writes every point once."""
    points = math.prod(_shape(case))
    calls = 2 if case["kind"] == "grad" or case.get("dir") == "both" else 1
    size = 8 if case.get("dtype", "c64") == "c64" else 4
    if case["kind"] == "many":
        flops = sum(5.0 * n * math.log2(n) for n in _sizes(case))
    else:
        n = case["rows"] * case["cols"] if case["kind"] == "image" else case["n"]
        flops = 5.0 * points * math.log2(n)
    return {"bytes": 2.0 * size * points * calls, "flops": flops * calls}


def exact(case, seed):
    x, up = _inputs(case, seed)
    wide = x.to(torch.complex128) if x.is_complex() else torch.view_as_complex(x.to(torch.float64))
    kind = case["kind"]
    if kind == "grad":
        n = case["n"]
        return {"y": torch.fft.fft(wide), "grad": torch.fft.ifft(up.to(torch.complex128)) * n}

    def pack(z):
        return z if x.is_complex() else torch.view_as_real(z)

    if kind == "many":
        f = torch.fft.ifft if case["dir"] == "inv" else torch.fft.fft
        sizes = _sizes(case)
        at = [0]
        for n in sizes:
            at.append(at[-1] + n)
        out = torch.empty_like(wide)
        for n in sorted(set(sizes)):
            mine = [a for a, m in zip(at, sizes) if m == n]
            z = f(torch.stack([wide[a:a + n] for a in mine]))
            for i, a in enumerate(mine):
                out[a:a + n] = z[i]
        return pack(out)
    dims = (-2, -1) if kind == "image" else (-1,)
    if case["dir"] == "both":
        return {"y": pack(torch.fft.fftn(wide, dim=dims)), "z": pack(wide)}
    f = torch.fft.ifftn if case["dir"] == "inv" else torch.fft.fftn
    return pack(f(wide, dim=dims))
