"""Workloads of the compressor that its performance is measured by.

Each case is one pass through the Python entry points on device buffers that a
program keeps (fields, streams, plans), on seeded synthetic fields of the
shapes and value structures the evaluation of the method uses: sums of sine
modes with noise, a climate-like plane with a region of exact zeros, a
hurricane-like volume with a vortex, a lognormal (cosmology-like) volume.

op:
  compress      a snapshot in device memory is compressed there
  decompress    a stream in device memory is read back
  roundtrip     both, back to back on one stream (a cached field, a restart)
  evaluate      both, then the distortion of the result (choosing a bound)
  batch         two plans over many fields of mixed rank and size, both ways

A compressed buffer is kept from pass to pass and returned up to the worst-case
stream (``stream_bound``): the stream, then the zeros it was made with.
"""
import math
import random

import numpy as np
import torch

import paper_2304_12557_amd as fz

# mean stream bits per value met on these fields (measured once, rounded): the
# size of what compression writes and decompression reads
_BITS = {"sine": {1e-2: 3.6, 1e-3: 5.5, 1e-4: 9.0}, "climate": {1e-2: 1.5, 1e-3: 3.0, 1e-4: 5.7},
         "hurricane": {1e-2: 2.3, 1e-3: 3.5, 1e-4: 5.0}, "lognormal": {1e-2: 0.7, 1e-3: 2.6, 1e-4: 5.7}}


def listed():
    return [
        # one small block of a simulation: the latency of the calls
        {"name": "sine64-roundtrip", "op": "roundtrip", "field": "sine", "nz": 64, "ny": 64, "nx": 64,
         "mode": "rel", "eb": 1e-3, "dtype": "f32"},
        # a climate field (CESM-like plane), written and read back
        {"name": "climate-compress", "op": "compress", "field": "climate", "nz": 0, "ny": 1800, "nx": 3600,
         "mode": "rel", "eb": 1e-4, "dtype": "f32"},
        {"name": "climate-decompress", "op": "decompress", "field": "climate", "nz": 0, "ny": 1800, "nx": 3600,
         "mode": "rel", "eb": 1e-4, "dtype": "f32"},
        # an ordinary weather volume (ragged against the chunk box)
        {"name": "hurricane-compress", "op": "compress", "field": "hurricane", "nz": 100, "ny": 500, "nx": 500,
         "mode": "rel", "eb": 1e-3, "dtype": "f32"},
        {"name": "hurricane-decompress", "op": "decompress", "field": "hurricane", "nz": 100, "ny": 500, "nx": 500,
         "mode": "rel", "eb": 1e-3, "dtype": "f32"},
        # a cosmology volume: the largest single calls, where bandwidth counts
        {"name": "lognormal512-compress", "op": "compress", "field": "lognormal", "nz": 512, "ny": 512, "nx": 512,
         "mode": "rel", "eb": 1e-3, "dtype": "f32"},
        {"name": "lognormal512-decompress", "op": "decompress", "field": "lognormal", "nz": 512, "ny": 512,
         "nx": 512, "mode": "rel", "eb": 1e-3, "dtype": "f32"},
        # the point-wise relative bound on a field spanning many binades
        {"name": "lognormal256-pwrel", "op": "roundtrip", "field": "lognormal", "nz": 256, "ny": 256, "nx": 256,
         "mode": "pwrel", "eb": 1e-3, "dtype": "f32"},
        # double precision output of a solver
        {"name": "hurricane-f64", "op": "roundtrip", "field": "hurricane", "nz": 100, "ny": 500, "nx": 500,
         "mode": "rel", "eb": 1e-3, "dtype": "f64"},
        # the predictor over the whole field
        {"name": "hurricane-global", "op": "roundtrip", "field": "hurricane", "nz": 100, "ny": 500, "nx": 500,
         "mode": "rel", "eb": 1e-3, "dtype": "f32", "global": True},
        # a bound tried out on a particle-like 1-D array of odd length
        {"name": "line-evaluate-abs", "op": "evaluate", "field": "sine", "nz": 0, "ny": 0, "nx": 20000003,
         "mode": "abs", "eb": 4e-3, "dtype": "f32"},
        # the fields of one time step together: mixed rank, 16 KiB to 64 MiB
        {"name": "mixed-batch", "op": "batch", "field": "sine", "count": 24, "lo": 16 << 10, "hi": 64 << 20,
         "mode": "rel", "eb": 0.0, "dtype": "f32"},
    ]


def _extents(rng, rank, n):
    """rank extents of about n values: aspect ratios log-uniform in [1/4, 4];
    a third of the shapes rounded to whole multiples of 64."""
    asp = [math.exp(rng.uniform(math.log(0.25), math.log(4.0))) for _ in range(rank - 1)]
    base = (n / math.prod(asp)) ** (1.0 / rank)
    ext = [max(1, round(base))] + [max(1, round(base * a)) for a in asp]
    if rank > 1 and rng.random() < 1 / 3:
        ext = [max(64, round(e / 64) * 64) for e in ext]
    return [0] * (3 - rank) + ext


def draw(rng):
    op = rng.choice(["compress", "compress", "decompress", "decompress", "roundtrip", "evaluate", "batch"])
    if op == "batch":
        count = rng.randint(2, 28)
        hi = rng.choice([1 << 20, 8 << 20, 32 << 20])
        return {"op": op, "field": "sine", "count": count, "lo": 16 << 10, "hi": hi, "mode": "rel", "eb": 0.0,
                "dtype": "f32", "shapes": rng.randint(0, 1 << 30)}
    kind = "plain"
    top = 2.0 ** 26.5 if op in ("compress", "decompress") else 2.0 ** 24.8
    if op == "roundtrip":
        kind = rng.choice(["plain", "pwrel", "f64", "global"])
    rank = 3 if kind == "pwrel" else rng.choice([1, 2, 3, 3])
    low = 2.0 ** 18 if kind == "pwrel" else 2.0 ** 14
    n = math.exp(rng.uniform(math.log(low), math.log(top)))
    nz, ny, nx = _extents(rng, rank, n)
    field = {1: ["sine"], 2: ["climate", "sine"], 3: ["sine", "hurricane", "lognormal"]}[rank]
    field = "lognormal" if kind == "pwrel" else rng.choice(field)
    mode = "pwrel" if kind == "pwrel" else rng.choice(["rel", "rel", "abs"])
    if field == "lognormal" and mode == "abs":  # its range spans decades: a fixed bound says little
        mode = "rel"
    eb = rng.choice([1e-2, 1e-3]) if kind == "pwrel" else rng.choice([1e-2, 1e-3, 1e-4])
    if mode == "abs":  # the fields' ranges are about 8 to 30
        eb = 10 * eb
    c = {"op": op, "field": field, "nz": nz, "ny": ny, "nx": nx, "mode": mode, "eb": eb,
         "dtype": "f64" if kind == "f64" else "f32"}
    if kind == "global":
        c["global"] = True
    return c


# ------------------------------------------------------------------- fields
def _shape(case):
    return tuple(int(v) for v in (case["nz"], case["ny"], case["nx"]) if v)


def _coords(shape):
    r = len(shape)
    return [torch.arange(n, dtype=torch.float64, device="cuda").view(*[n if d == i else 1 for d in range(r)])
            for i, n in enumerate(shape)]


def _modes(shape, count, rng, dtype=torch.float32):
    """Sum of plane-wave sine modes, wavelengths 8 to 64 cells.  The phase is
    reduced in double along each axis, the sine taken of the small sum."""
    f = torch.zeros(shape, dtype=dtype, device="cuda")
    xs = _coords(shape)
    for _ in range(count):
        amp, wl, ph = rng.uniform(0.5, 1.0), rng.uniform(8.0, 64.0), rng.uniform(0.0, 2 * math.pi)
        k = np.array([rng.gauss(0.0, 1.0) for _ in shape])
        k = 2 * math.pi / wl * k / np.linalg.norm(k)
        arg = torch.full((1,) * len(shape), ph, dtype=dtype, device="cuda")
        for kd, x in zip(k, xs):
            arg = arg + torch.remainder(float(kd) * x, 2 * math.pi).to(dtype)
        f.add_(torch.sin(arg), alpha=amp)
    return f


def _sine(shape, rng, gen, dtype=torch.float32):
    f = _modes(shape, 8, rng, dtype)
    return f.add_(torch.randn(shape, generator=gen, device="cuda", dtype=dtype), alpha=1e-3)


def _climate(shape, rng, gen, dtype=torch.float32):
    f = _modes(shape, 16, rng, dtype)
    ny, nx = shape
    h = max(1, round(ny * rng.uniform(0.3, 0.7)))
    w = min(nx, max(1, round(0.2 * ny * nx / h)))
    y0, x0 = rng.randint(0, ny - h), rng.randint(0, nx - w)
    f[y0:y0 + h, x0:x0 + w] = 0.0
    return f


def _hurricane(shape, rng, gen, dtype=torch.float32):
    f = _modes(shape, 12, rng, dtype)
    z, y, x = _coords(shape)
    x0, y0 = rng.uniform(0.3, 0.7) * shape[2], rng.uniform(0.3, 0.7) * shape[1]
    r2 = ((x - (x0 + 0.3 * z)).square().to(dtype) + (y - (y0 + 0.2 * z)).square().to(dtype))
    return f.add_(r2.sqrt() * torch.exp(-r2 / 1600.0))


def _lognormal(shape, rng, gen, dtype=torch.float32):
    w = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    W = torch.fft.rfftn(w)
    k2 = sum((torch.fft.fftfreq(n, 1.0 / n, device="cuda") if i < 2 else torch.fft.rfftfreq(n, 1.0 / n, device="cuda"))
             .view(*[-1 if d == i else 1 for d in range(3)]).square() for i, n in enumerate(shape))
    W *= torch.where(k2 >= 1.0, k2.clamp(min=1.0).pow(-0.75), torch.zeros_like(k2))
    g = torch.fft.irfftn(W, s=shape)
    g -= g.mean()
    g *= 1.5 / g.std()
    return g.to(dtype).exp_()


_FIELDS = {"sine": _sine, "climate": _climate, "hurricane": _hurricane, "lognormal": _lognormal}


def _field(case, seed):
    rng = random.Random(1000003 * int(seed) + 17)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
    return _FIELDS[case["field"]](_shape(case), rng, gen, dtype).contiguous()


def _batch_jobs(case, seed):
    """(field, bound, mode) of a batch: ranks 1 to 3, byte sizes log-uniform,
    bounds 1e-2, 1e-3 and 1e-4 of the range.  The shapes belong to the case."""
    rs = random.Random(3000 + case.get("shapes", 0))
    jobs = []
    for i in range(case["count"]):
        rank = rs.randint(1, 3)
        n = math.exp(rs.uniform(math.log(case["lo"]), math.log(case["hi"]))) / 4
        shape = tuple(e for e in _extents(rs, rank, n) if e)
        jobs.append((shape, rs.choice([1e-2, 1e-3, 1e-4]), "rel"))
    if seed is None:
        return jobs
    out = []
    for i, (shape, eb, mode) in enumerate(jobs):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed) * 1000 + i)
        out.append((_sine(shape, random.Random(1000003 * int(seed) + i), gen).contiguous(), eb, mode))
    return out


# -------------------------------------------------------------------- passes
def prepare(case, seed):
    st = {"op": case["op"]}
    if case["op"] == "batch":
        jobs = _batch_jobs(case, seed)
        bufs = [torch.zeros(fz.compress_bound(tuple(x.shape)), dtype=torch.uint8, device="cuda") for x, _, _ in jobs]
        st["c"] = fz.Batch.compress([(x, eb, mode, b) for (x, eb, mode), b in zip(jobs, bufs)])
        st["d"] = fz.Batch.decompress([(b, tuple(x.shape), None, None) for b, (x, _, _) in zip(bufs, jobs)])
        st["bounds"] = [fz.stream_bound(tuple(x.shape)) for x, _, _ in jobs]
        return st
    x = _field(case, seed)
    st.update(eb=case["eb"], mode=case["mode"], glob=bool(case.get("global")), shape=tuple(x.shape))
    st["buf"] = torch.zeros(fz.compress_bound(st["shape"], f64=x.dtype == torch.float64, global_lorenzo=st["glob"]),
                            dtype=torch.uint8, device="cuda")
    st["bound"] = fz.stream_bound(st["shape"])
    if case["op"] == "decompress":  # the stream alone is in memory
        fz.compress(x, st["eb"], st["mode"], out=st["buf"])
        st["s"] = st["buf"][:fz.stream_size(st["buf"])].clone()
        del st["buf"]
    else:
        st["x"] = x
    if case["op"] != "compress":
        st["y"] = torch.empty_like(x)
    if st["glob"]:
        n = int(fz.lib().fz_decompress_global_work_bytes(fz.dims_of(st["shape"])))
        st["work"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    if case["op"] == "evaluate":
        st["err"] = torch.empty(1, dtype=torch.int32, device="cuda")
    return st


def run(st):
    op = st["op"]
    if op == "batch":
        streams = st["c"].run()
        fields = st["d"].run()
        return [{"stream": s[:n], "y": y} for s, n, y in zip(streams, st["bounds"], fields)]
    if op == "decompress":
        return fz.decompress(st["s"], st["shape"], out=st["y"])
    s = fz.compress(st["x"], st["eb"], st["mode"], out=st["buf"], global_lorenzo=st["glob"])
    if op == "compress":
        return s[:st["bound"]]
    y = fz.decompress(s, st["shape"], out=st["y"], err=st.get("err"), global_lorenzo=st["glob"], work=st.get("work"))
    got = {"stream": s[:st["bound"]], "y": y}
    if op == "evaluate":
        got["err"] = st["err"]
        got["quality"] = fz.quality(st["x"], y)
    return got


def _bits(field, mode, eb):
    if mode == "pwrel":
        return 12.8 if eb < 5e-3 else 9.3
    if mode == "abs":
        eb = eb / 10
    t = _BITS[field]
    return t[min(t, key=lambda e: abs(math.log(e / eb)))]


def work(case):
    """One read of the field and one write of the stream, and the reverse."""
    if case["op"] == "batch":
        each = [(math.prod(s), _bits("sine", m, eb)) for s, eb, m in _batch_jobs(case, None)]
        return {"bytes": sum(2 * (4 * n + n * b / 8) for n, b in each), "flops": 0}
    n = math.prod(_shape(case))
    f = (8 if case["dtype"] == "f64" else 4) * n
    s = n * _bits(case["field"], case["mode"], case["eb"]) / 8
    return {"bytes": {"compress": f + s, "decompress": f + s, "roundtrip": 2 * (f + s),
                      "evaluate": 2 * (f + s) + 2 * f}[case["op"]], "flops": 0}


# ---------------------------------------------------------------- 64-bit values
def _exact_field(x, eb, mode):
    if mode == "pwrel":  # the bit pattern as a piecewise-linear logarithm, on a grid of step s
        s = math.floor(eb * 2.0 ** 24 / (1.0 + eb))
        bits = x.view(torch.int32).to(torch.int64)
        q = torch.div((bits & 0x7FFFFFFF) + s // 2, s, rounding_mode="floor")
        y = torch.clamp(q * s, max=0x7F7FFFFF).to(torch.int32).view(torch.float32).double()
        return torch.where(x < 0, -y, y)
    x = x.double()
    step = 2.0 * (eb * float(x.max() - x.min()) if mode == "rel" else eb)
    return torch.round(x / step) * step


def exact(case, seed):
    op = case["op"]
    if op == "compress":
        return None
    if op == "batch":
        return [{"stream": None, "y": _exact_field(*job)} for job in _batch_jobs(case, seed)]
    x = _field(case, seed)
    y = _exact_field(x, case["eb"], case["mode"])
    if op == "decompress":
        return y
    got = {"stream": None, "y": y}
    if op == "evaluate":
        x = x.double()
        d = (x - y).abs()
        mse = float(d.square().mean())
        lo, hi = float(x.min()), float(x.max())
        got["err"] = None
        got["quality"] = {"max_abs_err": float(d.max()), "mse": mse, "n": x.numel(), "nonfinite": 0,
                          "psnr": 20 * math.log10(hi - lo) - 10 * math.log10(mse), "vmin": lo, "vmax": hi}
    return got
