"""Performance cases of the multi-component progressive codec.

listed() names the cases, draw() makes more of the same ranges, prepare()
builds what a program holds before the call (fields on the device, stores,
plans, a server), run() is one pass through the public entry points, work()
the bytes and operations such a pass cannot do without, exact() the values
plain torch gives in 64 bits where outputs have such values.

Fields are the repository's synthetic ones (random-phase spectral fields with
shell spectrum k^(-5/3) on [-1, 1], optionally with white noise; for the small
one Gaussian blobs with sinusoids), drawn on the device so that large ones are
quick.  A case is a dict of plain values:

  op         what a pass does (run below)
  nx, ny, nz field extents, x fastest;  dtype "f32" or "f64"
  n          components;  step: tau_i = scale * step^-i, where scale is the
             field's range if relative is true, else 1
  k          components retrieved;  noise: white noise relative to the range
  codec      0 the block transform, 1 prediction and quantisation
  shapes_seed, count, lo, hi
             the fields of a batch or a served set: edges log-uniform in
             [lo, hi] (per axis in a batch, cubes when served), types
             alternating
"""
import math
import random
import time

import torch

from paper_2308_11759_amd import pmc


def listed():
    return [
        # a small snapshot (the 64^3 workload) written and read back at full
        # accuracy: calls where launches and the host round trips weigh most
        dict(name="small_cycle_f64", op="cycle", field="blobs", nx=64, ny=64, nz=64, dtype="f64", n=4, step=10.0,
             relative=True, noise=0.0, k=4, codec=0),
        # the bulk workload (512^3 float32, 8 components): writing a large
        # simulation snapshot; range for the schedule, then Alg. 1
        dict(name="bulk_compress_f32", op="compress", field="spectral", nx=512, ny=512, nz=512, dtype="f32", n=8,
             step=8.0, relative=False, noise=0.0),
        # ... and reading it at full accuracy (Alg. 2, all components)
        dict(name="bulk_retrieve_f32", op="retrieve", field="spectral", nx=512, ny=512, nz=512, dtype="f32", n=8,
             step=8.0, relative=False, noise=0.0, k=8),
        # the bulk float64 workload (256^3, 8 components), both directions
        dict(name="bulk_compress_f64", op="compress", field="spectral", nx=256, ny=256, nz=256, dtype="f64", n=8,
             step=8.0, relative=False, noise=0.0),
        dict(name="bulk_retrieve_f64", op="retrieve", field="spectral", nx=256, ny=256, nz=256, dtype="f64", n=8,
             step=8.0, relative=False, noise=0.0, k=8),
        # a ragged field (no extent a multiple of 4) with a noise floor, as a
        # measured field has: late components code noise
        dict(name="ragged_compress_f32", op="compress", field="spectral", nx=251, ny=203, nz=181, dtype="f32", n=10,
             step=4.0, relative=True, noise=1e-4),
        # progressive refinement of a ragged field component by component, as
        # a viewer does: x~_1, then each next component added in place
        dict(name="ragged_refine_f32", op="refine", field="spectral", nx=251, ny=203, nz=181, dtype="f32", n=6,
             step=4.0, relative=True, noise=0.0, k=6),
        # a 64^3 region out of the bulk field, only its blocks decoded
        dict(name="region_f32", op="region", field="spectral", nx=512, ny=512, nz=512, dtype="f32", n=8, step=8.0,
             relative=False, noise=0.0, k=8, box=64),
        # the batched workload's mix (edges 16 to 256 per axis, types
        # alternating, 6 components, tau_i = range 4^-i) in one planned call,
        # with the schedule that its tuner picks
        dict(name="batch_mixed", op="batch", shapes_seed=100, count=24, lo=16, hi=256, n=6, step=4.0, relative=True,
             noise=0.0),
        # the served workload's mix (cubes from 64 up, types alternating, 10
        # components, tau_i = range 10^(-i/2)): a burst of queries at mixed
        # tolerances, with memory for part of the partial sums only
        dict(name="served_burst", op="serve", shapes_seed=200, count=8, lo=64, hi=224, n=10,
             step=math.sqrt(10.0), relative=True, noise=0.0, queries=32),
        # the second compressor behind the same driver (prediction and
        # quantisation): a field written and read back
        dict(name="prediction_cycle_f32", op="cycle", field="spectral", nx=256, ny=256, nz=256, dtype="f32", n=8,
             step=8.0, relative=False, noise=0.0, k=8, codec=1),
        # a saved snapshot brought back from host memory and read
        dict(name="load_f32", op="load", field="spectral", nx=160, ny=144, nz=130, dtype="f32", n=6, step=4.0,
             relative=True, noise=0.0, k=6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["compress", "compress", "retrieve", "retrieve", "refine", "region", "batch", "serve", "cycle", "load"])
    step, relative = rng.choice([(8.0, False), (4.0, True), (4.0, False), (10.0, True), (math.sqrt(10.0), True)])
    case = dict(op=op, step=step, relative=relative, noise=rng.choice([0.0, 0.0, 1e-4]))
    if op == "batch":
        case.update(shapes_seed=rng.randrange(1000, 100000), count=rng.randrange(6, 25), lo=16, hi=192,
                    n=rng.randrange(2, 7))
        return case
    if op == "serve":
        case.update(shapes_seed=rng.randrange(1000, 100000), count=rng.randrange(3, 9), lo=64, hi=192,
                    n=rng.randrange(3, 11), queries=rng.randrange(8, 33))
        return case
    f64 = rng.random() < 0.5
    # one volume over the whole range, split unevenly over the axes; two
    # draws in five are multiples of 4 in every extent
    top = 160.0 if op == "load" else 320.0 if f64 else 480.0
    vol = math.exp(rng.uniform(math.log(16.0 ** 3), math.log(top ** 3)))
    edge = vol ** (1.0 / 3.0)
    ax, ay = rng.uniform(0.7, 1.4), rng.uniform(0.7, 1.4)
    dims = [max(5, int(round(edge * a))) for a in (ax, ay, 1.0 / (ax * ay))]
    if rng.random() < 0.4:
        dims = [max(8, d // 4 * 4) for d in dims]
    case.update(field="spectral", nx=dims[0], ny=dims[1], nz=dims[2], dtype="f64" if f64 else "f32",
                n=rng.randrange(2, 9))
    if not f64:  # tolerances down to float32's spacing
        case["n"] = min(case["n"], int(24.0 / math.log2(step) + 1e-9))
    if op in ("retrieve", "region", "cycle", "load"):
        case["k"] = rng.randrange(1, case["n"] + 1)
    if op == "refine":
        case["k"] = case["n"]
    if op == "region":
        case["box"] = max(1, min(min(dims), _log_int(rng, 5, 128)))
    if op == "cycle":
        case["codec"] = rng.randrange(2)
    return case


# ---------------------------------------------------------------------------
# inputs

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _spectral(shape, dtype, seed, noise):
    """Random-phase field, |k|^(-11/6) amplitudes, affinely on [-1, 1]."""
    nz, ny, nx = shape
    g = _gen(seed)
    kz = (torch.fft.fftfreq(nz, device="cuda", dtype=torch.float64) * nz)[:, None, None]
    ky = (torch.fft.fftfreq(ny, device="cuda", dtype=torch.float64) * ny)[None, :, None]
    kx = (torch.fft.rfftfreq(nx, device="cuda", dtype=torch.float64) * nx)[None, None, :]
    k2 = kz * kz + ky * ky + kx * kx
    k2[0, 0, 0] = 1.0
    amp = k2.pow_(-11.0 / 12.0)
    amp[0, 0, 0] = 0.0
    phase = torch.rand(amp.shape, generator=g, device="cuda", dtype=torch.float64).mul_(2.0 * math.pi)
    f = torch.fft.irfftn(torch.polar(amp, phase), s=(nz, ny, nx))
    del amp, phase, k2
    lo, hi = f.min(), f.max()
    f = ((f - lo) * (2.0 / (hi - lo)) - 1.0).clamp_(-1.0, 1.0)
    if noise > 0.0:
        f += torch.randn(f.shape, generator=g, device="cuda", dtype=torch.float64).mul_(noise * 2.0)
    return f.to(dtype).contiguous()


def _blobs(shape, dtype, seed):
    """Gaussian blobs, three sinusoids and a little white noise."""
    nz, ny, nx = shape
    g = _gen(seed)
    z = torch.arange(nz, device="cuda", dtype=torch.float64)[:, None, None]
    y = torch.arange(ny, device="cuda", dtype=torch.float64)[None, :, None]
    x = torch.arange(nx, device="cuda", dtype=torch.float64)[None, None, :]
    u = torch.rand(16, 5, generator=g, device="cuda", dtype=torch.float64).tolist()
    f = torch.zeros(shape, device="cuda", dtype=torch.float64)
    for a, s, cx, cy, cz in u:
        r2 = (x - cx * nx) ** 2 + (y - cy * ny) ** 2 + (z - cz * nz) ** 2
        f += (2.0 * a - 1.0) * torch.exp(-r2 / (2.0 * (2.0 + 8.0 * s) ** 2))
    v = torch.rand(3, 5, generator=g, device="cuda", dtype=torch.float64).tolist()
    for a, b, c, d, ph in v:
        kx, ky, kz = 1 + int(4 * b), int(5 * c), int(5 * d)
        f += (a - 0.5) * torch.sin(2.0 * math.pi * (kx * x / nx + ky * y / ny + kz * z / nz + ph))
    f += torch.randn(shape, generator=g, device="cuda", dtype=torch.float64).mul_(1e-3)
    return f.to(dtype).contiguous()


def _field(case, seed):
    shape = (case["nz"], case["ny"], case["nx"])
    if case["field"] == "blobs":
        return _blobs(shape, _dtype(case), seed)
    return _spectral(shape, _dtype(case), seed, case["noise"])


def _shapes(case):
    """(shape, dtype) of the fields of a batch or a served set."""
    rng = random.Random(case["shapes_seed"])
    out = []
    for i in range(case["count"]):
        if case["op"] == "serve":
            e = _log_int(rng, case["lo"], case["hi"])
            dims = (e, e, e)
        else:
            dims = tuple(_log_int(rng, case["lo"], case["hi"]) for _ in range(3))
        out.append((dims, torch.float32 if i % 2 == 0 else torch.float64))
    return out


def _queries(case):
    """(field, component count asked for) of a burst."""
    rng = random.Random(case["shapes_seed"] + 1)
    return [(rng.randrange(case["count"]), rng.randrange(1, case["n"] + 1)) for _ in range(case["queries"])]


def _fields(case, seed):
    return [_spectral(s, dt, seed * 1000 + i, case["noise"]) for i, (s, dt) in enumerate(_shapes(case))]


def _scale(case, x):
    return float(x.max()) - float(x.min()) if case["relative"] else 1.0


def _taus(case, scale):
    return [scale * case["step"] ** -(i + 1) for i in range(case["n"])]


# ---------------------------------------------------------------------------
# a program's state and one pass over it

def _stored(ctx, case, x):
    """A store whose stream buffer is no larger than its streams need (what a
    program keeps when it holds many stores)."""
    store = ctx.compress(x, _taus(case, _scale(case, x)))
    return ctx.deserialize(store.serialize())


def _stream_buffer(case):
    """A stream buffer for one field: the block indexes and n streams at the
    rate these fields have, with a margin (a fixed capacity, as a program that
    knows its data gives one; the library refuses a buffer that is too small).
    Zeroed once, so that the alignment gaps between streams are defined."""
    blocks = 1
    for a in ("nx", "ny", "nz"):
        blocks *= (case[a] + 3) // 4
    n = case["n"]
    payload = blocks * 64 * (1.25 * _bits(case, n) + 6.0) / 8.0
    return torch.zeros(int(payload) + n * (5 * blocks + 2048), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    op = case["op"]
    ctx = pmc.Context(0)
    st = dict(op=op, ctx=ctx, case=case)
    if op == "compress":
        x = _field(case, seed)
        st["x"] = x
        st["streams"] = _stream_buffer(case)
    elif op in ("retrieve", "refine", "region"):
        x = _field(case, seed)
        st["store"] = _stored(ctx, case, x)
        if op == "region":
            b = case["box"]
            ext = (case["nx"], case["ny"], case["nz"])
            st["lo"] = [(e - b) // 2 for e in ext]
            st["hi"] = [lo + b for lo in st["lo"]]
            st["out"] = torch.empty((b, b, b), dtype=x.dtype, device="cuda")
        else:
            st["out"] = torch.empty_like(x)
    elif op == "batch":
        xs = _fields(case, seed)
        st["xs"] = xs
        st["batch"] = ctx.batch([(tuple(x.shape), x.dtype) for x in xs], [_taus(case, _scale(case, x)) for x in xs])
        st["batch"].schedule(8, 2)
        st["streams"] = torch.zeros_like(st["batch"].streams)
    elif op == "serve":
        xs = _fields(case, seed)
        stores = [_stored(ctx, case, x) for x in xs]
        scales = [_scale(case, x) for x in xs]
        queries = [(f, scales[f] * case["step"] ** -k * 1.01) for f, k in _queries(case)]
        total = sum(x.numel() * x.element_size() for x in xs)
        largest = max(x.numel() * x.element_size() for x in xs)
        outs = [torch.empty_like(xs[f]) for f, _ in queries]
        running = sum(o.numel() * o.element_size() for o in outs)
        # budget: the burst's outputs, and cached partial sums of about two
        # components' worth of the fields (of n)
        arena = (64 << 20) + largest + 2 * total
        srv = pmc.Server(ctx, arena_bytes=arena, budget_bytes=arena + running, max_batch=64)
        st.update(srv=srv, ids=[srv.add(s) for s in stores], stores=stores, queries=queries, outs=outs)
    elif op == "load":
        x = _field(case, seed)
        st["blob"] = ctx.compress(x, _taus(case, _scale(case, x))).serialize()
        st["loaded"] = torch.empty(ctx.deserialize(st["blob"]).streams.numel(), dtype=torch.uint8, device="cuda")
        st["out"] = torch.empty_like(x)
    else:  # cycle
        x = _field(case, seed)
        st["x"] = x
        ctx.set_option(pmc.OPT_CODEC, case["codec"])
        st["streams"] = _stream_buffer(case)
        st["out"] = torch.empty_like(x)
    torch.cuda.synchronize()
    return st


def run(st):
    op, ctx, case = st["op"], st["ctx"], st["case"]
    if op == "compress":
        lo, hi, bad = ctx.range(st["x"])
        store = ctx.compress(st["x"], _taus(case, hi - lo if case["relative"] else 1.0), streams=st["streams"])
        return dict(range=[lo, hi], nonfinite=bad, linf=[c["linf"] for c in store.info],
                    bytes=[c["bytes"] for c in store.info], streams=st["streams"])
    if op == "retrieve":
        return ctx.retrieve(st["store"], case["k"], out=st["out"])
    if op == "refine":
        for k in range(case["k"]):
            ctx.refine(st["store"], k, k + 1, st["out"])
        return st["out"]
    if op == "region":
        return ctx.retrieve_box(st["store"], case["k"], st["lo"], st["hi"], out=st["out"])
    if op == "batch":
        stores = st["batch"].compress(st["xs"], streams=st["streams"])
        return dict(streams=st["streams"], fields=len(stores))
    if op == "serve":
        # the outputs of the burst before are reused by the server's stream:
        # what the program still does with them has to end first
        torch.cuda.current_stream().synchronize()
        srv = st["srv"]
        tickets = [srv.submit(st["ids"][f], tol, out=o) for (f, tol), o in zip(st["queries"], st["outs"])]
        for t in tickets:
            while not srv.poll(t)[0]:
                time.sleep(0)
        for t in tickets:
            srv.release(t)
        return list(st["outs"])
    if op == "load":
        return ctx.retrieve(ctx.deserialize(st["blob"], streams=st["loaded"]), case["k"], out=st["out"])
    # cycle: write the field, read it back
    lo, hi, _ = ctx.range(st["x"])
    store = ctx.compress(st["x"], _taus(case, hi - lo if case["relative"] else 1.0), streams=st["streams"])
    ctx.retrieve(store, case["k"], out=st["out"])
    return dict(streams=st["streams"], out=st["out"])


# ---------------------------------------------------------------------------
# what a pass cannot do without

# integer operations per value and component: three 4-point lifts (12 to 15
# operations per 4 values each), the quantisation or its inverse, the sum
OPS_PER_VALUE = 14


def _bits(case, ncomp):
    """Stream bits per value of the first ncomp components: the codec spends
    log2(step) bits of accuracy plus about 1.2 per component on these fields."""
    return ncomp * (math.log2(case["step"]) + 1.2)


def work(case):
    op = case["op"]
    if op in ("batch", "serve"):
        shapes = _shapes(case)
        vals = [a * b * c for (a, b, c), _ in shapes]
        size = [4 if dt == torch.float32 else 8 for _, dt in shapes]
        if op == "batch":
            by = sum(v * (s + _bits(case, case["n"]) / 8.0) for v, s in zip(vals, size))
            return {"bytes": int(by), "flops": int(sum(vals) * case["n"] * OPS_PER_VALUE)}
        per = case["queries"] / float(len(vals))
        half = (case["n"] + 1) / 2.0
        by = per * sum(v * (s + _bits(case, half) / 8.0) for v, s in zip(vals, size))
        return {"bytes": int(by), "flops": int(per * sum(vals) * half * OPS_PER_VALUE)}
    s = 4 if case["dtype"] == "f32" else 8
    vals = case["nx"] * case["ny"] * case["nz"]
    if op == "compress":
        # the range has to be known before the first component: x twice
        # where the schedule is relative to it
        reads = 2 if case["relative"] else 1
        return {"bytes": int(vals * (reads * s + _bits(case, case["n"]) / 8.0)),
                "flops": int(vals * case["n"] * OPS_PER_VALUE)}
    if op == "refine":
        k = case["k"]
        return {"bytes": int(vals * ((2 * k - 1) * s + _bits(case, k) / 8.0)), "flops": int(vals * k * OPS_PER_VALUE)}
    if op == "region":
        vals = case["box"] ** 3
    k = case["k"]
    by, ops = vals * (s + _bits(case, k) / 8.0), vals * k * OPS_PER_VALUE
    if op == "cycle":
        by += vals * ((2 if case["relative"] else 1) * s + _bits(case, case["n"]) / 8.0)
        ops += vals * case["n"] * OPS_PER_VALUE
    if op == "load":  # every component comes from the host, and is written
        by += 2 * vals * _bits(case, case["n"]) / 8.0
    return {"bytes": int(by), "flops": int(ops)}


def exact(case, seed):
    """The range is min and max in float64.  A reconstruction has the field
    itself as the value it stands for; streams and measured errors have no
    value outside the codec."""
    op = case["op"]
    if op == "batch":
        return None
    if op == "serve":
        xs = _fields(case, seed)
        return [xs[f].double() for f, _ in _queries(case)]
    x = _field(case, seed).double()
    n = case["n"]
    if op == "compress":
        return dict(range=[float(x.min()), float(x.max())], nonfinite=0, linf=[None] * n, bytes=[None] * n, streams=None)
    if op == "region":
        b = case["box"]
        z, y, w = ((e - b) // 2 for e in (case["nz"], case["ny"], case["nx"]))
        return x[z:z + b, y:y + b, w:w + b].contiguous()
    if op == "cycle":
        return dict(streams=None, out=x)
    return x
