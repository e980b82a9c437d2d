"""Performance cases: what a user of this library has it do, through its public entry points.

A case is a dict of plain values with a "kind":

  nest     one planned nest run on the current stream (Plan.run)
  static   one nest through the allocation-free one-call entry point (reduce_static)
  ordered  an ordered product of affine maps or 2x2 matrices modulo 2^64 (Plan.run)
  stencil  five-point Jacobi sweeps of a 2-D array (Stencil.run)
  batch    many uneven nests in one persistent launch (Batch.run)
  serve    a burst of requests through the continuous-batching server

Shapes are part of the case; only values depend on the seed.  Integer extents of a
nest are written "64x128x64x64", its operators "NONE,SUM,MAX,ARGMIN".
"""
import math
import os
import random
import weakref

import numpy as np
import torch

import paper_2309_01906_amd as hp

DTYPES = {"i32": hp.I32, "f32": hp.F32, "bf16": hp.BF16, "affine": hp.AFFINE64, "mat2": hp.MAT2X2_64}
ELEM_BYTES = {"i32": 4, "f32": 4, "bf16": 2, "affine": 16, "mat2": 32}


def listed():
    return [
        # The smallest call: a tight loop, or code under capture, that may not allocate.
        {"name": "static_small_f32", "kind": "static", "extents": "64x16x64", "ops": "NONE,SUM,SUM", "dtype": "f32",
         "f32_out": False},
        # Row sums of a small integer array: the two-level benchmark nest, bound by latency.
        {"name": "rows_i32_4mib", "kind": "nest", "extents": "1024x1024", "ops": "NONE,SUM", "dtype": "i32",
         "low": -1000, "high": 1000},
        # A different operator on every level: the four-level benchmark nest.
        {"name": "chain_i32_128mib", "kind": "nest", "extents": "64x128x64x64", "ops": "NONE,SUM,MAX,ARGMIN",
         "dtype": "i32", "low": 0, "high": 1 << 20},
        # The same kind of nest with the sizes that real data has: nothing a power of two.
        {"name": "odd_chain_i32", "kind": "nest", "extents": "61x125x67x59", "ops": "NONE,SUM,MAX,ARGMIN",
         "dtype": "i32", "low": -1000, "high": 1000},
        # The index of the largest row sum in each group: an ARG level over 64-bit sums.
        {"name": "argmax_of_sums_i32", "kind": "nest", "extents": "1024x64x1024", "ops": "NONE,ARGMAX,SUM",
         "dtype": "i32", "low": -1000, "high": 1000},
        # The headline benchmark nest: 1 GiB of fp32, a sum of sums per output.
        {"name": "nest_f32_1gib", "kind": "nest", "extents": "4096x256x256", "ops": "NONE,SUM,SUM", "dtype": "f32",
         "f32_out": False},
        # Rows that are no multiple of a vector, fp32 results.
        {"name": "odd_rows_f32", "kind": "nest", "extents": "1500x30011", "ops": "NONE,SUM", "dtype": "f32",
         "f32_out": True},
        # The sum of a whole array: one output, split over the grid.
        {"name": "total_bf16", "kind": "nest", "extents": "1x134217728", "ops": "NONE,SUM", "dtype": "bf16",
         "f32_out": False},
        # End states of long linear recurrences: ordered products of affine maps.
        {"name": "recurrences_affine", "kind": "ordered", "extents": "300x20011", "ops": "NONE,PROD",
         "dtype": "affine"},
        # A relaxation step of the benchmark array: eight sweeps per call.
        {"name": "stencil_8192_8", "kind": "stencil", "rows": 8192, "cols": 8192, "steps": 8},
        # The batched benchmark: 10,000 uneven bf16 nests, replayed from a graph.
        {"name": "batch_bf16_10000", "kind": "batch", "mix": "bf16", "nests": 10000, "median": 4096,
         "shapes": 230901910, "graph": True},
        # A burst of requests of the serving benchmark: mixed depths, types and operators.
        {"name": "serve_burst_1000", "kind": "serve", "nests": 1000, "median": 16384, "shapes": 230901911},
    ]


# ---------------------------------------------------------------------------
# drawn cases: the same kinds over their whole ranges


def _log_int(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def _extents(rng, depth, total):
    """Extents of about `total` elements: half of the nests with powers of two inside, half with any sizes."""
    pow2 = rng.random() < 0.5
    inner = []
    rest = total
    for _ in range(depth - 1):
        e = _log_int(rng, 2, max(2, min(1 << 17, rest)))
        if pow2:
            e = 1 << max(1, int(math.log2(e)))
        inner.append(e)
        rest = max(1, rest // e)
    rng.shuffle(inner)
    return [max(1, min(rest, total // math.prod(inner)))] + inner


def draw(rng):
    kind = rng.choice(["i32", "i32", "float", "float", "ordered", "stencil", "batch", "serve", "static"])
    if kind == "i32":
        depth = rng.randint(2, 4)
        ext = _extents(rng, depth, _log_int(rng, 1 << 16, 1 << 26))
        ops = ["NONE"] + [rng.choice(["SUM", "SUM", "MAX", "ARGMIN", "MIN", "ARGMAX"]) for _ in range(depth - 1)]
        for k in range(depth - 2, 0, -1):  # positions are summed: their extremes would be the same for most inputs
            if any(o.startswith("ARG") for o in ops[k + 1:]) and ops[k] != "SUM":
                ops[k] = "MAX" if k == 2 and ext[2] <= ext[3] else "SUM"
        if ops[1] != "SUM" and ext[0] < 16:  # and so would a few extremes or positions
            ext[0] += 16
            k = ext.index(max(ext[1:]), 1)
            ext[k] = max(2, ext[k] // 16)
        low, high = rng.choice([(-(1 << 30), 1 << 30), (0, 1 << 20)])
        return {"kind": "nest", "extents": "x".join(map(str, ext)), "ops": ",".join(ops), "dtype": "i32",
                "low": low, "high": high}
    if kind == "float":
        depth = rng.randint(2, 4)
        dtype = rng.choice(["f32", "bf16"])
        ext = _extents(rng, depth, _log_int(rng, 1 << 16, 1 << 27))
        return {"kind": "nest", "extents": "x".join(map(str, ext)), "ops": "NONE" + ",SUM" * (depth - 1),
                "dtype": dtype, "f32_out": rng.random() < 0.3}
    if kind == "ordered":
        dtype = rng.choice(["affine", "mat2"])
        total = _log_int(rng, 1 << 12, 1 << 24)
        e0 = _log_int(rng, 1, min(total, 4096))
        return {"kind": "ordered", "extents": "%dx%d" % (e0, max(1, total // e0)), "ops": "NONE,PROD", "dtype": dtype}
    if kind == "stencil":
        side = [_log_int(rng, 200, 8192), _log_int(rng, 200, 8192)]
        if rng.random() < 0.5:
            side[1] = -(-side[1] // 64) * 64
        return {"kind": "stencil", "rows": side[0], "cols": side[1], "steps": rng.randint(1, 16)}
    if kind == "batch":
        mix = rng.choice(["bf16", "served"])
        return {"kind": "batch", "mix": mix, "nests": _log_int(rng, 50, 10000 if mix == "bf16" else 1500),
                "median": rng.choice([1024, 4096]) if mix == "bf16" else 16384, "shapes": rng.randrange(1 << 30),
                "graph": rng.random() < 0.5}
    if kind == "serve":
        return {"kind": "serve", "nests": _log_int(rng, 20, 1000), "median": rng.choice([4096, 16384]),
                "shapes": rng.randrange(1 << 30)}
    depth = rng.randint(2, 3)
    ext = _extents(rng, depth, _log_int(rng, 1 << 8, 1 << 20))
    dtype = rng.choice(["i32", "f32", "bf16"])
    c = {"kind": "static", "extents": "x".join(map(str, ext)), "ops": "NONE" + ",SUM" * (depth - 1), "dtype": dtype}
    if dtype == "i32":
        c.update(low=-1000, high=1000)
    else:
        c.update(f32_out=rng.random() < 0.3)
    return c


# ---------------------------------------------------------------------------
# shapes


def _ext(case):
    return tuple(int(e) for e in case["extents"].split("x"))


def _int_out(ops):
    """Output type of an int32 nest: that of the outermost operator that changes the type."""
    for o in ops:
        if o == "SUM":
            return torch.int64
        if o.startswith("ARG"):
            return torch.int32
    return torch.int32


def _many(case):
    """The nests of a batch or burst: (extents, ops, dtype name) each."""
    rng = random.Random(case["shapes"])
    out = []
    for _ in range(case["nests"]):
        if case.get("mix") == "bf16":
            # log-normal lengths up to 2^22; e0 outputs of any reduced length, seen as (j, k)
            n = int(min(max(rng.lognormvariate(math.log(case["median"]), 1.864), 64), 1 << 22))
            e0 = 1 << rng.randint(0, min(6, int(math.log2(n / 64))))
            block = -(-n // e0)
            k = math.gcd(block, 64)
            out.append(((e0, block // k, k), ("NONE", "SUM", "SUM"), "bf16"))
            continue
        # requests: log-normal sizes (elements), 2 to 4 levels, inner extents powers of two, half of them
        # int32 with an operator per level
        n = int(min(max(rng.lognormvariate(math.log(case["median"]), 1.883), 64), 1 << 24))
        depth = rng.randint(2, 4)
        inner, rest = [], n
        for lv in range(depth - 1):
            e = 1 << rng.randint(0, max(0, min(10, int(math.log2(rest)) - (depth - 2 - lv))))
            inner.append(e)
            rest = max(1, rest // e)
        ext = (max(1, -(-n // math.prod(inner))),) + tuple(reversed(inner))
        if rng.random() < 0.5:
            out.append((ext, ("NONE",) + tuple(rng.choice(["SUM", "MAX", "ARGMIN"]) for _ in inner), "i32"))
        else:
            out.append((ext, ("NONE",) + ("SUM",) * (depth - 1), "f32"))
    return out


def _many_layout(nests):
    """Where each nest's input and output lie: one packed buffer per input type (16-byte steps) and per output type."""
    in_at, out_at, ins, outs = [], [], {}, {}
    for ext, ops, dt in nests:
        step = 16 // ELEM_BYTES[dt]
        in_at.append((dt, ins.get(dt, 0)))
        ins[dt] = ins.get(dt, 0) + -(-math.prod(ext) // step) * step
        kind = _int_out(ops) if dt == "i32" else torch.float64
        out_at.append((kind, outs.get(kind, 0)))
        outs[kind] = outs.get(kind, 0) + ext[0]
    return in_at, out_at, ins, outs


# ---------------------------------------------------------------------------
# inputs and handles


def _values(dtype, n, seed, low=-1000, high=1000):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if dtype == "i32":
        return torch.randint(low, high + 1, (n,), dtype=torch.int32, device="cuda", generator=g)
    if dtype == "f32":
        return torch.randn(n, device="cuda", generator=g)
    if dtype == "bf16":
        return torch.randn(n, device="cuda", generator=g).to(torch.bfloat16)
    w = 2 if dtype == "affine" else 4
    x = torch.randint(-(1 << 63), (1 << 63) - 1, (n, w), dtype=torch.int64, device="cuda", generator=g)
    # odd scale factors and determinants, so that long products stay invertible
    x[:, 0] |= 1
    if w == 4:
        x[:, 3] |= 1
        x[:, 1] &= -2
    return x


def _out_tensor(case, ext, ops):
    n = math.prod(e for e, o in zip(ext, ops) if o == "NONE")
    dt = _int_out(ops) if case["dtype"] == "i32" else torch.float32 if case.get("f32_out") else torch.float64
    return torch.empty(n, dtype=dt, device="cuda")


def _input(case, seed):
    return _values(case["dtype"], math.prod(_ext(case)), seed, case.get("low", 0), case.get("high", 0))


class State:
    """What a program has in hand before the call: inputs, outputs and the plan or handle."""

    def __init__(self, kind):
        self.kind = kind


def prepare(case, seed):
    s = State(case["kind"])
    if s.kind in ("nest", "static", "ordered"):
        s.extents, s.ops = _ext(case), tuple(case["ops"].split(","))
        s.flags = hp.FLAG_OUT_F32 if case.get("f32_out") else 0
        s.x = _input(case, seed)
        if s.kind == "static":
            s.out = _out_tensor(case, s.extents, s.ops)
        else:
            s.plan = hp.Plan(s.extents, s.ops, DTYPES[case["dtype"]], flags=s.flags)
            s.out = s.plan.empty_out("cuda")
    elif s.kind == "stencil":
        s.x = _values("f32", case["rows"] * case["cols"], seed).view(case["rows"], case["cols"])
        s.plan = hp.Stencil(case["rows"], case["cols"], case["steps"], 0.6, 0.1)
        weakref.finalize(s, s.plan.close)
        s.out = torch.empty_like(s.x)
    else:
        nests = _many(case)
        in_at, out_at, ins, outs = _many_layout(nests)
        s.x = {dt: _values(dt, n, seed + i) for i, (dt, n) in enumerate(sorted(ins.items()))}
        s.out = {str(k).split(".")[1]: torch.empty(n, dtype=k, device="cuda") for k, n in outs.items()}
        s.nests = [(ext, ops, DTYPES[dt]) for ext, ops, dt in nests]
        hp.tune_cache_load(os.path.join(os.path.dirname(hp.__file__), "tune_gfx950.txt"))
        s.in_ptrs = [s.x[dt].data_ptr() + at * ELEM_BYTES[dt] for dt, at in in_at]
        s.out_ptrs = [s.out[str(k).split(".")[1]].data_ptr() + at * k.itemsize for k, at in out_at]
        if s.kind == "batch":
            s.batch = hp.Batch(s.nests, hp.BATCH_GRAPH if case["graph"] else 0)
            s.batch.set_io_ptrs(s.in_ptrs, s.out_ptrs)
        else:
            s.server = hp.Server(slot_bytes=64 << 20, streams=4, max_batch=512)
            weakref.finalize(s, s.server.close)
            s.due = [0.0] * len(nests)  # a burst: every request has already arrived
            torch.cuda.synchronize()  # the server's streams do not wait for this one
    return s


def run(s):
    if s.kind in ("nest", "ordered"):
        return s.plan.run(s.x, s.out)
    if s.kind == "static":
        return hp.reduce_static(s.x, s.out, s.extents, s.ops, flags=s.flags)
    if s.kind == "stencil":
        return s.plan.run(s.x, s.out)
    if s.kind == "batch":
        s.batch.run()
        return s.out
    tickets = s.server.replay(s.nests, s.in_ptrs, s.out_ptrs, s.due)
    for t in tickets:
        s.server.wait(t)
        s.server.forget(t)
    return s.out


# ---------------------------------------------------------------------------
# the least work, and the results in 64 bits


def work(case):
    if case["kind"] == "stencil":
        n = case["rows"] * case["cols"]
        return {"bytes": 8.0 * n, "flops": 6.0 * n * case["steps"]}
    if case["kind"] in ("batch", "serve"):
        nests = _many(case)
        b = sum(math.prod(e) * ELEM_BYTES[dt] + e[0] * (_int_out(o) if dt == "i32" else torch.float64).itemsize
                for e, o, dt in nests)
        return {"bytes": float(b), "flops": float(sum(math.prod(e) for e, _, _ in nests))}
    ext, ops = _ext(case), case["ops"].split(",")
    n_out = math.prod(e for e, o in zip(ext, ops) if o == "NONE")
    n = math.prod(ext)
    if case["kind"] == "ordered":
        # multiplies and adds of one product: affine 2 and 1, matrices 8 and 4
        return {"bytes": float(ELEM_BYTES[case["dtype"]] * (n + n_out)),
                "flops": (3.0 if case["dtype"] == "affine" else 12.0) * n}
    out = _int_out(ops).itemsize if case["dtype"] == "i32" else 4 if case["f32_out"] else 8
    return {"bytes": float(ELEM_BYTES[case["dtype"]] * n + out * n_out), "flops": float(n)}


def _exact_int(x, ext, ops):
    v = x.cpu().numpy().reshape(ext)
    for o in reversed(ops):
        if o == "SUM":
            v = v.sum(-1, dtype=np.int64)
        elif o == "MIN":
            v = v.min(-1)
        elif o == "MAX":
            v = v.max(-1)
        elif o == "ARGMIN":  # numpy keeps the first occurrence
            v = v.argmin(-1)
        elif o == "ARGMAX":
            v = v.argmax(-1)
    return torch.from_numpy(np.ascontiguousarray(v).reshape(-1)).to(_int_out(ops))


def _exact_float(x, n_out):
    return x.view(n_out, -1).sum(1, dtype=torch.float64)


def _exact_ordered(x, ext, dtype):
    """Adjacent pairs multiplied until one element per output is left (int64 wraps modulo 2^64)."""
    v = x.view(ext[0], -1, x.shape[-1])
    while v.shape[1] > 1:
        even = v.shape[1] // 2 * 2
        a, b = v[:, 0:even:2], v[:, 1:even:2]
        if dtype == "affine":
            p = torch.stack([a[..., 0] * b[..., 0], b[..., 0] * a[..., 1] + b[..., 1]], -1)
        else:
            p = torch.stack([a[..., 0] * b[..., 0] + a[..., 1] * b[..., 2], a[..., 0] * b[..., 1] + a[..., 1] * b[..., 3],
                             a[..., 2] * b[..., 0] + a[..., 3] * b[..., 2], a[..., 2] * b[..., 1] + a[..., 3] * b[..., 3]], -1)
        v = torch.cat([p, v[:, even:]], 1)
    return v[:, 0].contiguous()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("nest", "static"):
        ext, ops = _ext(case), case["ops"].split(",")
        x = _input(case, seed)
        return _exact_int(x, ext, ops) if case["dtype"] == "i32" else _exact_float(x, ext[0])
    if kind == "ordered":
        return _exact_ordered(_input(case, seed), _ext(case), case["dtype"])
    if kind == "stencil":
        a = _values("f32", case["rows"] * case["cols"], seed).view(case["rows"], case["cols"]).double()
        c0, c1 = (float(np.float32(c)) for c in (0.6, 0.1))
        for _ in range(case["steps"]):
            b = a.clone()
            b[1:-1, 1:-1] = c0 * a[1:-1, 1:-1] + c1 * (a[:-2, 1:-1] + a[2:, 1:-1] + a[1:-1, :-2] + a[1:-1, 2:])
            a = b
        return a
    nests = _many(case)
    in_at, out_at, ins, outs = _many_layout(nests)
    x = {dt: _values(dt, n, seed + i) for i, (dt, n) in enumerate(sorted(ins.items()))}
    x_int = x["i32"].cpu() if "i32" in x else None
    got = {k: torch.empty(n, dtype=k) for k, n in outs.items()}
    flt = []
    for (ext, ops, dt), (_, at), (kind, o) in zip(nests, in_at, out_at):
        if dt == "i32":
            got[kind][o:o + ext[0]] = _exact_int(x_int[at:at + math.prod(ext)], ext, ops)
        else:
            flt.append(_exact_float(x[dt][at:at + math.prod(ext)], ext[0]))
    if flt:
        got[torch.float64] = torch.cat(flt)  # float outputs lie in the order of their nests
    return {str(k).split(".")[1]: v for k, v in got.items()}
