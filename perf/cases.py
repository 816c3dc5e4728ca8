"""Performance cases of the framework: the calls a program makes, over their real ranges.

Every case is a dict of plain values.  ``prepare`` makes what a program holds before the
call (seeded inputs on the GPU, the segment list of a batch, the parameters of a network),
``run`` makes one pass through the public entry points, ``work`` says what a pass cannot do
without, ``exact`` computes the floating results in 64 bits with plain torch.  Sizes come from
the benchmark's workloads, the tests and the tuner's instance range (10^2 .. 2^28 elements).
"""
from __future__ import annotations

import math

import torch

import paper_2106_03219_amd as om

DTYPES = {"i32": torch.int32, "i64": torch.int64, "f32": torch.float32, "f64": torch.float64,
          "bf16": torch.bfloat16}
BYTES = {"i32": 4, "i64": 8, "f32": 4, "f64": 8, "bf16": 2}
A = 0.7   # the AXPY body's factor


# ---------------------------------------------------------------- cases

def listed():
    return [
        # the smallest reductions (the low end of the tuner's range): the launch and the team tree
        dict(name="reduce_tiny", kind="reduce", n=1000, dtype="f32", op="sum", offset=0),
        # the headline: one reduction over a large array, bound by memory
        dict(name="reduce_large", kind="reduce", n=1 << 28, dtype="f32", op="sum", offset=0),
        # statistics of an odd-sized 16-bit array in one region: sum, max and min together
        dict(name="stats_ragged", kind="stats", which="multi", n=10_000_019, dtype="bf16",
             offset=1),
        # the worksharing body under the static schedule, at the benchmark's size
        dict(name="axpy_static", kind="axpy", schedule="static", n=1 << 26, chunk=64, offset=0),
        # the same body under a guided schedule, an odd trip count
        dict(name="axpy_guided", kind="axpy", schedule="guided", n=7_000_003, chunk=16, offset=0),
        # the batched workload: 4096 packed segments of mixed types, operators and lengths
        dict(name="batched_mixed", kind="batched", count=4096, low=2.0, high=7.0),
        # column sums of a tall matrix whose rows are not whole 16-byte vectors
        dict(name="array_ragged", kind="array", rows=65_536, m=1001, dtype="f32", op="sum"),
        # an ordinary histogram: a million keys, a thousand bins
        dict(name="hist_ordinary", kind="hist", n=1_000_003, bins=1000),
        # the benchmark's wide histogram: bins far past one team's shared memory
        dict(name="hist_wide", kind="hist", n=1 << 28, bins=1 << 20),
        # device atomics, one word per operation, at the benchmark's size
        dict(name="atomics", kind="atomics", op="add", n=1 << 24, targets=1 << 24),
        # a region with sequential code between its loops: 100 steps of the power iteration
        dict(name="power", kind="power", n=1 << 20, iters=100),
        # one training step of the launch picker's network at the trainer's batch size
        dict(name="picker_step", kind="mlp", batch=256, hidden=64, classes=64),
    ]


def _log(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi], most of them odd."""
    v = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    return min(max(v | 1 if rng.random() < 0.75 else v, lo), hi)


def draw(rng):
    kind = rng.choice(["reduce", "reduce", "stats", "axpy", "axpy", "batched", "array", "hist",
                       "hist", "atomics", "power", "mlp"])
    if kind == "reduce":
        return dict(kind=kind, n=_log(rng, 100, 1 << 28), dtype=rng.choice(sorted(DTYPES)),
                    op=rng.choice(["sum", "sum", "max", "min"]), offset=rng.randrange(4))
    if kind == "stats":
        return dict(kind=kind, which=rng.choice(["multi", "maxloc", "minloc"]),
                    n=_log(rng, 1000, 1 << 27), dtype=rng.choice(sorted(DTYPES)),
                    offset=rng.randrange(4))
    if kind == "axpy":
        return dict(kind=kind, schedule=rng.choice(["static", "static", "dynamic", "guided", "nowait"]),
                    n=_log(rng, 1000, 1 << 26), chunk=rng.choice([0, 1, 7, 16, 64, 100, 1024]),
                    offset=rng.choice([0, 0, 1, 3]))
    if kind == "batched":
        return dict(kind=kind, count=_log(rng, 16, 4096), low=2.0,
                    high=round(rng.uniform(3.5, 6.5), 3))
    if kind == "array":
        m = _log(rng, 2, 20_000)
        return dict(kind=kind, rows=max(1, _log(rng, 10_000, 1 << 26) // m), m=m,
                    dtype=rng.choice(sorted(DTYPES)), op=rng.choice(["sum", "sum", "max", "min"]))
    if kind == "hist":
        return dict(kind=kind, n=_log(rng, 1000, 1 << 28), bins=_log(rng, 10, 1 << 22))
    if kind == "atomics":
        n = _log(rng, 1000, 1 << 24)
        # a program's own word for every operation, or a few words that many operations meet on
        return dict(kind=kind, op=rng.choice(["add", "inc", "max", "exchange", "cas"]), n=n,
                    targets=n) if rng.random() < 0.75 else \
            dict(kind=kind, op=rng.choice(["add", "max"]), n=n, targets=rng.choice([256, 4096]))
    if kind == "power":
        return dict(kind=kind, n=_log(rng, 1 << 10, 1 << 23), iters=rng.randrange(1, 101))
    return dict(kind="mlp", batch=_log(rng, 1, 4096), hidden=rng.choice([32, 64, 96]),
                classes=rng.choice([8, 24, 64]))


# ---------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _values(n, dtype, g):
    """The distributions of the workloads: N(0, 1), small 32-bit and 40-bit 64-bit integers."""
    if dtype == "i32":
        return torch.randint(-1000, 1001, (n,), device="cuda", dtype=torch.int32, generator=g)
    if dtype == "i64":
        return torch.randint(-(1 << 40), (1 << 40) + 1, (n,), device="cuda", dtype=torch.int64,
                             generator=g)
    if dtype == "bf16":
        return torch.randn(n, device="cuda", generator=g).to(torch.bfloat16)
    return torch.randn(n, device="cuda", dtype=DTYPES[dtype], generator=g)


def _zeros(n, dtype):
    return torch.zeros(n, device="cuda", dtype=DTYPES[dtype])


def _sum_type(dtype):
    return "f32" if dtype == "bf16" else dtype   # bf16 sums return the fp32 accumulator


def _segments(case):
    """(length, type, operator) of a batch's segments: the case's own, whatever the data."""
    count = case["count"]
    r = torch.Generator().manual_seed(count)
    lens = torch.pow(10.0, case["low"] + (case["high"] - case["low"]) *
                     torch.rand(count, generator=r, dtype=torch.float64)).floor().long().tolist()
    kinds = torch.randint(0, 3, (count,), generator=r).tolist()
    ops = torch.randint(0, 3, (count,), generator=r).tolist()
    return [(n, ("i64", "f32", "bf16")[k], ("sum", "max", "min")[o])
            for n, k, o in zip(lens, kinds, ops)]


def _batch(case, seed):
    """Segments packed one behind another in an array per element type."""
    g = _gen(seed)
    spec = _segments(case)
    total = {t: 0 for t in ("i64", "f32", "bf16")}
    outs = {"i64": 0, "f32": 0, "bf16": 0}
    place = []
    for n, t, op in spec:
        ot = _sum_type(t) if op == "sum" else t
        place.append((total[t], ot, outs[ot]))
        total[t] += n
        outs[ot] += 1
    data = {t: _values(max(n, 1), t, g) for t, n in total.items()}
    x = {t: _zeros(max(n, 1), t) for t, n in outs.items()}
    items = [(data[t][at:at + n], op, x[ot][j:j + 1]) for (n, t, op), (at, ot, j) in zip(spec, place)]
    return data, x, items


def _dims(case):
    return (16, case["hidden"], case["hidden"], case["classes"])


def _inputs(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "reduce":
        base = _values(case["n"] + case["offset"], case["dtype"], g)
        return dict(inp=base[case["offset"]:],
                    x=_zeros(1, _sum_type(case["dtype"]) if case["op"] == "sum" else case["dtype"]))
    if kind == "stats":
        base = _values(case["n"] + case["offset"], case["dtype"], g)
        inp = base[case["offset"]:]
        if case["which"] == "multi":
            return dict(inp=inp, sum=_zeros(1, _sum_type(case["dtype"])),
                        max=_zeros(1, case["dtype"]), min=_zeros(1, case["dtype"]))
        return dict(inp=inp, val=_zeros(1, case["dtype"]),
                    idx=torch.full((1,), -1, device="cuda", dtype=torch.int64))
    if kind == "axpy":
        o = case["offset"]
        return dict(x=_values(case["n"] + o, "f32", g)[o:], y=_values(case["n"] + o, "f32", g)[o:],
                    s=_zeros(1, "f32"))
    if kind == "array":
        return dict(inp=_values(case["rows"] * case["m"], case["dtype"], g),
                    x=_zeros(case["m"], _sum_type(case["dtype"]) if case["op"] == "sum"
                             else case["dtype"]))
    if kind == "hist":
        return dict(keys=torch.randint(0, case["bins"], (case["n"],), device="cuda",
                                       dtype=torch.int32, generator=g),
                    hist=torch.zeros(case["bins"], device="cuda", dtype=torch.int32))
    if kind == "atomics":
        n, t = case["n"], case["targets"]
        index = torch.randperm(n, device="cuda", generator=g).to(torch.int32) if t == n else \
            torch.randint(0, t, (n,), device="cuda", dtype=torch.int32, generator=g)
        target = torch.randint(0, 1000, (t,), device="cuda", dtype=torch.int32, generator=g)
        e = torch.randint(0, 1000, (n,), device="cuda", dtype=torch.int32, generator=g)
        d = torch.randint(0, 1000, (n,), device="cuda", dtype=torch.int32, generator=g)
        return dict(target=target, index=index, e=e, d=d,
                    old=torch.zeros(n, device="cuda", dtype=torch.int32))
    if kind == "power":
        u = torch.rand(case["n"], device="cuda", generator=g) * 0.25 + 0.75
        sign = torch.randint(0, 2, (case["n"],), device="cuda", generator=g) * 2 - 1
        return dict(diag=u * sign, v=_values(case["n"], "f32", g), lam=_zeros(1, "f32"))
    F, H1, H2, K = _dims(case)
    parts = []
    for o, i, f in ((H1, F, 1.0), (H2, H1, 1.0), (K, H2, 0.1)):
        w = (torch.rand(o * i, device="cuda", generator=g) * 2 - 1) * math.sqrt(6.0 / i) * f
        parts += [w, torch.zeros(o, device="cuda")]
    params = torch.cat(parts)
    return dict(params=params, m=torch.zeros_like(params), v=torch.zeros_like(params),
                grads=torch.zeros_like(params),
                X=torch.randn(case["batch"], F, device="cuda", generator=g),
                y=torch.randint(0, K, (case["batch"],), device="cuda", dtype=torch.int32,
                                generator=g),
                loss=_zeros(1, "f32"), step=torch.zeros(1, device="cuda", dtype=torch.int32))


def prepare(case, seed):
    if case["kind"] == "batched":
        data, x, items = _batch(case, seed)
        return dict(case=case, data=data, x=x, segments=om.make_segments(items))
    return dict(_inputs(case, seed), case=case)


# ---------------------------------------------------------------- one pass

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "reduce":
        om.reduce(s["inp"], case["op"], s["x"])
        return s["x"]
    if kind == "stats":
        if case["which"] == "multi":
            om.reduce_multi(s["inp"], [("sum", s["sum"]), ("max", s["max"]), ("min", s["min"])])
            return dict(sum=s["sum"], max=s["max"], min=s["min"])
        om.reduce_loc(s["inp"], case["which"][:3], s["val"], s["idx"])
        return dict(val=s["val"], idx=s["idx"])
    if kind == "axpy":
        if case["schedule"] == "static":
            om.axpy_sum(A, s["x"], s["y"], s["s"], chunk=case["chunk"])
        elif case["schedule"] == "nowait":
            om.region_axpy_sum(A, s["x"], s["y"], s["s"], chunk=case["chunk"], nowait=True)
        else:
            om.axpy_sum_queue(case["schedule"], A, s["x"], s["y"], s["s"], chunk=case["chunk"])
        return dict(y=s["y"], sum=s["s"])
    if kind == "batched":
        om.reduce_batched(s["segments"])
        return s["x"]
    if kind == "array":
        om.reduce_array(s["inp"], case["rows"], case["m"], case["op"], s["x"])
        return s["x"]
    if kind == "hist":
        om.histogram(s["keys"], case["bins"], s["hist"])
        return s["hist"]
    if kind == "atomics":
        om.atomic_apply(case["op"], s["target"], s["index"], s["e"], s["old"],
                        s["d"] if case["op"] == "cas" else None)
        # which operation reads which value is not defined where several meet on a word
        return dict(target=s["target"], old=s["old"]) if case["targets"] == case["n"] else \
            dict(target=s["target"])
    if kind == "power":
        om.generic_power(s["diag"], s["v"], case["iters"], s["lam"])
        return dict(v=s["v"], lam=s["lam"])
    dims = _dims(case)
    om.mlp_loss_grad(dims, s["params"], s["X"], s["y"], s["loss"], s["grads"])
    om.mlp_adam_counted(s["params"], s["m"], s["v"], s["grads"], s["step"])
    return dict(loss=s["loss"], grads=s["grads"], params=s["params"], m=s["m"], v=s["v"])


# ---------------------------------------------------------------- work and exact values

def work(case):
    kind = case["kind"]
    if kind in ("reduce", "stats"):
        return dict(bytes=case["n"] * BYTES[case["dtype"]], flops=case["n"])
    if kind == "axpy":
        return dict(bytes=12 * case["n"], flops=3 * case["n"])
    if kind == "batched":
        mean = (10 ** case["high"] - 10 ** case["low"]) / \
            ((case["high"] - case["low"]) * math.log(10.0))   # of the log-uniform lengths
        return dict(bytes=case["count"] * mean * (8 + 4 + 2) / 3, flops=case["count"] * mean)
    if kind == "array":
        n = case["rows"] * case["m"]
        return dict(bytes=n * BYTES[case["dtype"]] + 2 * case["m"] * BYTES[case["dtype"]], flops=n)
    if kind == "hist":
        return dict(bytes=4 * case["n"] + 8 * case["bins"], flops=case["n"])
    if kind == "atomics":
        operands = 3 if case["op"] == "cas" else 2
        return dict(bytes=case["n"] * 4 * (operands + 1) + 8 * case["targets"], flops=case["n"])
    if kind == "power":
        return dict(bytes=12 * case["n"], flops=4 * case["n"] * case["iters"])
    F, H1, H2, K = _dims(case)
    p = H1 * F + H1 + H2 * H1 + H2 + K * H2 + K
    macs = 3 * (F * H1 + H1 * H2 + H2 * K) - F * H1   # forward, weight and input gradients
    return dict(bytes=4 * (case["batch"] * (F + 1) + 7 * p), flops=2 * macs * case["batch"])


def _f32(a):
    return torch.tensor(a, dtype=torch.float32).double().item()


def _fold(t, op):
    """The reduction of t with an incoming 0, in 64 bits."""
    t = t.double()
    return t.sum() if op == "sum" else t.max().clamp(min=0) if op == "max" else t.min().clamp(max=0)


def _exact_step(case, s):
    F, H1, H2, K = _dims(case)
    sizes = [(H1, F), (H1,), (H2, H1), (H2,), (K, H2), (K,)]
    p, at = [], 0
    for sh in sizes:
        n = math.prod(sh)
        p.append(s["params"][at:at + n].double().reshape(sh))
        at += n
    W1, b1, W2, b2, W3, b3 = p
    X, B = s["X"].double(), case["batch"]
    a1 = torch.relu(X @ W1.t() + b1)
    a2 = torch.relu(a1 @ W2.t() + b2)
    z = a2 @ W3.t() + b3
    lp = z - torch.logsumexp(z, 1, keepdim=True)
    y = s["y"].long()
    loss = -lp.gather(1, y[:, None]).mean()
    dz = lp.exp()
    dz.scatter_add_(1, y[:, None], torch.full((B, 1), -1.0, dtype=torch.float64, device="cuda"))
    dz /= B
    d2 = (dz @ W3) * (a2 > 0)
    d1 = (d2 @ W2) * (a1 > 0)
    g = torch.cat([t.reshape(-1) for t in (d1.t() @ X, d1.sum(0), d2.t() @ a1, d2.sum(0),
                                           dz.t() @ a2, dz.sum(0))])
    lr, be1, be2, eps = _f32(1e-3), _f32(0.9), _f32(0.999), _f32(1e-8)
    m, v = (1 - be1) * g, (1 - be2) * g * g
    w = s["params"].double() - lr * (m / (1 - be1)) / ((v / (1 - be2)).sqrt() + eps)
    return dict(loss=loss.reshape(1), grads=g, params=w, m=m, v=v)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("hist", "atomics"):
        return None   # whole numbers
    if kind == "batched":
        _, x, items = _batch(case, seed)
        out = {t: torch.zeros(v.numel(), dtype=torch.float64, device="cuda")
               for t, v in x.items() if t != "i64"}
        for inp, op, xv in items:
            t = {torch.float32: "f32", torch.bfloat16: "bf16"}.get(xv.dtype)
            if t:
                out[t][xv.storage_offset()] = _fold(inp, op)
        return dict(out, i64=None)
    s = _inputs(case, seed)
    if kind == "reduce":
        return None if case["dtype"][0] == "i" else _fold(s["inp"], case["op"]).reshape(1)
    if kind == "stats":
        if case["dtype"][0] == "i":
            return None
        if case["which"] == "multi":
            return {op: _fold(s["inp"], op).reshape(1) for op in ("sum", "max", "min")}
        return dict(val=_fold(s["inp"], case["which"][:3]).reshape(1), idx=None)
    if kind == "axpy":
        y = _f32(A) * s["x"].double() + s["y"].double()
        return dict(y=y, sum=y.float().double().sum().reshape(1))
    if kind == "array":
        if case["dtype"][0] == "i":
            return None
        a = s["inp"].reshape(case["rows"], case["m"]).double()
        return a.sum(0) if case["op"] == "sum" else a.amax(0).clamp(min=0) \
            if case["op"] == "max" else a.amin(0).clamp(max=0)
    if kind == "power":
        d, v = s["diag"].double(), s["v"].double()
        for _ in range(case["iters"]):
            v = d * v
            lam = v.square().sum().sqrt()
            v = v / lam
        return dict(v=v, lam=lam.reshape(1))
    return _exact_step(case, s)
