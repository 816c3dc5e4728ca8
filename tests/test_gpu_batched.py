"""GPU parity of the batched persistent launch (graph captured once, then
replayed) against the oracle per segment, plus the plain one-launch-per-
segment form; both ticket and round-robin tile dealing; replays without
any counter reset.
"""
import time
from concurrent.futures import ThreadPoolExecutor

import pytest
import torch

import synth
from gpu_util import check_value, identity, oracle_value, to_device, to_host, x_tensor, x_value

pytestmark = pytest.mark.gpu

OPN = {synth.SUM: "sum", synth.MAX: "max", synth.MIN: "min"}


def _make(count, seed, lo_exp, hi_exp, dtypes=(synth.I64, synth.F32, synth.BF16)):
    lens, dts, ops = synth.batched_spec(count, seed, lo_exp, hi_exp, dtypes)
    ins, xs, meta = [], [], []
    for i in range(count):
        n, dt, op = int(lens[i]), int(dts[i]), OPN[int(ops[i])]
        host = synth.host(dt, n, 10_000 + i)
        ins.append(to_device(host, dt))
        x0 = identity(dt, op) if i % 2 == 0 else (3 if dt in (synth.I32, synth.I64) else 0.5)
        xs.append(x_tensor(dt, op, x0))
        meta.append((host, dt, op, x0))
    return ins, xs, meta


def _check_all(xs, meta):
    torch.cuda.synchronize()
    for x, (host, dt, op, x0) in zip(xs, meta):
        ref, sabs = oracle_value(host, dt, op, x0)
        check_value(x_value(x), ref, sabs, dt, op)


def _reset(xs, meta):
    for x, (_, dt, op, x0) in zip(xs, meta):
        x.copy_(x_tensor(dt, op, x0))


@pytest.mark.parametrize("config", [None, {"tile_kib": 16}, {"tile_kib": 64, "threads": 512, "unroll": 8},
                                    {"tile_kib": 32, "flags": 2, "teams": 37},
                                    {"tile_kib": 8, "vec": 8, "unroll": 2, "threads": 128}])
def test_batched_mixed_segments_replayed(gpu_lib, config):
    om = gpu_lib
    ins, xs, meta = _make(300, 61, 0.0, 5.3, (synth.I32, synth.I64, synth.F32, synth.F64, synth.BF16))
    segs = om.make_segments([(i, m[2], x) for i, x, m in zip(ins, xs, meta)])
    for rep in range(3):
        _reset(xs, meta)
        om.reduce_batched(segs, config=config)
        _check_all(xs, meta)


def test_reduce_each_matches_oracle(gpu_lib):
    om = gpu_lib
    ins, xs, meta = _make(200, 62, 2.0, 5.0)
    segs = om.make_segments([(i, m[2], x) for i, x, m in zip(ins, xs, meta)])
    om.reduce_each(segs)
    _check_all(xs, meta)


def test_batched_empty_and_single(gpu_lib):
    om = gpu_lib
    a = torch.arange(10, dtype=torch.int64, device="cuda")
    x = torch.zeros(1, dtype=torch.int64, device="cuda")
    y = torch.full((1,), 5, dtype=torch.int64, device="cuda")
    om.reduce_batched([(a, "sum", x), (a[:0], "sum", y, 0)])
    torch.cuda.synchronize()
    assert x.item() == 45 and y.item() == 5


def test_batched_many_replays_no_reset(gpu_lib):
    om = gpu_lib
    ins, xs, meta = _make(64, 63, 3.0, 6.0, (synth.I64,))
    segs = om.make_segments([(i, "sum", x) for i, x in zip(ins, xs)])
    for x in xs:
        x.zero_()
    reps = 200
    for _ in range(reps):
        om.reduce_batched(segs, config={"tile_kib": 16})
    torch.cuda.synchronize()
    for x, (host, _, _, _) in zip(xs, meta):
        s = int(host.astype(object).sum())
        want = (reps * s + 2**63) % 2**64 - 2**63
        assert x.item() == want
    assert om.workspace_status() == 0


def check_every_segment(ins, xs, info, x0s=None, what=""):
    """Every segment's result against the oracle, from host copies, several segments at
    a time (the oracle's C loops run outside the interpreter lock).  Returns the
    (rel, kappa) records of the floating sums."""
    torch.cuda.synchronize()

    def one(i):
        dt, op = info[i]
        x0 = identity(dt, op) if x0s is None else x0s[i]
        ref, sabs = oracle_value(to_host(ins[i]), dt, op, x0)
        return check_value(x_value(xs[i]), ref, sabs, dt, op, f"{what} segment {i}",
                           n=int(ins[i].numel()))

    with ThreadPoolExecutor(8) as ex:
        return [r for r in ex.map(one, range(len(ins))) if r is not None]


@pytest.mark.slow
def test_batched_full_4096_every_segment(gpu_lib):
    """4096 segments, lengths log-uniform in [1e2, 1e7] (about 16 GB), int64 / fp32 /
    bf16, sum / max / min: every segment of the persistent graph-replayed launch, and
    of the plain one-launch-per-segment form, against the oracle."""
    om = gpu_lib
    lens, dts, ops = synth.batched_spec(4096, synth.SEED_BATCH)
    ins, xs, info = [], [], []
    for i in range(4096):
        dt, op = int(dts[i]), OPN[int(ops[i])]
        ins.append(synth.device(dt, int(lens[i]), 20_000 + i))
        xs.append(x_tensor(dt, op, identity(dt, op)))
        info.append((dt, op))
    segs = om.make_segments([(t, op, x) for t, x, (dt, op) in zip(ins, xs, info)])
    om.reduce_batched(segs)
    om.reduce_batched(segs)           # a replay of the cached graph, from the identity again
    for x, (dt, op) in zip(xs, info):
        x.copy_(x_tensor(dt, op, identity(dt, op)))
    om.reduce_batched(segs)
    errs = check_every_segment(ins, xs, info, what="batched")
    assert len(errs) == sum(1 for dt, op in info if op == "sum" and dt != synth.I64)
    for x, (dt, op) in zip(xs, info):
        x.copy_(x_tensor(dt, op, identity(dt, op)))
    om.reduce_each(segs)
    check_every_segment(ins, xs, info, what="plain")
    assert om.workspace_status() == 0


@pytest.mark.parametrize("config", [None, {"teams": 2}, {"threads": 64}, {"threads": 192, "teams": 3},
                                    {"flags": 2, "teams": 5}, {"vec": 8, "unroll": 1}])
def test_short_segments(gpu_lib, config):
    """Segments around the sizes up to which one wave takes one (8 KB; 32 KB with at least
    eight segments a workgroup, as with two teams), off 16-byte alignment, in bundles with a
    remainder, between longer ones and an empty one: called twice, then captured by the caller
    and replayed, with the library's own calls in between."""
    om = gpu_lib
    ins, xs, meta = [], [], []
    for dt, eb in ((synth.I32, 4), (synth.I64, 8), (synth.F32, 4), (synth.F64, 8), (synth.BF16, 2)):
        for j, b in enumerate((eb, 5 * eb, 64 * eb, 8192 - eb, 8192, 8192 + eb, 32768, 32768 + eb, 150000 * eb)):
            op = ("sum", "max", "min")[j % 3]
            host = synth.host(dt, b // eb + j % 4, 30_000 + j)
            ins.append(to_device(host, dt)[j % 4:])
            x0 = 3 if dt in (synth.I32, synth.I64) else 0.5
            xs.append(x_tensor(dt, op, x0))
            meta.append((host[j % 4:], dt, op, x0))
    empty = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    items = [(i, m[2], x) for i, x, m in zip(ins, xs, meta)]
    segs = om.make_segments(items[:7] + [(ins[0], "sum", empty, 0)] + items[7:])
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        for _ in range(2):
            _reset(xs, meta)
            om.reduce_batched(segs, config=config)
            _check_all(xs, meta)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            om.reduce_batched(segs, config=config)
        for _ in range(3):
            _reset(xs, meta)
            g.replay()
            _check_all(xs, meta)
            _reset(xs, meta)
            om.reduce_batched(segs, config=config)
            _check_all(xs, meta)
        assert empty.item() == 5 and om.workspace_status() == 0


def test_large_plan_replay_and_capture(gpu_lib):
    """A plan of more tiles than workgroups (tickets, several rounds): repeat calls, and the call
    inside a graph of the caller's, replayed with the library's own calls in between."""
    om = gpu_lib
    big = torch.ones((512 << 20) // 8 + 5, dtype=torch.int64, device="cuda")
    small = torch.arange(1001, dtype=torch.int64, device="cuda")
    x, y = (torch.zeros(1, dtype=torch.int64, device="cuda") for _ in range(2))
    segs = om.make_segments([(small, "sum", y), (big, "sum", x)])
    calls = 0
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        for _ in range(3):
            om.reduce_batched(segs)
            calls += 1
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            om.reduce_batched(segs)
        for _ in range(3):
            g.replay()
            om.reduce_batched(segs)
            calls += 2
            s.synchronize()
            assert x.item() == calls * big.numel() and y.item() == calls * 500500
        assert om.workspace_status() == 0


@pytest.mark.parametrize("streams", [1, 2])
def test_alternating_lists(gpu_lib, streams):
    """A new list every call, on one stream or two in turn, with no synchronisation between:
    each plan's tables are up before its launch and not overwritten under it."""
    om = gpu_lib
    lists = []
    for k in range(3):
        ins = [torch.full((n,), k + 1, dtype=torch.int64, device="cuda")
               for n in (5, 700 + k, 3000, 70001 + 13 * k, 9) for _ in range(20 + 7 * k)]
        for _ in range(streams):
            xs = [torch.zeros(1, dtype=torch.int64, device="cuda") for _ in ins]
            lists.append((ins, xs, om.make_segments([(i, "sum", x) for i, x in zip(ins, xs)]), k + 1))
    torch.cuda.synchronize()
    sides = [torch.cuda.Stream() for _ in range(streams)]
    reps = 30
    for _ in range(reps):
        for j, (_, _, segs, _) in enumerate(lists):
            with torch.cuda.stream(sides[j % streams]):
                om.reduce_batched(segs)
    torch.cuda.synchronize()
    for ins, xs, _, v in lists:
        assert [x.item() for x in xs] == [reps * v * i.numel() for i in ins]


def _sleep_rate():
    """Cycles of torch.cuda._sleep a second."""
    start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    torch.cuda._sleep(1000)
    start.record()
    torch.cuda._sleep(10_000_000)
    end.record()
    end.synchronize()
    return 10_000_000 / (start.elapsed_time(end) * 1e-3)


def _filled_list(om, value, seed):
    ins = [torch.full((n + seed,), value, dtype=torch.int64, device="cuda")
           for n in (5, 700, 3000, 70001, 300007) for _ in range(12)]
    xs = [torch.zeros(1, dtype=torch.int64, device="cuda") for _ in ins]
    return ins, xs, om.make_segments([(i, "sum", x) for i, x in zip(ins, xs)])


def test_new_list_behind_queued_work(gpu_lib):
    """New lists on a stream whose earlier work is far from done, and on another stream: neither
    call waits for that work, and the plan is whole when the call returns, so a graph of it,
    captured at once, replays on an idle stream before the building stream gets to it.  (Two
    streams may share one of the device's few hardware queues, whose work waits in line: one
    pair of streams that do not is enough.)"""
    om = gpu_lib
    rate = _sleep_rate()
    om.reduce_batched(_filled_list(om, 1, 0)[2])   # what the library sets up once
    ahead = False
    for attempt in range(8):
        first, second, other = (_filled_list(om, v, 11 * v + attempt) for v in (1, 2, 3))
        busy, idle = torch.cuda.Stream(), torch.cuda.Stream()
        done = torch.cuda.Event()
        torch.cuda.synchronize()
        began = time.perf_counter()
        with torch.cuda.stream(busy):
            torch.cuda._sleep(int(0.4 * rate))
            done.record()
            om.reduce_batched(first[2])
            om.reduce_batched(second[2])
            g = torch.cuda.CUDAGraph()
            g.capture_begin(capture_error_mode="thread_local")
            om.reduce_batched(second[2])
            g.capture_end()
        late = time.perf_counter() - began > 0.2
        if late:   # a plan's launches must not overlap
            idle.wait_stream(busy)
        with torch.cuda.stream(idle):
            om.reduce_batched(other[2])
            for _ in range(3):
                g.replay()
        idle.synchronize()
        ahead = not late and not done.query()
        assert [x.item() for x in other[1]] == [3 * i.numel() for i in other[0]]
        if ahead:
            assert [x.item() for x in second[1]] == [3 * 2 * i.numel() for i in second[0]]
        torch.cuda.synchronize()
        assert [x.item() for x in first[1]] == [i.numel() for i in first[0]]
        assert [x.item() for x in second[1]] == [4 * 2 * i.numel() for i in second[0]]
        if ahead:
            break
    assert ahead
