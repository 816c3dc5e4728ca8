"""Host checks of the array-section reduction (no GPU): argument errors, and
the launch geometry's index arithmetic replayed on the CPU.

The replay follows the kernel's mapping from the plan the library reports:
team (c, r) -> tile c, balanced periods of row team r; lane slot (u, t)
covers flat offsets o = (u*P + t)*E .. +E-1 of a period, address
(o // w)*m + o % w + k from the period start, list item c*W + (o + k) % w;
the last row team adds the rows after the whole periods.  Every element of
the rows x m block must be read exactly once, inside the block, by a slot
whose list item is the element's column.
"""
import ctypes

import numpy as np
import pytest

import paper_2106_03219_amd as om
from paper_2106_03219_amd import _lib

ESIZE = {om.I32: 4, om.I64: 8, om.F32: 4, om.F64: 8, om.BF16: 2}


def acc_bytes(dt, op):
    if dt in (om.F32, om.BF16):
        return 8 if op == "sum" else 4
    if dt == om.F64:
        return 16 if op == "sum" else 8
    return ESIZE[dt]


def lds_entries(R, W, m, tiles, layer, U):
    """Private copies a team gathers in LDS: a period's span, or one layer of
    P*E offsets when all U layers are live and each holds whole tile rows."""
    need = 0
    for wc in (min(W, m), m - (tiles - 1) * W):
        span = R * wc
        fold = U > 1 and span == U * layer and layer % wc == 0
        need = max(need, layer if fold else span)
    return need


def bal(n, p, t):
    q, r = divmod(n, p)
    lo = t * q + min(t, r)
    return lo, lo + q + (1 if t < r else 0)


def replay(rows, m, dt, plan):
    W, R, tiles, rt, ng, vb, P, U = plan
    esize = ESIZE[dt]
    E = vb // esize
    np_ = rows // R
    hits = np.zeros(rows * m, dtype=np.int64)
    for c in range(tiles):
        c0 = c * W
        wc = min(W, m - c0)
        span = R * wc
        o = ((np.arange(U)[:, None] * P + np.arange(P)[None, :]) * E).ravel()
        o = o[o < span]
        k = np.arange(E)
        flat = (o[:, None] + k[None, :]).ravel()            # LDS index of every element
        addr0 = ((o // wc) * m + o % wc)[:, None] + k[None, :]
        addr0 = addr0.ravel()
        item = c0 + flat % wc
        assert flat.max() < span and np.unique(flat).size == flat.size
        for r in range(rt):
            lo, hi = bal(np_, rt, r)
            for p in range(lo, hi):
                a = c0 + p * R * m + addr0
                assert a.min() >= 0 and a.max() < rows * m
                assert np.array_equal(a % m, item)
                np.add.at(hits, a, 1)
            if r == rt - 1:
                tl = (rows - np_ * R) * wc
                ot = np.arange(U * P * E)
                ot = ot[ot < tl]
                a = c0 + np_ * R * m + (ot // wc) * m + ot % wc
                if a.size:
                    assert a.max() < rows * m
                    assert np.array_equal(a % m, c0 + ot % wc)
                np.add.at(hits, a, 1)
    assert np.all(hits == 1)


CASES = [(1, 1), (5, 1), (3, 7), (1000, 1), (1000, 3), (777, 8), (513, 100), (300, 256),
         (300, 257), (97, 1000), (50, 1001), (40, 4096), (9, 5000), (3, 20000), (2000, 33)]


@pytest.mark.parametrize("dt", [om.I32, om.I64, om.F32, om.F64, om.BF16])
@pytest.mark.parametrize("aligned", [1, 0])
def test_geometry_covers_every_element_once(dt, aligned):
    for rows, m in CASES:
        for op in ("sum", "max"):
            plan = om.reduce_array_plan(rows, m, dt, op, aligned16=aligned)
            W, R, tiles, rt, ng, vb, P, U = plan
            E = vb // ESIZE[dt]
            assert vb in (16, ESIZE[dt]) and (vb == 16) <= bool(aligned)
            assert R * min(W, m) <= P * E * U
            assert lds_entries(R, W, m, tiles, P * E, U) * acc_bytes(dt, op) <= 64 * 1024 - 256
            assert tiles == -(-m // W) and W % E == 0 or tiles == 1
            if tiles == 1:
                assert W == m and (vb != 16 or (R * m * ESIZE[dt]) % 16 == 0)
            else:
                assert m % E == 0 and m - (tiles - 1) * W > 0
            assert 1 <= rt <= max(1, rows // R)
            wc = min(W, m)
            per_col = 1 if wc * 2 > P else P // wc
            gs = min(rt, max(2, 16 * per_col // -(-wc // P)))
            assert ng == -(-rt // gs)
            replay(rows, m, dt, plan)


def test_geometry_under_explicit_configs():
    for cfg in [dict(threads=64, unroll=1), dict(threads=512, unroll=1), dict(threads=128, unroll=8),
                dict(threads=512), dict(teams=3), dict(teams=65535), dict(vec=4)]:
        for rows, m in [(1000, 3), (300, 257), (97, 1000), (64, 4096), (5000, 1)]:
            plan = om.reduce_array_plan(rows, m, om.F32, "sum", config=cfg)
            replay(rows, m, om.F32, plan)
    # teams of more than 512 threads are refused; an explicit unroll whose
    # private copies fit LDS only with element loads falls back to them
    with pytest.raises(om.OmprtError):
        om.reduce_array_plan(100, 100, om.F32, "sum", config=dict(threads=1024))
    assert om.reduce_array_plan(100, 100, om.BF16, "sum", config=dict(threads=512, unroll=4))[5] == 2
    # whole rows in every layer: the lane's slots fold in registers, so
    # 512 threads x 4 loads of fp32 sums fit
    assert om.reduce_array_plan(1 << 20, 8, om.F32, "sum", config=dict(threads=512))[7] == 4


def test_tiles_are_balanced():
    W, R, tiles, *_ = om.reduce_array_plan(100, 257, om.F32, "sum", aligned16=False)
    assert tiles == 2 and W == 129
    W, R, tiles, *_ = om.reduce_array_plan(100, 1 << 20, om.F32, "sum")
    assert W == 256 and tiles == 4096


def test_argument_errors_before_device():
    lib = _lib.load()
    x = ctypes.c_float(0)
    A = lib.omprt_reduce_array
    assert A(None, 5, 5, 9, 0, ctypes.byref(x), None, None) == _lib.ERR_UNSUPPORTED
    assert A(None, 5, 5, 0, 9, ctypes.byref(x), None, None) == _lib.ERR_UNSUPPORTED
    assert A(None, 5, 5, 2, 4, ctypes.byref(x), None, None) == _lib.ERR_UNSUPPORTED   # fp32 &
    assert A(None, -1, 5, 0, 0, ctypes.byref(x), None, None) == _lib.ERR_INVALID
    assert A(None, 5, -1, 0, 0, ctypes.byref(x), None, None) == _lib.ERR_INVALID
    assert A(None, 1 << 30, 1 << 30, 0, 0, ctypes.byref(x), None, None) == _lib.ERR_INVALID
    assert A(None, 0, 5, 0, 0, None, None, None) == _lib.OK        # nothing to do
    assert A(None, 5, 0, 0, 0, None, None, None) == _lib.OK
    assert A(None, 5, 5, 0, 0, ctypes.byref(x), None, None) == _lib.ERR_INVALID   # NULL in
    assert A(ctypes.c_void_p(0x1002), 5, 5, 0, 0, ctypes.c_void_p(0x100000), None, None) == _lib.ERR_INVALID
    assert A(ctypes.c_void_p(0x1000), 5, 5, 0, 0, ctypes.c_void_p(0x1010), None, None) == _lib.ERR_INVALID
    assert b"overlaps" in lib.omprt_last_error()
    c = _lib.Config(0, 100, 0, 0, 0, 0)
    assert A(ctypes.c_void_p(0x1000), 5, 5, 0, 0, ctypes.c_void_p(0x100000), ctypes.byref(c), None) == _lib.ERR_INVALID
    c = _lib.Config(0, 0, 8, 0, 0, 0)
    assert A(ctypes.c_void_p(0x1000), 5, 5, 2, 0, ctypes.c_void_p(0x100000), ctypes.byref(c), None) == _lib.ERR_INVALID
    c = _lib.Config(0, 0, 0, 3, 0, 0)
    assert A(ctypes.c_void_p(0x1000), 5, 5, 2, 0, ctypes.c_void_p(0x100000), ctypes.byref(c), None) == _lib.ERR_INVALID
    c = _lib.Config(70000, 0, 0, 0, 0, 0)
    assert A(ctypes.c_void_p(0x1000), 5, 5, 2, 0, ctypes.c_void_p(0x100000), ctypes.byref(c), None) == _lib.ERR_INVALID
    out = (ctypes.c_int64 * 8)()
    assert lib.omprt_reduce_array_plan(0, 5, 0, 0, 1, None, out) == _lib.ERR_INVALID
    assert lib.omprt_reduce_array_plan(5, 5, 0, 0, 1, None, None) == _lib.ERR_INVALID


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("rows,m,dt,op,config", [
    (44894, 88, om.F64, "sum", {"unroll": 8}),
    (131072, 131, om.F64, "sum", {"unroll": 8}),
    (56513, 77, om.F64, "prod", {"unroll": 4}),
    (9202, 495, om.F64, "sum", {"unroll": 8, "threads": 512}),
    (155000, 101, om.F32, "sum", {"unroll": 4}),
    (243819, 226, om.BF16, "max", {"unroll": 2}),
    (20000, 101, om.BF16, "sum", {"vec": 2}),       # 4 MB
    (100000, 101, om.BF16, "sum", {"vec": 2}),      # 20 MB
    (40000, 100, om.F32, "max", {"vec": 4}),        # 15.3 MiB
    (48000, 100, om.F32, "max", {"vec": 4}),        # 18.3 MiB
    (1008246, 65, om.I64, "sum", {"vec": 8}),
])
def test_explicit_unroll_and_element_loads_keep_their_tiles(rows, m, dt, op, config, aligned):
    """A given unroll, and element loads, keep the fewest tiles of up to 256 columns at any size of
    the block, so that the call is taken, and whole rows of any width keep 16-byte loads."""
    plan = om.reduce_array_plan(rows, m, dt, op, aligned16=aligned, config=config)
    assert plan[2] == -(-m // 256)
    u = config.get("unroll")
    vectors = aligned and u and m <= 256
    assert plan[5] == (16 if vectors else ESIZE[dt])
    if u:
        assert plan[7] == (min(u, 4) if vectors else u)
