"""Argument marshalling of the per-task calls: the common forms (plain ints,
floats and names in lists or tuples), marshalled natively, and all others,
through ctypes, must reach the library alike and fail alike."""
import numpy as np
import pytest

import paper_2406_18109_amd as dfx
from paper_2406_18109_amd import _binding as B


class _Int(int):
    """An int whose exact type is another (so it takes the ctypes route)."""


def _forms(i):
    """The same value as a native-form and as ctypes-form arguments."""
    return [i, _Int(i), np.int64(i)]


def _run(cast, seq, op, priv, dtype, imm):
    c = dfx.Context(device=-1, window_size=8)
    x, y, z = (c.store_create(seq([cast(10), cast(6)]), dtype) for _ in range(3))
    t, n = c.part_tiling(seq([cast(5), cast(6)])), c.part_none()
    c.submit(op("add"), seq([cast(2), cast(1)]), seq([(x, t, priv("R")), (y, t, priv("R")), (z, t, priv("W"))]))
    c.submit(op("mul_imm"), seq([cast(2), cast(1)]), seq([seq([z, t, priv("R")]), (y, t, priv("W"))]), seq(imm))
    c.store_release(cast(z))
    c.flush()
    info = B.dfx_group_info()
    groups = []
    cnt = B.C.c_int64()
    c._chk(c.L.dfx_group_count(c.h, B.C.byref(cnt)))
    for g in range(cnt.value):
        c._chk(c.L.dfx_group_get(c.h, g, B.C.byref(info)))
        groups.append((info.prefix_len, info.n_passes, info.n_temporaries, info.alg_bytes, list(info.temporaries[:4])))
    st = {k: v for k, v in c.stats().items() if "seconds" not in k}
    c.close()
    return (x, y, z, t, n), groups, st


@pytest.mark.parametrize("seq", [list, tuple])
@pytest.mark.parametrize("form", [0, 1, 2])
@pytest.mark.parametrize("named", [True, False])
def test_forms_reach_the_library_alike(seq, form, named):
    ident = (lambda v: v) if named else None
    got = _run(lambda i: _forms(i)[form], seq, ident or (lambda o: B.OPS[o]), ident or (lambda p: B.PRIV[p]),
               "f64" if named else B.F64, [2.5] if form != 1 else [np.float64(2.5)])
    want = _run(int, list, lambda v: v, lambda v: v, "f64", [2.5])
    assert got == want
    assert want[2]["tasks_submitted"] == 2 and len(want[1]) == 1


@pytest.mark.parametrize("call,exc", [
    (lambda c, s, t: c.submit("no_such_op", [1], [(s, t, "R"), (s, t, "W")]), KeyError),
    (lambda c, s, t: c.submit("copy", [1], [(s, t, "Q"), (s, t, "W")]), KeyError),
    (lambda c, s, t: c.submit("copy", [1], [(s, t), (s, t, "W")]), ValueError),
    (lambda c, s, t: c.submit("copy", [1], [("s", t, "R"), (s, t, "W")]), TypeError),
    (lambda c, s, t: c.submit("copy", [1.5], [(s, t, "R"), (s, t, "W")]), TypeError),
    (lambda c, s, t: c.submit("mul_imm", [1], [(s, t, "R"), (s, t, "W")], ("x",)), TypeError),
    (lambda c, s, t: c.submit("copy", [1], [(s, t, "R")] * 17), dfx.DfxError),
    (lambda c, s, t: c.submit("copy", [1] * 5, [(s, t, "R"), (s, t, "W")]), dfx.DfxError),
    (lambda c, s, t: c.submit("copy", [1], [(s + 99, t, "R"), (s, t, "W")]), dfx.DfxError),
    (lambda c, s, t: c.store_create([4], "f16"), KeyError),
    (lambda c, s, t: c.store_create([-4], "f64"), dfx.DfxError),
    (lambda c, s, t: c.store_create([2] * 5, "f64"), dfx.DfxError),
    (lambda c, s, t: c.store_release(s + 99), dfx.DfxError),
    (lambda c, s, t: c.store_release("s"), B.C.ArgumentError),
    (lambda c, s, t: c.part_tiling([1] * 5), dfx.DfxError),
])
def test_wrong_arguments_are_refused(call, exc):
    c = dfx.Context(device=-1)
    s, t = c.store_create([8]), c.part_tiling([8])
    with pytest.raises(exc):
        call(c, s, t)
    c.submit("mul_imm", [1], [(s, t, "R"), (c.store_create([8]), t, "W")], (2,))   # the context still works
    c.flush()
    c.close()


def test_closed_context_is_refused():
    c = dfx.Context(device=-1)
    c.close()
    with pytest.raises(dfx.DfxError):
        c.part_none()
    with pytest.raises(dfx.DfxError):
        c.submit("copy", [1], [(1, 1, "R"), (2, 1, "W")])
