"""Batches of different needs (a pass of one reduction, one of four: 32 and
128 KB of LDS a block) run from two threads at once, each over its own
stream: every run must give what the ordinary flush gives."""
import threading

import numpy as np
import pytest

import paper_2406_18109_amd as dfx
import synth
from gpu_util import note, upload

pytestmark = pytest.mark.gpu
N = 20001
REDS = (("sum", "x"), ("sumsq", "x"), ("dot", "xy"), ("sum", "y"))


def _tasks(c, h, k):
    T, none = c.part_tiling([N]), c.part_none()
    for (op, ins), s in zip(REDS[:k], h[2:]):
        c.submit(op, [1], [(h["xy".index(a)], T, "R") for a in ins] + [(s, none, "Rd")], (1,))


def _stores(c):
    return [upload(c, synth.uniform(40, i, N, -1.0, 1.0)) for i in range(2)] + [c.store_create([]) for _ in REDS]


def _work(k, want, bad):
    c = dfx.Context(device=0, window_size=8)
    h = _stores(c)
    _tasks(c, h, k)
    c.sync()   # every store has its memory
    b = dfx.Batch(device=0)
    b.record_begin(c)
    _tasks(c, h, k)
    b.record_end(c)
    for _ in range(12):
        b.run()
        b.wait()
        got = [float(c.store_read(s, [], "f64")) for s in h[2:2 + k]]
        if got != want[:k]:
            bad.append((k, got))
    b.close()
    c.close()


def test_batches_of_two_threads(monkeypatch):
    note("batches from two threads")
    monkeypatch.setenv("DFX_COOP", "0")
    c = dfx.Context(device=0, window_size=8, fuse=False)
    h = _stores(c)
    _tasks(c, h, 4)
    want = [float(c.store_read(s, [], "f64")) for s in h[2:]]
    c.close()
    bad, errs = [], []

    def guarded(k):
        try:
            _work(k, want, bad)
        except Exception as e:   # noqa: BLE001  (reported below)
            errs.append(repr(e))
    ts = [threading.Thread(target=guarded, args=(k,)) for k in (1, 4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errs and not bad
    assert np.isfinite(want).all()
