"""Tiles run by a whole block (coop_exec.h) at the sizes where they can go
wrong: SpMV rows of no, few and many entries up to the end of the arrays,
partial rows and tiles, several reductions in one pass, single-element
passes.  Every result must have the bits of the ordinary (unfused, one wave
per tile) execution of the same tasks."""
import numpy as np
import pytest

import paper_2406_18109_amd as dfx
import synth
from gpu_util import note, upload
from test_gpu_parity import _irregular_csr

pytestmark = pytest.mark.gpu


def _tasks(c, h, n):
    """y = A x; s0 = x.y; s1 = y.y; z = y / s1 + x; s2 = sum z."""
    rp, col, val, x, y, z, s0, s1, s2, t = h
    N, T, img = c.part_none(), c.part_tiling([n]), c.part_image(col, c.part_none())
    c.submit("spmv_csr", [1], [(rp, N, "R"), (col, N, "R"), (val, N, "R"), (x, img, "R"), (y, T, "W")])
    c.submit("dot", [1], [(x, T, "R"), (y, T, "R"), (s0, N, "Rd")], (1,))
    c.submit("dot", [1], [(y, T, "R"), (y, T, "R"), (s1, N, "Rd")], (1,))
    c.submit("add_imm", [], [(s1, N, "R"), (t, N, "W")], (1.0,))
    c.submit("copy", [1], [(x, T, "R"), (z, T, "W")])
    c.submit("axpy", [1], [(t, N, "R"), (y, T, "R"), (z, T, "RW")], (-1.0,))
    c.submit("sum", [1], [(z, T, "R"), (s2, N, "Rd")], (1,))


def _stores(c, n, dtype, mats):
    rp, col, val, x = mats
    npdt = np.float64 if dtype == "f64" else np.float32
    h = [upload(c, rp), upload(c, col), upload(c, val.astype(npdt)), upload(c, x.astype(npdt))]
    h += [upload(c, np.zeros(n, npdt)) for _ in range(2)] + [upload(c, np.zeros((), npdt)) for _ in range(4)]
    return h


def _read(c, h, n, dtype):
    return [c.store_read(h[4], [n], dtype), c.store_read(h[5], [n], dtype)] + [c.store_read(s, [], dtype) for s in h[6:]]


def _mats(n):
    rp, col, val = _irregular_csr(n, 70 + n)
    return rp, col, val, synth.uniform(71 + n, 0, n, -1.0, 1.0)


def _ordinary(n, dtype):
    c = dfx.Context(device=0, window_size=8, fuse=False)
    h = _stores(c, n, dtype, _mats(n))
    _tasks(c, h, n)
    out = _read(c, h, n, dtype)
    c.close()
    return out


SIZES = [1, 2, 5, 63, 64, 65, 127, 128, 129, 257, 1000, 4095, 4096, 4097, 9001]


@pytest.mark.parametrize("n", SIZES)
def test_batch_tiles_equal_ordinary(n):
    note("coop batch n=%d" % n)
    ref = _ordinary(n, "f64")
    c = dfx.Context(device=0, window_size=8)
    h = _stores(c, n, "f64", _mats(n))
    b = dfx.Batch(device=0)
    b.record_begin(c)
    _tasks(c, h, n)
    b.record_end(c)
    for _ in range(2):   # the second run restarts on the first one's stores
        b.run()
        b.wait()
        for g, r in zip(_read(c, h, n, "f64"), ref):
            assert np.array_equal(g, r)
    b.close()
    c.close()


@pytest.mark.parametrize("nnz_row", [0, 1, 7, 8, 9, 40])
def test_batch_spmv_rows_of_every_length(nnz_row):
    """Equal rows of one length, so that the last rows end at the arrays' end
    (an empty matrix among them)."""
    note("coop batch rows of %d" % nnz_row)
    n = 200
    rng = np.random.RandomState(nnz_row)
    rp = (np.arange(n + 1) * nnz_row).astype(np.int32)
    col = np.concatenate([np.sort(rng.permutation(n)[:nnz_row]) for _ in range(n)] or [[]]).astype(np.int32)
    val = rng.uniform(-1, 1, col.size)
    if col.size == 0:   # a store needs an element
        col, val = np.zeros(1, np.int32), np.zeros(1)
    x = rng.uniform(-1, 1, n)
    out = []
    for batched in (False, True):
        c = dfx.Context(device=0, window_size=8, fuse=batched)
        h = _stores(c, n, "f64", (rp, col, val, x))
        if batched:
            b = dfx.Batch(device=0)
            b.record_begin(c)
            _tasks(c, h, n)
            b.record_end(c)
            b.run()
            b.wait()
            b.close()
        else:
            _tasks(c, h, n)
        out.append(_read(c, h, n, "f64"))
        c.close()
    for g, r in zip(*out):
        assert np.array_equal(g, r)


def _pass_results(n, dtype, monkeypatch, coop, **cfg):
    monkeypatch.setenv("DFX_COOP", "1" if coop else "0")
    c = dfx.Context(device=0, window_size=8, **cfg)
    h = _stores(c, n, dtype, _mats(n))
    for _ in range(2):
        _tasks(c, h, n)
    out = _read(c, h, n, dtype)
    c.close()
    return out


@pytest.mark.parametrize("jit", [0, 2])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 127, 129, 4095, 4096, 4097, 8193, 16385, 70001])
def test_pass_with_a_block_per_tile_equals_ordinary(n, dtype, jit, monkeypatch):
    """Reducing passes over one tile, 2 to 4 (one block of the ordinary kernel)
    and more, ending in a partial row or tile, with one and two reductions."""
    want = _pass_results(n, dtype, monkeypatch, False, fuse=False)
    got = _pass_results(n, dtype, monkeypatch, True, jit=jit)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("jit", [0, 2])
@pytest.mark.parametrize("shape", [(1, 1), (33, 127), (31, 129), (70, 300), (4100, 3)])
def test_2d_sum_with_a_block_per_tile(shape, jit, monkeypatch):
    """Two-dimensional reductions with ragged rows and strips."""
    res = []
    for coop in (False, True):
        monkeypatch.setenv("DFX_COOP", "1" if coop else "0")
        c = dfx.Context(device=0, window_size=4, fuse=coop, jit=jit if coop else 0)
        v = synth.uniform(90, 0, shape[0] * shape[1], -1.0, 1.0).reshape(shape)
        x, y, s = upload(c, v), upload(c, np.zeros(shape)), upload(c, np.zeros(()))
        T, N = c.part_tiling(list(shape)), c.part_none()
        c.submit("mul_imm", [1, 1], [(x, T, "R"), (y, T, "W")], (3.0,))
        c.submit("sum", [1, 1], [(y, T, "R"), (s, N, "Rd")], (1,))
        res.append((c.store_read(y, list(shape), "f64"), c.store_read(s, [], "f64")))
        c.close()
    for a, b in zip(res[1], res[0]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("dtype,n", [("f64", 255 * 4096 + 1), ("f64", 256 * 4096), ("f32", 255 * 8192 + 70)])
def test_large_spmv_with_a_block_per_tile(dtype, n, monkeypatch):
    """An SpMV without reductions over 256 tiles, its last one partial: rows of
    0 to 11 entries, fused with an axpy, compiled."""
    rng = np.random.default_rng(5)
    rp = np.concatenate([[0], np.cumsum(rng.integers(0, 12, n))]).astype(np.int32)
    col = rng.integers(0, n, rp[-1]).astype(np.int32)
    npdt = np.float64 if dtype == "f64" else np.float32
    val, x = rng.uniform(-1, 1, rp[-1]).astype(npdt), rng.uniform(-1, 1, n).astype(npdt)
    res = []
    for coop in ("0", "1"):
        monkeypatch.setenv("DFX_COOP", coop)
        c = dfx.Context(device=0, window_size=4, jit=2)
        h = [upload(c, a) for a in (rp, col, val, x)]
        y, r, s = c.store_create([n], dtype), upload(c, x), upload(c, np.asarray(0.5, npdt))
        N, T, img = c.part_none(), c.part_tiling([n]), c.part_image(h[1], c.part_none())
        c.submit("spmv_csr", [1], [(h[0], N, "R"), (h[1], N, "R"), (h[2], N, "R"), (h[3], img, "R"), (y, T, "W")])
        c.submit("axpy", [1], [(s, N, "R"), (y, T, "R"), (r, T, "RW")], (-1.0,))
        c.flush()
        res.append((c.store_read(y, [n], dtype), c.store_read(r, [n], dtype)))
        c.close()
    for a, b in zip(*res):
        np.testing.assert_array_equal(b, a)
