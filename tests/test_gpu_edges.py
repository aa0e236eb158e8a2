"""Rows whose width is no multiple of a lane's vector, and streams with one
value per row or per column, interpreted and compiled: every element must be
numpy's (each operation rounds on its own), and the sum that of the unfused
run, bit for bit."""
import numpy as np
import pytest

import paper_2406_18109_amd as dfx
import synth
import test_gpu_stencil as st
from gpu_util import note, upload

pytestmark = pytest.mark.gpu


def _run(dtype, R, C, off, jit, fuse, monkeypatch, arrs):
    monkeypatch.delenv("DFX_JIT", raising=False)
    c = dfx.Context(device=0, window_size=8, fuse=fuse, jit=jit)
    A, mu, w = arrs
    h, k = R - off[0], C - off[1]
    ha, hm, hw = upload(c, A), upload(c, mu[:k]), upload(c, w[:h])
    hy = upload(c, np.zeros((R, C), A.dtype))
    hs = c.store_create([], dtype)
    V = c.part_tiling([h, k], list(off))
    T = c.part_tiling([h, k])
    by, br, N = c.part_tiling([k], proj=c.proj_drop(2, 2)), c.part_tiling([h], proj=c.proj_drop(2, 1)), c.part_none()
    t1, t2 = c.store_create([h, k], dtype), c.store_create([h, k], dtype)
    d = [1, 1]
    c.submit("sub", d, [(ha, V, "R"), (hm, by, "R"), (t1, T, "W")])
    c.submit("mul", d, [(t1, T, "R"), (hw, br, "R"), (t2, T, "W")])
    c.submit("add", d, [(t2, T, "R"), (ha, V, "R"), (hy, V, "W")])
    c.store_release(t1)
    c.store_release(t2)
    c.submit("sumsq", d, [(hy, V, "R"), (hs, N, "Rd")], (1,))
    y, s = c.store_read(hy, [R, C], dtype), c.store_read(hs, [], dtype)
    c.close()
    return y, s


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("off", [(0, 0), (1, 1)])
@pytest.mark.parametrize("C", [1, 2, 3, 4, 5, 6, 127, 128, 130, 255, 257, 259, 514])
def test_ragged_rows_and_broadcasts(dtype, off, C, monkeypatch):
    if C <= off[1]:
        pytest.skip("no column left")
    note("edges %s off=%s C=%d" % (dtype, off, C))
    R = 67
    npdt = np.float64 if dtype == "f64" else np.float32
    A = synth.uniform(21, 0, R * C, -1.0, 1.0).astype(npdt).reshape(R, C)
    mu, w = synth.uniform(21, 1, C, 0.0, 1.0).astype(npdt), synth.uniform(21, 2, R, 0.5, 1.0).astype(npdt)
    a = A[off[0]:, off[1]:]
    ey = np.zeros((R, C), npdt)
    ey[off[0]:, off[1]:] = (a - mu[None, :C - off[1]]) * w[:R - off[0], None] + a
    ref = _run(dtype, R, C, off, 0, False, monkeypatch, (A, mu, w))
    for jit in (0, 2):
        y, s = _run(dtype, R, C, off, jit, True, monkeypatch, (A, mu, w))
        assert np.array_equal(y, ey), jit
        assert np.array_equal(s, ref[1]), jit


@pytest.mark.parametrize("make", [st._five_point, st._diagonal, st._horizontal])
@pytest.mark.parametrize("shape", [(66, 131), (67, 259), (66, 257), (99, 5), (34, 388), (130, 130)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("jit,coop", [(0, "0"), (2, "0"), (0, "1"), (2, "1")])
def test_stencil_strip_across_the_right_edge(make, shape, dtype, jit, coop, monkeypatch):
    """Staged tiles whose last strip is 1, 2, 3, ... columns wide, with a stream
    that is not staged; and the same passes with a block for every tile."""
    tasks, outs, temps = make(shape)
    n = shape[0] * shape[1]
    G = synth.uniform(17, 0, n, 0.5, 2.0).reshape(shape)
    H = synth.uniform(17, 1, n, 0.5, 2.0).reshape(shape)
    want = st._run_gpu(tasks, outs, temps, G, H, dtype, False)
    monkeypatch.setenv("DFX_COOP", coop)
    monkeypatch.setattr(st, "ctx", lambda fuse, window: dfx.Context(device=0, window_size=window, fuse=fuse, jit=jit))
    got = st._run_gpu(tasks, outs, temps, G, H, dtype, True)
    for k in outs:
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)
