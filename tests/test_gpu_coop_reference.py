"""The block-per-tile kernel against one wave per tile, without the kernel on
the reference's side: an unfused run takes the block-per-tile kernel for its
own small reductions unless it is turned off, and would then share a mistake
in the order of the sums."""
import numpy as np
import pytest

import synth
import test_gpu_coop as tc
import test_gpu_edges as te
from gpu_util import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", tc.SIZES)
def test_batch_tiles_equal_one_wave(n, monkeypatch):
    # (the batch's own kernel does not look at DFX_COOP)
    monkeypatch.setenv("DFX_COOP", "0")
    tc.test_batch_tiles_equal_ordinary(n)


@pytest.mark.parametrize("nnz_row", [0, 1, 7, 8, 9, 40])
def test_batch_spmv_rows_equal_one_wave(nnz_row, monkeypatch):
    monkeypatch.setenv("DFX_COOP", "0")
    tc.test_batch_spmv_rows_of_every_length(nnz_row)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 127, 129, 4095, 4097, 16385, 70001])
def test_unfused_passes_equal_one_wave(n, dtype, monkeypatch):
    want = tc._pass_results(n, dtype, monkeypatch, False, fuse=False)
    got = tc._pass_results(n, dtype, monkeypatch, True, fuse=False)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("off", [(0, 0), (1, 1)])
@pytest.mark.parametrize("C", [2, 4, 5, 127, 128, 130, 257, 514])
def test_ragged_table_sums_equal_one_wave(dtype, off, C, monkeypatch):
    note("ragged sums %s off=%s C=%d" % (dtype, off, C))
    R, npdt = 67, np.float64 if dtype == "f64" else np.float32
    A = synth.uniform(22, 0, R * C, -1.0, 1.0).astype(npdt).reshape(R, C)
    mu, w = synth.uniform(22, 1, C, 0.0, 1.0).astype(npdt), synth.uniform(22, 2, R, 0.5, 1.0).astype(npdt)
    monkeypatch.setenv("DFX_COOP", "0")
    ref = te._run(dtype, R, C, off, 0, False, monkeypatch, (A, mu, w))
    monkeypatch.setenv("DFX_COOP", "1")
    for jit, fuse in ((0, False), (0, True), (2, True)):
        y, s = te._run(dtype, R, C, off, jit, fuse, monkeypatch, (A, mu, w))
        assert np.array_equal(y, ref[0]) and np.array_equal(s, ref[1]), (jit, fuse)
