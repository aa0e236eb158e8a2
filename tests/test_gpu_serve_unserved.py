"""A persistent round of the solve server that reaches only some XCDs: the
solves pinned to the others are untouched by it and run by phase launches from
the next round on, with the bits and counts of a server that never used the
persistent round."""
import numpy as np
import pytest

import synth
from gpu_util import note
from test_gpu_serve_round import _serve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 3, 8])
def test_unserved_solves_run_by_phases(blocks, monkeypatch):
    note("serve with %d blocks a round" % blocks)
    sides = (1, 16, 63, 64, 65, 91, 110, 20, 33, 130)
    mats = [synth.poisson_csr(m, 2) for m in sides]
    bs = [synth.rhs(m * m, 8000 + m) for m in sides]
    monkeypatch.setenv("DFX_SERVE_ROUND", "0")
    want = _serve(mats, bs, 400, 7)
    monkeypatch.setenv("DFX_SERVE_ROUND", "1")
    monkeypatch.setenv("DFX_SERVE_BLOCKS", str(blocks))
    got = _serve(mats, bs, 400, 7)
    assert got[0] == want[0]
    for a, b in zip(got[1], want[1]):
        assert np.array_equal(a, b)
