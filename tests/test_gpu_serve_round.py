"""The solve server's two kinds of round, one persistent launch and phase
launches, at the sizes where the persistent one can go wrong: a partial
tile, the last element of one, one to three tiles, more than 256 tiles (two
levels of tile sums).  Both must give the bits and counts of the other, and
of apps.CG."""
import numpy as np
import pytest

import paper_2406_18109_amd as dfx
import synth
from gpu_util import note, upload

pytestmark = pytest.mark.gpu


def _serve(mats, bs, iters, ipr):
    c = dfx.Context(device=0)
    c.serve_start(hbm_budget=8 << 30, max_slots=16, tol=1e-8, max_iter=iters, iters_per_round=ipr)
    tickets = [c.serve_submit(*m, b) for m, b in zip(mats, bs)]
    res = [c.serve_wait(t, 100) for t in tickets]
    xs = [c.serve_read_x(t, b.size) for t, b in zip(tickets, bs)]
    c.serve_stop()
    c.close()
    return [(r["status"], r["iterations"], r["rel_residual"]) for r in res], xs


@pytest.mark.parametrize("sides,iters,ipr", [
    ((1, 2, 5, 11, 16, 63, 64, 65, 91, 110), 400, 7),
    ((16, 1030), 12, 4),    # 1030^2: 260 tiles
])
def test_rounds_agree(monkeypatch, sides, iters, ipr):
    note("serve rounds sides=%s" % (sides,))
    mats = [synth.poisson_csr(m, 2) for m in sides]
    bs = [synth.rhs(m * m, 7000 + m) for m in sides]
    out = []
    for mode in ("1", "0"):
        monkeypatch.setenv("DFX_SERVE_ROUND", mode)
        out.append(_serve(mats, bs, iters, ipr))
    assert out[0][0] == out[1][0]
    for a, b in zip(out[0][1], out[1][1]):
        assert np.array_equal(a, b)
    # the same solve through the task-stream executor
    m, (status, its, _), x = sides[-1], out[0][0][-1], out[0][1][-1]
    c = dfx.Context(device=0, window_size=16)
    cg = dfx.apps.CG(c, *[upload(c, v) for v in mats[-1] + (bs[-1],)], m * m)
    for _ in range(its):
        cg.iteration()
    assert np.array_equal(c.store_read(cg.x, [m * m], "f64"), x)
    c.close()
