"""Steps at a space's edge whose vectors are inside or outside as a whole, and
those a vector crosses: sums of one to six streams over rows of whole and
split widths, over a view one element in (strips shifted, both edges split),
and in one dimension; interpreted and compiled.  Every element must be
numpy's, and nothing outside the space may be written."""
import numpy as np
import pytest

import paper_2406_18109_amd as dfx
import synth
from gpu_util import note, upload

pytestmark = pytest.mark.gpu


def _sum(shape, off, dtype, S, jit):
    """out[view] = x0[view] + x1[view] + ... (S = 1: times 1.5, in place)."""
    npdt = np.float64 if dtype == "f64" else np.float32
    full = [d + 2 * off for d in shape]
    n = int(np.prod(full))
    xs = [synth.uniform(50, k, n, -1.0, 1.0).astype(npdt).reshape(full) for k in range(S)]
    c = dfx.Context(device=0, window_size=8, jit=jit)
    hs = [upload(c, x) for x in xs]
    out0 = np.full(full, 7.0, npdt)
    ho = hs[0] if S == 1 else upload(c, out0)
    V, T, d = c.part_tiling(list(shape), [off] * len(shape)), c.part_tiling(list(shape)), [1] * len(shape)
    if S == 1:
        c.submit("mul_imm", d, [(ho, V, "R"), (ho, V, "W")], (1.5,))
    cur, part, tmp = hs[0], V, []
    for k in range(1, S):
        last = k == S - 1
        t = ho if last else c.store_create(list(shape), dtype)
        c.submit("add", d, [(cur, part, "R"), (hs[k], V, "R"), (t, V if last else T, "W")])
        cur, part = t, T
        tmp += [] if last else [t]
    for t in tmp:
        c.store_release(t)
    got = c.store_read(ho, full, dtype)
    c.close()
    view = tuple(slice(off, off + w) for w in shape)
    want = xs[0].copy() if S == 1 else out0
    acc = xs[0][view]
    for x in xs[1:]:
        acc = acc + x[view]
    want[view] = acc * npdt(1.5) if S == 1 else acc
    return got, want


@pytest.mark.parametrize("jit", [0, 2])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("S", [1, 2, 3, 4, 5, 6])
def test_edges_of_whole_and_split_vectors(S, dtype, jit):
    note("edge modes S=%d %s jit=%d" % (S, dtype, jit))
    for shape in ((67, 4), (33, 6), (67, 100), (32, 128), (67, 131), (35, 260), (31, 254),
                  (4,), (6,), (130,), (4100,), (4103,), (8192,), (8190,)):
        for off in (0, 1):
            got, want = _sum(shape, off, dtype, S, jit)
            assert np.array_equal(got, want), (shape, off)
