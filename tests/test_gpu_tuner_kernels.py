"""What the launch-shape tuner times: not a pass that runs with a block for
every tile (the shape changes nothing there), and no mixture of a pass's
interpreted and compiled runs.  Its decisions are read from the trace of a
process of its own."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = r'''
import sys
import torch
sys.path.insert(0, sys.argv[1])
import paper_2406_18109_amd as dfx
op, n, jit, before = sys.argv[2], int(sys.argv[3]), int(sys.argv[4]), int(sys.argv[5])
c = dfx.Context(device=0, window_size=1, tune=True, jit=jit)
x, y, s = c.store_create([n]), c.store_create([n]), c.store_create([])
T, N = c.part_tiling([n]), c.part_none()
c.submit("fill", [1], [(x, T, "W")], (0.5,))
for i in range(before + 14):
    if i == before:
        c.sync()
        dfx.jit_wait()
        compiled = c.stats()["compiled_launches"]
    if op == "sum":
        c.submit("sum", [1], [(x, T, "R"), (s, N, "Rd")], (1,))
    else:
        c.submit(op, [1], [(x, T, "R"), (y, T, "W")])
    c.sync()
    print("run %d" % i, file=sys.stderr, flush=True)
print("compiled %d then %d" % (compiled, c.stats()["compiled_launches"]), flush=True)
c.close()
'''


def _runs(tmp_path, op, n, jit, before=0):
    """Execution at which the pass's shape was decided (None: never), and how
    many compiled launches there were at the wait and at the end."""
    env = dict(os.environ, DFX_TRACE="1", DFX_JIT_CACHE=str(tmp_path), DFX_COOP="1")
    env.pop("DFX_JIT", None)
    p = subprocess.run([sys.executable, "-c", CHILD, ROOT, op, str(n), str(jit), str(before)], env=env, text=True,
                       capture_output=True, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    at, k = None, 0
    for line in p.stderr.splitlines():
        if line.startswith("run "):
            k += 1
        elif line.startswith("dfx: tuned pass") and "tiles=%d " % ((n + 4095) // 4096) in line:
            at = k
    w = [l.split() for l in p.stdout.splitlines() if l.startswith("compiled ")][0]
    return at, int(w[1]), int(w[3])


@pytest.mark.parametrize("jit", [0, 2])
def test_block_per_tile_passes_are_not_tuned(tmp_path, jit):
    n = 100 * 4096
    assert _runs(tmp_path, "sum", n, jit)[0] is None
    # (warm-up, three shapes twice, and the execution that decides)
    assert _runs(tmp_path, "neg", n, jit)[0] == 7


def test_timings_of_the_interpreted_runs_are_dropped(tmp_path):
    """Four interpreted runs, a warm-up and three timings, then the compiled
    kernel: it is warmed up and timed at every shape itself."""
    at, then, end = _runs(tmp_path, "exp", 300 * 4096, 1, before=4)
    assert end == 14
    if then == 0:
        assert at == 4 + 1 + 6
