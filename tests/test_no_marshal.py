"""The binding without its marshalling module (not built, or built for another
Python): every call takes the ctypes route, with the same results; and the
build goes on without a C++ compiler for it."""
import os
import subprocess
import sys

import paper_2406_18109_amd as dfx
from paper_2406_18109_amd import _binding as B
from paper_2406_18109_amd import build as bld
from test_marshal import _run

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_ctypes_route_alone(monkeypatch):
    args = (int, list, lambda v: v, lambda v: v, "f64", [2.5])
    B.lib()
    want = _run(*args)
    monkeypatch.setattr(B, "_fast", B._CtypesOnly)
    assert _run(*args) == want


def test_package_loads_without_the_module():
    code = ("import sys; sys.path.insert(0, %r); sys.modules['paper_2406_18109_amd._marshal'] = None\n"
            "import paper_2406_18109_amd as dfx\n"
            "c = dfx.Context(device=-1); x = c.store_create([8]); y = c.store_create([8]); t = c.part_tiling([8])\n"
            "c.submit('copy', [1], [(x, t, 'R'), (y, t, 'W')]); c.store_release(x); c.part_none(); c.flush()\n"
            "print(c.stats()['tasks_submitted'])" % ROOT)
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    assert p.returncode == 0 and p.stdout.split() == ["1"], p.stderr


def test_build_goes_on_without_a_compiler(monkeypatch, tmp_path):
    (tmp_path / "csrc").mkdir()
    monkeypatch.setattr(bld, "HERE", str(tmp_path))
    monkeypatch.setattr(bld, "CSRC", str(tmp_path / "csrc"))   # no source: the compiler fails
    assert bld.build_marshal() == ""
    monkeypatch.setenv("PATH", str(tmp_path))                  # no compiler at all
    assert bld.build_marshal() == ""
    assert not [f for f in os.listdir(tmp_path) if f.startswith("_marshal")]
    assert dfx.Context(device=-1).part_none() >= 0
