"""How many blocks a persistent round of the solve server takes on each XCD
(serve.h): never more than its fullest XCD has tiles, and not every compute
unit, so that kernels of the device's other streams run beside it, unless a
solve needs them all.  The host function is compiled here."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r'''
#include "serve.h"
using namespace dfx;
extern "C" int blocks(int n, const int* tiles, const int* at, int n_xcd, int units) {
  XcdLoad load[MAX_XCD] = {};
  for (int i = 0; i < n; ++i) {
    load[at[i]].tiles += tiles[i];
    load[at[i]].solves += 1;
  }
  return blocks_per_xcd(load, n_xcd, units);
}
'''


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    d = tmp_path_factory.mktemp("round_blocks")
    (d / "t.cpp").write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2406_18109_amd", "csrc"), str(d / "t.cpp"), "-o", str(d / "t.so")],
                   check=True)
    f = C.CDLL(str(d / "t.so")).blocks

    def call(solves, n_xcd=8, units=32):
        ints = lambda v: (C.c_int * max(1, len(v)))(*v)
        return f(len(solves), ints([t for t, _ in solves]), ints([x for _, x in solves]), n_xcd, units)
    return call


@pytest.mark.parametrize("solves,want", [
    ([], 1),
    ([(1, 0)], 1),
    ([(16, 3)], 16),
    ([(16, x) for x in range(8)], 16),
    ([(28, 0)], 28),
    # shared XCDs: seven eighths of the compute units
    ([(16, x % 8) for x in range(16)], 28),
    ([(16, x % 8) for x in range(48)], 28),
    ([(20, 0), (12, 0)], 28),
    # alone, a pass more with 28 blocks: all
    ([(29, 0)], 29),
    ([(32, 0)], 32),
    ([(57, 1)], 32),
    ([(64, x) for x in range(8)], 32),
    ([(16, x) for x in range(7)] + [(32, 7)], 32),
    # alone, the same passes: 28
    ([(33, 0)], 28),
    ([(56, 0)], 28),
    ([(98, 5)], 28),
])
def test_blocks_of_a_round(blocks, solves, want):
    assert blocks(solves) == want


@pytest.mark.parametrize("units", [1, 2, 7, 8, 20, 32, 38])
def test_some_block_always(blocks, units):
    for t in (1, units, units + 1, 3 * units):
        got = blocks([(t, 0), (1, 0)], 1, units)
        assert 1 <= got <= min(t + 1, units)
