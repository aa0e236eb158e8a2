"""What the host concludes from the control words of a persistent launch
(claim.h, serve.h): every stream settled, some XCD never ran its own, or a
solve was left half done.  The host functions are compiled here and called
with the words such launches leave."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r'''
#include "serve.h"
using namespace dfx;
// solves 0 .. n-1 of tiles[i] tiles, solve i on XCD at[i] of n_xcd
struct Case {
  ServeRound R = {};
  ServeClaim given[64] = {}, now[64] = {};
  int32_t list[64] = {};
  Case(int n, const int* tiles, const int* at, int n_xcd) {
    R.n_xcd = n_xcd;
    int k = 0;
    for (int x = 0; x < n_xcd; ++x) {
      R.x[x].first = k;
      for (int i = 0; i < n; ++i)
        if (at[i] == x) {
          list[k++] = i;
          R.x[x].n_streams += 1;
          given[i].claim = claim_word(PH_INIT, tiles[i], 0);
        }
    }
    for (int i = 0; i < n; ++i) now[i] = given[i];
  }
};
// ran[i]: 0 untouched, 1 settled, 2 begun (a tile claimed), 3 a tile finished
extern "C" int end_of(int n, const int* tiles, const int* at, int n_xcd, const int* ran, const int* error, int* whole) {
  static_assert(sizeof(XcdCtl) == 256, "a line of its own");
  Case c(n, tiles, at, n_xcd);
  for (int i = 0; i < n; ++i) {
    XcdCtl& X = c.R.x[at[i]];
    if (ran[i] == 1) {
      X.n_settled += 1;
      c.now[i].claim = claim_word(23, 0, 1);
      c.now[i].round_iters = 8;
    }
    if (ran[i] >= 2) c.now[i].claim += 1;
    if (ran[i] == 3) c.now[i].done = 1;
  }
  for (int x = 0; x < n_xcd; ++x) c.R.x[x].error = error[x];
  *whole = all_settled(c.R.x, n_xcd) ? 1 : 0;
  return (int)round_end(c.R, c.list, c.given, c.now);
}
'''
WHOLE, UNSERVED, BROKEN = 0, 1, 2


@pytest.fixture(scope="module")
def end_of(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_end")
    (d / "t.cpp").write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2406_18109_amd", "csrc"), str(d / "t.cpp"), "-o", str(d / "t.so")],
                   check=True)
    f = C.CDLL(str(d / "t.so")).end_of

    def call(at, ran, n_xcd=8, error=()):
        n = len(at)
        ints = lambda v: (C.c_int * max(1, len(v)))(*v)
        err = [0] * n_xcd
        for x in error:
            err[x] = 1
        w = C.c_int()
        return f(n, ints([1 + i % 5 for i in range(n)]), ints(at), n_xcd, ints(ran), ints(err), C.byref(w)), w.value
    return call


@pytest.mark.parametrize("at,ran,n_xcd,error,want", [
    ([0, 1, 2, 3, 4, 5, 6, 7, 0], [1] * 9, 8, (), WHOLE),
    ([0, 0, 0], [1, 1, 1], 1, (), WHOLE),
    # an XCD's idle blocks took a long wait for a stall; its solves settled all the same
    ([0, 1, 1], [1, 1, 1], 8, (1, 5), WHOLE),
    # XCD 2, and XCDs 4 to 7, got no block
    ([0, 1, 2, 2], [1, 1, 0, 0], 4, (), UNSERVED),
    ([0, 1, 2, 3, 4, 5, 6, 7], [1, 1, 1, 1, 0, 0, 0, 0], 8, (), UNSERVED),
    ([0, 1], [0, 0], 2, (), UNSERVED),
    # a solve begun and not settled
    ([0, 1, 1], [1, 1, 2], 8, (), BROKEN),
    ([0, 1, 1], [1, 0, 3], 8, (1,), BROKEN),
    ([0, 1, 2], [1, 0, 2], 4, (), BROKEN),
])
def test_end_of_a_round(end_of, at, ran, n_xcd, error, want):
    got, whole = end_of(at, ran, n_xcd, error)
    assert got == want and whole == (want == WHOLE)
