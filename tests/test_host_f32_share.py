"""How the float32 attention deals a launch out: every 16 queries of every half block belong to one workgroup, whatever mixture
of halves and pieces the rule takes.  The kernel's own functions, compiled for the CPU."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_14708_amd", "csrc")
SOURCE = """#include "f32_share.h"
using namespace da;
extern "C" unsigned pieces(long long halves, int even, int d, int* out) {
  const F32Share s = f32_share_out(halves, even, d);
  for (unsigned b = 0; out && b < s.grid; ++b) {
    const F32Piece p = f32_piece(s, b);
    out[3 * b] = (int)p.half; out[3 * b + 1] = p.second; out[3 * b + 2] = p.queries;
  }
  return s.grid;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("f32_share")
    src, out = d / "f32_share.cpp", d / "libf32_share.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(out)], check=True)
    f = ctypes.CDLL(str(out))
    f.pieces.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    return f


@pytest.mark.parametrize("even", [0, 1])
@pytest.mark.parametrize("d", [64, 128])
def test_every_query_has_one_workgroup(lib, d, even):
    mixtures = set()
    for halves in [*range(2, 1400, 2), 1680, 2688, 3360, 6720]:
        grid = lib.pieces(halves, even, d, None)
        out = (ctypes.c_int * (3 * grid))()
        lib.pieces(halves, even, d, out)
        times = [[0, 0] for _ in range(halves)]
        sizes = set()
        for b in range(grid):
            half, second, queries = out[3 * b:3 * b + 3]
            assert half >= 0 and queries in (16, 32) and second in (0, 1) and second * 16 + queries <= 32
            if half >= halves:
                continue
            sizes.add(queries)
            for part in range(second, second + queries // 16):
                times[half][part] += 1
        assert all(t == [1, 1] for t in times)
        mixtures.add(tuple(sorted(sizes)))
    assert mixtures == {(16,), (32,), (16, 32)}


def test_which_last_rounds_are_cut(lib):
    """Where all half blocks last as long, a last round of more than half as many as CUs, and no more than CUs, takes as long in pieces: a
    CU has two, and K and V are read twice."""
    for d, places, most in ((128, 64, 40), (64, 96, 20)):
        for rounds in (1, 2, 3, 4):
            for last in range(1, places):
                chunk = rounds * places + last
                cut = [lib.pieces(8 * chunk, even, d, None) // 8 - chunk for even in (0, 1)]
                assert cut == [last if last <= most else 0, last if last <= 16 or 32 < last <= most else 0], (d, rounds, last)
