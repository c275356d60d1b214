"""How the bf16 attention deals a launch out: every query block of a head belongs to one place of one unit, every share of
every unit to one workgroup, the shares of a unit stay on one XCD (workgroups go to the XCDs in turn), and no more than a
few workgroups have nothing to do.  The kernel's own functions, compiled for the CPU."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_14708_amd", "csrc")
SOURCE = """#include "ring_turns.h"
using namespace da::ring;
extern "C" int units(int T, int fg, int per_frame) { return units_per_head(T, fg, per_frame); }
extern "C" void place(int n, int T, int log_fg, int per_frame, int* out) {
  const UnitPlace u = unit_place(n, T, log_fg, per_frame);
  for (int w = 0; w < 1 << log_fg; ++w) { out[2 * w] = unit_pos(u, w); out[2 * w + 1] = unit_frame(u, w); }
}
extern "C" void share(long long total, long long tiles, int any_length, int least, int* out) {
  const Share s = share_out(total, tiles, any_length, least);
  out[0] = s.first; out[1] = s.split[0]; out[2] = s.split[1]; out[3] = (int)s.grid;
}
extern "C" void shares(long long total, long long tiles, int any_length, int least, int grid, int* out) {
  const Share s = share_out(total, tiles, any_length, least);
  for (int b = 0; b < grid; ++b) {
    const ShareOf w = share_of(s, b);
    out[3 * b] = w.unit; out[3 * b + 1] = w.lsub; out[3 * b + 2] = w.sub;
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("unit_places")
    src, out = d / "unit_places.cpp", d / "libunit_places.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(out)], check=True)
    f = ctypes.CDLL(str(out))
    f.share.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    f.shares.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    return f


@pytest.mark.parametrize("log_fg", [2, 3])
@pytest.mark.parametrize("per_frame", [1, 2, 7, 8, 28, 60])
def test_every_block_has_one_place(lib, log_fg, per_frame):
    fg, out = 1 << log_fg, (ctypes.c_int * 16)()
    for T in list(range(1, 36)) + [65]:
        seen, positions = set(), []
        units = lib.units(T, fg, per_frame)
        for n in range(units):
            lib.place(n, T, log_fg, per_frame, out)
            blocks = [(out[2 * w], out[2 * w + 1]) for w in range(fg)]
            live = [b for b in blocks if b[0] < per_frame]
            assert blocks[:len(live)] == live and live          # empty places only at the end
            assert all(f < T for _, f in live)
            assert not seen & set(live)
            seen |= set(live)
            positions.append(len({p for p, _ in live}))
        assert len(seen) == T * per_frame
        assert units == -(-T * per_frame // fg)                 # at most one unit with empty places
        # left-over frames of a position are in one unit or in two: as few positions to a unit as that allows
        left = T % fg
        assert max(positions) <= (1 if not left else -(-fg // left) + 1)
        assert sum(positions) <= units + per_frame * (left > 0)


@pytest.mark.parametrize("least", [0, 1])
@pytest.mark.parametrize("any_length", [0, 1])
@pytest.mark.parametrize("tiles", [3, 200])
def test_every_share_has_one_workgroup(lib, tiles, any_length, least):
    s = (ctypes.c_int * 4)()
    for total in list(range(1, 540)) + [1023, 1024, 1025, 5952]:
        lib.share(total, tiles, any_length, least, s)
        first, split0, split1, grid = s
        assert min(split0, split1) >= least and grid > 0
        out = (ctypes.c_int * (3 * grid))()
        lib.shares(total, tiles, any_length, least, grid, out)
        seen, xcd, idle = set(), {}, 0
        for b in range(grid):
            unit, lsub, sub = out[3 * b:3 * b + 3]
            if unit >= total:
                idle += 1
                continue
            assert lsub == (split0 if unit < first else split1) and 0 <= sub < 1 << lsub
            assert (unit, sub) not in seen
            seen.add((unit, sub))
            assert xcd.setdefault(unit, b % 8) == b % 8
        assert len(seen) == sum(1 << (split0 if u < first else split1) for u in range(total))
        assert idle <= 7 << max(split0, split1)


def test_full_rounds_are_not_shared(lib):
    """Lists of one length: where the last of up to four rounds is empty or more than half full every unit is one workgroup, and no
    CU gets a third share of a launch of less than a round."""
    s = (ctypes.c_int * 4)()
    for tiles in (3, 26, 40, 200):
        for total in range(1, 1025):
            lib.share(total, tiles, 0, 0, s)
            first, split0, split1, grid = s
            if total > 256 and (total % 256 == 0 or total % 256 > 128) or 192 < total <= 256:
                assert (first, split0, grid) == ((total + 7) // 8 * 8, 0, (total + 7) // 8 * 8)
            if 128 < total <= 192:
                assert grid <= 512 and (split0 == 0 or tiles >= 36)
