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
extern "C" long long aux(long long g, long long k, int sub, int any_length, int split) { return aux_bytes(g, k, sub, any_length, split); }
extern "C" int fits(long long g, long long k, int sub, int any_length) { return lists_fit(g, k, sub, any_length); }
extern "C" int least(long long g, long long k, int sub, int any_length) { return least_split(g, k, sub, any_length); }
extern "C" int left(int T, int fg, int per_frame) { return left_units(T, fg, per_frame); }
extern "C" void share(long long heads, long long head_groups, long long tiles, int any_length, int least, int* out) {
  const Share s = share_out(heads, head_groups, tiles, any_length, least);
  out[0] = s.first; out[1] = s.split[0]; out[2] = s.split[1]; out[3] = (int)s.grid; out[4] = s.head_shares;
}
extern "C" void shares(long long heads, long long head_groups, long long tiles, int any_length, int least, int per_head, int left,
                       int grid, int* out) {
  const Share s = share_out(heads, head_groups, tiles, any_length, least);
  for (int b = 0; b < grid; ++b) {
    const ShareOf w = share_of(s, b, per_head, left);
    out[4 * b] = w.head; out[4 * b + 1] = w.unit; out[4 * b + 2] = w.lsub; out[4 * b + 3] = w.sub;
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
    f.share.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int] * 2 + [ctypes.c_void_p]
    f.aux.argtypes = f.fits.argtypes = f.least.argtypes = [ctypes.c_longlong] * 2 + [ctypes.c_int] * 3
    f.fits.argtypes, f.least.argtypes, f.aux.restype = f.fits.argtypes[:4], f.least.argtypes[:4], ctypes.c_longlong
    f.shares.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int] * 5 + [ctypes.c_void_p]
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
@pytest.mark.parametrize("tiles", [1, 3, 200])
def test_every_share_has_one_workgroup(lib, tiles, any_length, least):
    s = (ctypes.c_int * 5)()
    cases = [(total, 8, 1, 8) for total in list(range(1, 540)) + [1023, 1024, 1025, 5952]]               # (heads, T, positions, blocks to a unit)
    cases += [(heads, T, pf, fg) for heads in (1, 3, 12, 36, 250, 300) for T in (1, 2, 3, 7, 9) for pf in (1, 2, 5, 28, 42) for fg in (8, 4)]
    for heads, T, per_frame, fg in cases:
        head_groups, per_head, left = T * per_frame * (8 // fg), lib.units(T, fg, per_frame), lib.left(T, fg, per_frame)
        lib.share(heads, head_groups, tiles, any_length, least, s)
        first, split0, split1, grid, head_shares = s
        assert min(split0, split1) >= least and grid > 0 and first >= 0
        out = (ctypes.c_int * (4 * grid))()
        lib.shares(heads, head_groups, tiles, any_length, least, per_head, left, grid, out)

        def groups_in(unit):                                    # (places fill up from the front, and only the last left-over unit is not full)
            return 8 if not left or unit != left - 1 else (T % fg * per_frame * (8 // fg) - 1) % 8 + 1

        seen, xcd, idle = set(), {}, 0
        for b in range(grid):
            head, unit, lsub, sub = out[4 * b:4 * b + 4]
            assert head >= 0 and 0 <= unit < per_head and 0 <= sub < 1 << lsub
            if head >= heads or sub * (8 >> lsub) >= groups_in(unit):
                idle += 1
                continue
            assert lsub == (split0 if head_shares or head * per_head + unit < first else split1)
            assert (head, unit, sub) not in seen
            seen.add((head, unit, sub))
            xcd.setdefault((head, unit), []).append(b % 8)
        want = sum(-(-groups_in(u) // (8 >> (split0 if head_shares or h * per_head + u < first else split1)))
                   for h in range(heads) for u in range(per_head))
        assert len(seen) == want
        if head_shares:
            # shares of a unit stay together where a unit's are all there are: two heads meet where a head has an odd number
            assert idle == 0
            apart = sum(len(set(x)) > 1 for x in xcd.values())
            assert apart <= (0 if head_shares % (1 << split0) == 0 else len(xcd)) + 8
        else:
            assert all(len(set(x)) == 1 for x in xcd.values())
            assert idle <= (7 << max(split0, split1)) + (heads << max(split0, split1))


def test_full_rounds_are_not_shared(lib):
    """Lists of one length: where the last of up to four rounds is empty or more than three quarters full every unit is one workgroup.  A launch
    of less than a round leaves no CU a third share, and lists of any length in it are shared however short on average."""
    s = (ctypes.c_int * 5)()
    for tiles in (3, 26, 200):
        for any_length in (0, 1):
            for total in range(1, 1025):
                lib.share(total, 8, tiles, any_length, 0, s)
                first, split0, split1, grid, head_shares = s
                if not any_length and total > 256 and (total % 256 == 0 or total % 256 > 192) or 192 < total <= 256:
                    assert (first, split0, grid) == ((total + 7) // 8 * 8, 0, (total + 7) // 8 * 8)
                if 128 < total <= 192:
                    assert grid <= 512 and (split0 == 1) == ((any_length or tiles >= 24) and (total < 184 or total % 8 == 0))


def test_empty_shares_do_not_count(lib):
    """Twelve heads of 84 groups are 132 units, but 252 halves with a group: one round.  Likewise quarters and eighths."""
    s = (ctypes.c_int * 5)()
    for heads, head_groups, split in [(12, 84, 1), (12, 88, 0), (13, 84, 0), (9, 28, 3), (10, 28, 2), (18, 28, 2), (19, 28, 1),
                                      (128, 1, 3), (256, 1, 3), (257, 1, 1), (128, 2, 3), (256, 2, 2), (256, 4, 1), (128, 8, 1), (1000, 4, 1), (1000, 5, 0)]:
        lib.share(heads, head_groups, 8, 0, 0, s)
        assert s[1] == split and s[4] == (-(-head_groups // (8 >> split)) if split else 0), (heads, head_groups, list(s))


@pytest.mark.parametrize("any_length", [0, 1])
@pytest.mark.parametrize("sub", [1, 2])
def test_what_fits_also_fits_as_it_is_shared(lib, sub, any_length):
    """The lists of every problem that is accepted fit beside the ring at the least split and at any finer one, and an entry's key number has
    its bits; whole units are kept as long as they fit."""
    reached = set()
    for g in sorted({*range(1, 9000, 61), *range(6400, 7200, 7), 30000, 65535, 65536, 131072}):
        for k in sorted({1, 2, 7, 100, 800, 801, 1700, 2000, g // 10, g // 4, g // 2, g} & set(range(1, g + 1))):
            if not lib.fits(g, k, sub, any_length):
                continue
            least = lib.least(g, k, sub, any_length)
            reached.add(least)
            assert all(lib.aux(g, k, sub, any_length, split) <= 32 * 1024 for split in range(least, 4))
            assert least == 0 or lib.aux(g, k, sub, any_length, 0) > 32 * 1024
            assert g * sub < 2 ** 18
            if any_length or k == g:
                assert 4 * sub * g <= 32 * 1024
    assert reached == ({0} if sub == 2 and any_length else {0, 1})   # (two frames' lists of any length are as long as four's)
    # the sizes of the GPU tests at the limit
    if sub == 1:
        assert [lib.least(g, g, 1, 0) for g in (6440, 7000)] == [0, 1] and lib.least(7000, 1700, 1, any_length) == 1
        assert lib.fits(7000, 7000, 1, any_length) and not lib.fits(7200, 7200, 1, any_length)


def test_the_gpu_tests_reach_every_share(lib):
    """The launches of the GPU tests are shared out as those tests say, so a change of the rule cannot empty them unseen."""
    import test_gpu_attention_pairs as pairs
    import test_gpu_attention_shares as shares
    import test_gpu_attention_units as units
    launches = [(s[:5] + (keep,), s[5]) for s, keeps in pairs.SHARED.items() for keep in keeps]
    launches += [*shares.SHARED.items(), *units.SHARED.items()]
    s, reached = (ctypes.c_int * 5)(), set()
    for (T, fh, fw, pw, heads, keep), want in launches:
        g, sub = T * -(-fh // 8) * -(-fw // pw), pw // 8
        lib.share(heads, g * sub, min(keep, g) * sub, 0, lib.least(g, min(keep, g), sub, 0), s)
        alike = s[4] > 0 or s[0] >= heads * -(-g * sub // 8)
        assert ((s[1],) if alike else (s[1], s[2])) == want, (T, fh, fw, pw, heads, keep, list(s))
        reached.add((sub, want))
    assert reached >= {(sub, x) for sub in (1, 2) for x in ((3,), (2,), (1,), (0,), (1, 2))} | {(1, (0, 2)), (2, (0, 2)), (1, (0, 1))}
