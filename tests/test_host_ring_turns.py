"""How the bf16 attention deals a list's entries to the waves that share it: evenly, the first to the first wave (the others
look at it), and of blocks of 128 slots, which are two entries in a row, as many first halves as second ones to every wave.
The kernel's own function, compiled for the CPU."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_14708_amd", "csrc")


@pytest.fixture(scope="module")
def wave_of_turn(tmp_path_factory):
    d = tmp_path_factory.mktemp("ring_turns")
    src, lib = d / "ring_turns.cpp", d / "libring_turns.so"
    src.write_text('#include "ring_turns.h"\n'
                   'extern "C" int wave_of_turn(int turn, int sub, int parts) { return da::ring::wave_of_turn(turn, sub, parts); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    f = ctypes.CDLL(str(lib)).wave_of_turn
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_int
    return f


@pytest.mark.parametrize("sub", [1, 2])
@pytest.mark.parametrize("parts", [2, 4, 8])
def test_entries_are_dealt_evenly(wave_of_turn, sub, parts):
    assert wave_of_turn(0, sub, parts) == 0
    for start in range(0, 64 * parts, sub * parts):          # any stretch of as many blocks as waves
        turns = range(start, start + sub * parts)
        for half in range(sub):
            waves = [wave_of_turn(t, sub, parts) for t in turns if t % sub == half]
            counts = [waves.count(w) for w in range(parts)]
            assert max(counts) <= 2 and sum(counts) == parts
        waves = [wave_of_turn(t, sub, parts) for t in turns]
        assert [waves.count(w) for w in range(parts)] == [sub] * parts
    for half in range(sub):                                  # and over a long walk, every half
        waves = [wave_of_turn(t, sub, parts) for t in range(half, 64 * parts, sub)]
        assert [waves.count(w) for w in range(parts)] == [64 // sub] * parts
