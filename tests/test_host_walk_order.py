"""The order of the bf16 attention's walk is a counting sort by buckets of a float key, whose passes have to agree on an entry's bucket:
one more entry in a bucket than were counted overwrites another.  The key's arithmetic does differ with the contraction that a
compiler chooses where it is inlined, across bucket edges too, so the kernel may form it in one place only and every pass
reads it back.  The kernel's own functions, compiled for the CPU."""
import ctypes
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_14708_amd", "csrc")
SOURCE = """#include <math.h>
#include "ring_turns.h"
using namespace da::ring;
extern "C" void buckets(int cls, int n, int fused, float* key, int* bucket) {
  for (int p = 0; p < n; ++p) {
    const float inv = 1.0f / (float)n, u = (float)cls * 0.618034f;
    key[p] = fused ? ((float)p + fmaf((float)cls, 0.618034f, -(float)(int)u)) * inv : walk_key(cls, p, inv);
    bucket[p] = walk_bucket(key[p]);
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk_order")
    src, out = d / "walk.cpp", d / "libwalk.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(out)], check=True)
    return ctypes.CDLL(str(out))


def _run(lib, cls, n, fused=0):
    key, bucket = (ctypes.c_float * n)(), (ctypes.c_int * n)()
    lib.buckets(cls, n, fused, key, bucket)
    return list(key), list(bucket)


def test_key_is_formed_once(lib):
    # why it matters: the same key, formed twice, in two buckets
    assert any(_run(lib, cls, n)[1] != _run(lib, cls, n, 1)[1] for cls, n in [(15, 219), (30, 83), (30, 94), (42, 961), (42, 973)])
    source = open(os.path.join(CSRC, "k_attn_bf16_ring.hip")).read()
    assert len(re.findall(r"\b(?:walk_key|key_of)\(", source)) == 1


def test_keys_are_in_range_and_in_order(lib):
    for cls in (1, 2, 3, 7, 85, 128, 254, 255):
        for n in (1, 2, 3, 63, 64, 1000, 2047, 2048, 2049, 8192):
            key, bucket = _run(lib, cls, n)
            assert all(a < b for a, b in zip(key, key[1:]))
            assert all(a <= b for a, b in zip(bucket, bucket[1:])) and 0 <= bucket[0] and bucket[-1] < 2048
