"""Which rows of the selection may read past their end: every one of them stays inside the array, and the next row would not.
The launch's own function, compiled for the CPU; row lengths around those that one register or one more per lane holds."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_14708_amd", "csrc")


@pytest.fixture(scope="module")
def read_on(tmp_path_factory):
    d = tmp_path_factory.mktemp("select_rows")
    src, lib = d / "select_rows.cpp", d / "libselect_rows.so"
    src.write_text('#include "select_rows.h"\n'
                   'extern "C" long long read_on(long long rows, long long g, long long columns, int slack) {\n'
                   '  return da::rows_that_read_on(rows, g, columns, slack != 0);\n}\n')
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    f = ctypes.CDLL(str(lib)).read_on
    f.argtypes, f.restype = [ctypes.c_longlong] * 3 + [ctypes.c_int], ctypes.c_longlong
    return f


@pytest.mark.parametrize("per_lane", [16, 32, 64])
def test_rows_that_read_on(read_on, per_lane):
    columns = 64 * per_lane
    lengths = {1, 2, 3, 5, 63, 64, 65, columns // 3, columns // 2 - 1, columns // 2, columns // 2 + 1, columns - 65, columns - 64,
               columns - 63, columns - 1, columns}
    for g in sorted(lengths):
        for rows in sorted({1, 2, 3, 7, g - 1, g, g + 1, 3 * g, columns // g, columns // g + 1, columns // g + 2} - {0}):
            head = read_on(rows, g, columns, 0)
            assert 0 <= head <= rows
            if head:
                assert (head - 1) * g + columns <= rows * g, (g, rows)     # the last of them ends inside the array
            if head < rows:
                assert head * g + columns > rows * g, (g, rows)            # the next one would not
            assert read_on(rows, g, columns, 1) == rows
