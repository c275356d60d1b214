"""What the library launches for a call, without a GPU: a few functions of the HIP runtime, replaced by ones that note the launch and
return success, loaded ahead of the library in a process of its own.  Pointers are numbers that nobody follows."""
from __future__ import annotations

import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = r"""
#include <stdio.h>
#include <string.h>
#include <map>
#include <string>
#include <vector>
struct dim { unsigned x, y, z; };
static std::map<const void*, std::string> names;
static std::string log_;
static dim g_, b_;
static size_t s_;
static void* q_;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int __hipPushCallConfiguration(dim g, dim b, size_t s, void* q) { g_ = g; b_ = b; s_ = s; q_ = q; return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* s, void** q) { *g = g_; *b = b_; *s = s_; *q = q_; return 0; }
int hipLaunchKernel(const void* f, dim g, dim b, void**, size_t s, void*) {
  char t[512];
  snprintf(t, sizeof t, "%s %u %u %u %u %u %u %zu\n", names[f].c_str(), g.x, g.y, g.z, b.x, b.y, b.z, s);
  log_ += t;
  return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x100000; return 0; }
int hipMemcpyFromSymbol(void* p, const void*, size_t n, size_t, int) { memset(p, 0, n); return 0; }
const char* launches() { static std::string out; out.swap(log_); log_.clear(); return out.c_str(); }
}
"""
CHILD = r"""
import ctypes, json, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stub.launches.restype = ctypes.c_char_p
sys.path.insert(0, sys.argv[2])
from paper_2505_14708_amd import binding as da
L = ctypes.CDLL(da.LIB_PATH)
for line in sys.stdin:
    call = json.loads(line)
    p = da.da_problem(**call["problem"])
    P = ctypes.c_void_p
    q, k, v, o, idx, ws = (P((i + 1) << 20) for i in range(6))
    big = ctypes.c_size_t(2 ** 63)
    if call["entry"] == "da_forward":
        st = L.da_forward(ctypes.byref(p), q, k, v, o, idx, ws, big, None)
    elif call["entry"] == "da_forward_global":
        st = L.da_forward_global(ctypes.byref(p), q, k, v, o, None, None, ws, big, None)
    elif call["entry"] == "da_forward_blocks":
        st = L.da_forward_ex(ctypes.byref(p), None, None, 1, q, k, v, o, idx, ws, big, None)
    else:
        raise ValueError(call["entry"])
    got = [l.split() for l in stub.launches().decode().splitlines()]
    print(json.dumps([st, [[l[0], [int(x) for x in l[1:4]], [int(x) for x in l[4:7]], int(l[7])] for l in got]]), flush=True)
"""


def record(tmp_dir, calls):
    """[(status, [(kernel, grid, workgroup, dynamic LDS)])] for `calls`: (entry, fields of da_problem)."""
    src, out = os.path.join(tmp_dir, "stub.cpp"), os.path.join(tmp_dir, "libhipstub.so")
    open(src, "w").write(STUB)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", src, "-o", out], check=True)
    lines = "".join(json.dumps({"entry": e, "problem": f}) + "\n" for e, f in calls)
    r = subprocess.run([sys.executable, "-c", CHILD, out, ROOT], input=lines, capture_output=True, text=True, check=True, timeout=120)
    return [json.loads(l) for l in r.stdout.splitlines()]
