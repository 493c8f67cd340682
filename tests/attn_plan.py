"""The library's choices for the attention's work list (csrc/attn_plan.h, host arithmetic), for tests: compiled for the CPU on
first use."""
import ctypes as C
import os
import subprocess
import tempfile

import paper_2402_18789_amd.binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """#include "attn_plan.h"
extern "C" int turns_of(int n, int fold) { return flexco::turns_of(n, fold); }
extern "C" int item_of_turn(int turn, int n, int fold) { return flexco::item_of_turn(turn, n, fold); }
extern "C" void plan(const flexco_maps* m, int nkv, int* out) {
  const flexco::AttnPlan p = flexco::plan_attention(*m, nkv);
  out[0] = p.alone; out[1] = p.fold; out[2] = p.lag;
}
"""
_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as tmp:
            so = os.path.join(tmp, "plan.so")
            subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-shared", "-fPIC", "-x", "c++", "-I" + os.path.join(ROOT, "include"),
                            "-I" + os.path.join(ROOT, "paper_2402_18789_amd", "csrc"), "-", "-o", so], input=SOURCE, text=True, check=True)
            _lib = C.CDLL(so)
        _lib.plan.argtypes, _lib.plan.restype = [C.POINTER(B.Maps), C.c_int, C.POINTER(C.c_int)], None
    return _lib


def attention_plan(maps, n_kv_heads):
    """-> (key splits the four-wavefront kernel takes as one, 0: the one-wavefront kernel, the exponentials' reference may lag)"""
    out = (C.c_int * 3)()
    lib().plan(C.byref(maps), n_kv_heads, out)
    return out[1] if out[0] else 0, bool(out[2])
