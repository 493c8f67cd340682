"""The library's choices for the attention's work list (csrc/attn_plan.h, host arithmetic), for tests: compiled for the CPU on
first use."""
import ctypes as C
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """#include "attn_plan.h"
extern "C" int turns_of(int n, int fold) { return flexco::turns_of(n, fold); }
extern "C" int item_of_turn(int turn, int n, int fold) { return flexco::item_of_turn(turn, n, fold); }
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
    return _lib
