"""Plans of the tile searches where there is no GPU (test helper): rc_match_plan.hpp is plain C++."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "rc_match_plan.hpp"
extern "C" int shares(int mean, int64_t L, int64_t P, int64_t Q, int T, int H) { return rc::block_split_count(mean != 0, L, P, Q, T, H); }
extern "C" int alike(int64_t L, int64_t P, int64_t Q, int T, int H) { return rc::alike_split_count(RC_SCORE_BLOCK, L, P, Q, T, H); }
"""


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, out = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(PROGRAM)
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                               "-I", os.path.join(ROOT, "paper_2507_21433_amd", "csrc"), "-o", out, src])
        lib = ctypes.CDLL(out)
    i64, i32 = ctypes.c_int64, ctypes.c_int
    lib.shares.argtypes = [i32, i64, i64, i64, i32, i32]
    lib.alike.argtypes = [i64, i64, i64, i32, i32]
    return lib


def shares(mean, L, T, H, P, Q):
    """Shares per tile of a search by block score or layer mean with room for its plan, 1 = whole tiles."""
    return _lib().shares(int(mean), L, P, Q, T, H)


def alike(L, T, H, P, Q):
    """The number of shares of one length that the older rules give."""
    return _lib().alike(L, P, Q, T, H)
