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
extern "C" int64_t bytes(int mean, int S, int bq, int64_t L, int64_t P, int64_t Q) {
  return (int64_t)(mean ? rc::mean_plan_bytes(S, (int)L, P, Q) : rc::plan_bytes({S, {256, bq}}, L, P, Q));
}
extern "C" int64_t least(int mean, int64_t L, int64_t P, int64_t Q, int T, int H) {
  return (int64_t)(mean ? rc::mean_floor_bytes((int)L, P, Q, T, H) : rc::match_floor_bytes(RC_SCORE_BLOCK, L, P, Q, T, H));
}
extern "C" int shares_in(int mean, int64_t L, int64_t P, int64_t Q, int T, int H, int64_t avail, int* columns) {
  if (mean) return rc::mean_split_count((int)L, P, Q, T, H, (size_t)avail);
  const rc::MatchPlan p = rc::match_plan(RC_SCORE_BLOCK, L, P, Q, T, H, (size_t)avail);
  *columns = p.ts.bq;
  return p.S;
}
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
    lib.bytes.argtypes = [i32, i32, i32, i64, i64, i64]
    lib.bytes.restype = i64
    lib.least.argtypes = [i32, i64, i64, i64, i32, i32]
    lib.least.restype = i64
    lib.shares_in.argtypes = [i32, i64, i64, i64, i32, i32, i64, ctypes.POINTER(i32)]
    return lib


def shares(mean, L, T, H, P, Q):
    """Shares per tile of a search by block score or layer mean with room for its plan, 1 = whole tiles."""
    return _lib().shares(int(mean), L, P, Q, T, H)


def alike(L, T, H, P, Q):
    """The number of shares of one length that the older rules give."""
    return _lib().alike(L, P, Q, T, H)


def need(mean, S, columns, L, P, Q):
    """Workspace of S shares per tile, or of whole tiles of that many columns (block score)."""
    return _lib().bytes(int(mean), S, columns, L, P, Q)


def least(mean, L, T, H, P, Q):
    """The least workspace that a call takes."""
    return _lib().least(int(mean), L, P, Q, T, H)


def shares_in(avail, mean, L, T, H, P, Q):
    """(shares per tile, columns of the block score's whole tiles) of a call with that workspace."""
    columns = ctypes.c_int(0)
    return _lib().shares_in(int(mean), L, P, Q, T, H, avail, ctypes.byref(columns)), columns.value
