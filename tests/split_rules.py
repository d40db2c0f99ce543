"""The backward's work-split rules (csrc/flarepp_split.hpp), compiled on their
own with the host compiler, so that tests can ask for a shape's split."""

from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_11519_amd", "csrc")
SRC = """
#include "flarepp_split.hpp"
using namespace flarepp;
extern "C" {
void bwd(int64_t BH, int64_t Nl, int D, int Mp, int dec, int eb, int64_t* o) {
  const BwdSplit s = bwd_split(BH, Nl, D, Mp, dec, eb, 160 * 1024);
  o[0] = s.waves; o[1] = s.R; o[2] = s.tpw; o[3] = s.nsb;
}
double rounds_time(int64_t BH, int64_t tiles, int64_t waves, int64_t R) { return bwd_rounds_time(BH, tiles, waves, R); }
void rs(int64_t B, int64_t H, int64_t N, int D, int Mp, int64_t* o) {
  const RsSplit s = rs_split(B, H, N, D, Mp);
  o[0] = s.rb; o[1] = 1 << s.rw_log2; o[2] = s.nbw; o[3] = s.R; o[4] = s.steps; o[5] = rs_positions(D, 1 << s.rw_log2);
}
int wgrad(int64_t T, int nprob, int64_t* chunk) { return wgrad_chunks(T, nprob, chunk); }
}
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "split.cpp"), os.path.join(d, "split.so")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", so, src], check=True)
        lib = ctypes.CDLL(so)
    i64, i32, p = ctypes.c_int64, ctypes.c_int, ctypes.POINTER(ctypes.c_int64)
    lib.bwd.argtypes, lib.bwd.restype = [i64, i64, i32, i32, i32, i32, p], None
    lib.rounds_time.argtypes, lib.rounds_time.restype = [i64] * 4, ctypes.c_double
    lib.rs.argtypes, lib.rs.restype = [i64, i64, i64, i32, i32, p], None
    lib.wgrad.argtypes, lib.wgrad.restype = [i64, i32, p], i32
    return lib


def bwd_split(BH, N, D, Mp, dec, elem_bytes):
    o = (ctypes.c_int64 * 4)()
    _lib().bwd(BH, N, D, Mp, int(dec), elem_bytes, o)
    return dict(zip(("waves", "R", "tpw", "nsb"), o))


def rounds_time(BH, tiles, waves, R):
    return _lib().rounds_time(BH, tiles, waves, R)


def rs_split(B, H, N, D, M):
    o = (ctypes.c_int64 * 6)()
    _lib().rs(B, H, N, D, (M + 31) // 32 * 32, o)
    return dict(zip(("rb", "rw", "nbw", "R", "steps", "positions"), o))


def wgrad_chunks(T, nprob=7):
    """(chunks, tokens per chunk)"""
    c = ctypes.c_int64()
    n = _lib().wgrad(T, nprob, ctypes.byref(c))
    return n, c.value
