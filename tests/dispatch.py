"""The rules of csrc/dispatch.hpp, compiled for the host: which form of a kernel
a launch of the given sizes takes."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_20437_amd", "csrc")

SHIM = """
#include "dispatch.hpp"
using namespace galore;
extern "C" {
int narrow_sign_columns_(int rows, int r, int vec, long b) { return narrow_sign_columns(rows, r, vec, b); }
int narrow_align_columns_(int r, long b) { return narrow_align_columns(r, b); }
int f32_tile_(int M, int N, int kcontig, int adds, long b) { return f32_tile(M, N, kcontig, adds, b); }
int f32_tril_tile_(int M, int N, int K, long b) { return f32_tril_tile(M, N, K, b); }
int padded_projection_(int s, int l, int r, long b) { return padded_projection(s, l, r, b); }
int three_plane_half_(int M, int N, long b) { return three_plane_half(M, N, b); }
int six_plane_small_(int M, int N, int K, long b) { return six_plane_small(M, N, K, b); }
int step_pairs_(int k, int block) { return step_pairs(k, block); }
int wide_pairs_(int k, int pairs, long b, long in_flight) { return wide_pairs(k, pairs, b, in_flight); }
}
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, out = os.path.join(d, "shim.cpp"), os.path.join(d, "libdispatch.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", out], check=True)
        return ctypes.CDLL(out)


def rule(name, *args):
    return getattr(_lib(), name + "_")(*[ctypes.c_long(a) for a in args])
