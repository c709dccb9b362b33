"""The library's dispatch rules (csrc/rules.h, csrc/raster.h), compiled for the
host, so that a test can state which path its shapes take."""
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_36070_amd", "csrc")

SRC = """
#include <algorithm>
#include "rules.h"
using std::min;
#define DEV static inline
#include "raster.h"
extern "C" {
int t_quartered(long n) {
    int q, most = 0;
    for (int b = 0; b < deal_grid(n, RASTER_CHUNK); ++b) most |= deal_tile_split(b, (int)n, q) >= 0 ? 1 << (q >= 0) : 0;
    return most;
}
int t_dense_parts(long T, long d, long E, long k, long f, long fs) { return dense_parts(T, d, E, k, f, fs); }
int t_skinny_tiles(long T, long k, long E, long f, long fs) { return skinny_tiles(T, k, E, f, fs); }
int t_skinny_kslices(long T, long k, long E, long d, long f, long fs) {
    return skinny_kslices(T, k, E, d, f, fs, skinny_tiles(T, k, E, f, fs)); }
int t_route_direct(long T, long d, long E, long k) { return route_direct(T, d, E, k); }
int t_mx_keep_l2(long R, long E, long K, long N) { return mx_keep_l2(R, E, K, N); }
int t_deep_stages(long K, long rows, long groups) { return deep_stages(K, rows, groups); }
}
"""

HAVE_CXX = shutil.which("g++") is not None


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as tmp:
        src, out = os.path.join(tmp, "rules.cpp"), os.path.join(tmp, "rules.so")
        with open(src, "w") as fh:
            fh.write(SRC)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", out, src], check=True)
        return ctypes.CDLL(out)


def _call(fn, *args):
    return getattr(_lib(), fn)(*(ctypes.c_long(a) for a in args))


def small_tiles(w):
    """A forward that keeps no activations: 16-row tiles per workgroup of the streaming kernels, 0 the tile GEMMs."""
    return _call("t_skinny_tiles", w.T, w.k, w.E, w.f, w.f_s)


def kslices(w):
    """Workgroups of a small batch that share an up/gate tile's K."""
    return _call("t_skinny_kslices", w.T, w.k, w.E, w.d, w.f, w.f_s)


def dense_parts(w):
    """Dense routing: the experts' down products go to fp32 and are added, instead of one folded product."""
    return bool(_call("t_dense_parts", w.T, w.d, w.E, w.k, w.f, w.f_s))


def route_direct(T, d, E, k):
    """The router runs as one launch on W_r as it lies."""
    return bool(_call("t_route_direct", T, d, E, k))


def deep_stages(K, rows, groups):
    """A row product in a launch of its own holds three LDS stages of B instead of two."""
    return bool(_call("t_deep_stages", K, rows, groups))


def mx_keep_l2(R, E, K, N):
    """The MXFP8 up/gate product stores its kept pre-activations through the L2."""
    return bool(_call("t_mx_keep_l2", R, E, K, N))


def tile_shapes(tiles, K, rows, groups):
    """The tile shapes that a row product of `tiles` tiles runs in a launch of its own."""
    got = _call("t_quartered", tiles)
    whole = "three" if deep_stages(K, rows, groups) else "two"
    return ({whole} if got & 1 else set()) | ({"quarters"} if got & 2 else set())
