"""The GEMM rasters place every tile exactly once (CPU: raster.h compiled for the
host and walked over grids around its chunk and group sizes)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_36070_amd", "csrc")

PROG = r"""
#include <algorithm>
#include <cstdio>
#include <set>
#include <utility>
using std::min;
#define DEV static inline
#include "raster.h"
template <class F> static int walk(F f, long grid, int tm, int ntn) {
    std::set<std::pair<int, int>> seen;
    for (long b = 0; b < grid; ++b) {
        int mt = -1, nt = -1;
        if (!f((int)b, tm, ntn, mt, nt)) continue;
        if (mt < 0 || mt >= tm || nt < 0 || nt >= ntn || !seen.insert({mt, nt}).second) return 1;
    }
    return seen.size() == (size_t)tm * ntn ? 0 : 2;
}
int main() {
    int bad = 0;
    for (int tm : {1, 2, 3, 4, 5, 7, 8, 17, 31, 33, 41, 64, 130})
        for (int ntn : {1, 2, 3, 5, 8, 12, 16, 28, 56}) {
            if (walk(map_tile, raster_grid(tm, ntn), tm, ntn)) { std::printf("chunks %d %d\n", tm, ntn); ++bad; }
            if (walk(map_tile_groups, raster_grid_groups(tm, ntn), tm, ntn)) { std::printf("groups %d %d\n", tm, ntn); ++bad; }
            // a launch sized for more m-tiles than there are places the same tiles
            if (walk(map_tile, raster_grid(tm + 37, ntn), tm, ntn)) { std::printf("larger grid %d %d\n", tm, ntn); ++bad; }
            // no XCD runs more than its share of whole rounds
            int n[8] = {0}, mt, nt;
            for (long b = 0; b < raster_grid(tm, ntn); ++b) n[b % 8] += map_tile((int)b, tm, ntn, mt, nt);
            if (*std::max_element(n, n + 8) > (tm * ntn + 255) / 256 * 32) { std::printf("uneven %d %d\n", tm, ntn); ++bad; }
            // with a short last round split: every tile once, whole or in its four quarters
            std::set<std::pair<int, int>> seen;
            long whole = 0;
            for (long b = 0; b < raster_grid(tm, ntn); ++b) {
                int q;
                const int t = deal_tile_split((int)b, tm * ntn, q);
                if (t < 0) continue;
                if (t >= tm * ntn || q > 3 || !seen.insert({t, q}).second) { std::printf("split %d %d\n", tm, ntn); ++bad; }
                whole += q < 0 ? 4 : 1;
            }
            if (whole != 4L * tm * ntn) { std::printf("split misses %d %d\n", tm, ntn); ++bad; }
            for (int groups : {1, 2, 3, 8, 32}) {
                auto wg = [&](int b, int cmn, int ntn2, int &cm, int &nt2) {
                    return map_tile_wgrad(b, groups, cmn / groups, ntn2, cm, nt2);
                };
                if (walk(wg, wgrad_grid(groups, tm, ntn), groups * tm, ntn)) { std::printf("wgrad %d %d %d\n", groups, tm, ntn); ++bad; }
                int w[8] = {0};
                for (long b = 0; b < wgrad_grid(groups, tm, ntn); ++b) w[b % 8] += wg((int)b, groups * tm, ntn, mt, nt);
                if (*std::max_element(w, w + 8) > (groups * tm * ntn + 127) / 128 * 16) { std::printf("wgrad uneven %d %d %d\n", groups, tm, ntn); ++bad; }
            }
        }
    return bad;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="needs a host compiler")
def test_every_tile_placed_once(tmp_path):
    (tmp_path / "r.cpp").write_text(PROG)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(tmp_path / "r"), str(tmp_path / "r.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "r")], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
