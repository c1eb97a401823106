"""The tiles of a 1D launch (csrc/line_plan.h) on the host."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "line_plan.h"
using namespace lbm;
// 1 where a tile of R nodes per lane holds both ends of a domain it may take
static int both_ends(int nx, int K, int R)
{
    const int nout = line_out(K, R), hl = (K + R - 1) / R * R;
    if (nout <= 0 || !line_fits(nx, false, R)) return 0;
    for (int ob = 0; ob < nx; ob += nout)
        if (ob - hl <= 0 && ob - hl + 64 * R >= nx) return 1;
    return 0;
}
extern "C" int wrong_tiles()
{
    int n = 0;
    for (int nx = kLineWholeNodes + 1; nx <= 1400; ++nx)
        for (int K = 1; K <= kLineMaxK; ++K)
            for (const LineShape &s : kLineShapes) n += both_ends(nx, K, s.R);
    return n;
}
extern "C" int without_shape()
{
    int n = 0;
    for (int nx = kLineWholeNodes + 1; nx <= 1400; ++nx)
        for (int K = 1; K <= kLineMaxK; ++K)
            for (int f = 0; f < 4; ++f) n += line_shape(nx, false, f & 1, f & 2, K, nullptr) == 0;
    return n;
}
"""


def test_no_tile_holds_both_ends(tmp_path):
    """k_line applies the rule of one end per tile: whatever shape the cost prefers, a tile
    of a domain with non-periodic ends reaches one of them at most, and every domain that
    does not run in one workgroup has a shape at every depth."""
    src, lib = tmp_path / "plan.cpp", tmp_path / "plan.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_1401_0427_amd", "csrc"), str(src), "-o", str(lib)])
    L = ctypes.CDLL(str(lib))
    assert L.wrong_tiles() == 0 and L.without_shape() == 0
