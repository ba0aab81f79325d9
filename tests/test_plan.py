"""The host's choices of tiles and grids (csrc/plan.h), checked without a GPU through a small C++ shim."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
#include "plan.h"
using namespace spes;
extern "C" {
long set_grid_tiles(const int* m, const int* n, int sets, int bm, int bn) { return plan::set_grid_tiles(m, n, sets, bm, bn); }
int wgrad_small_tiles(long full, int mean, int most) { return plan::wgrad_small_tiles(full, mean, most); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2602_11543_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    p = ctypes.CDLL(str(lib))
    p.set_grid_tiles.restype = ctypes.c_long
    p.wgrad_small_tiles.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int]
    return p


@pytest.mark.parametrize("d,f", [(512, 512), (8192, 64), (8, 65536), (72, 24), (1, 1), (1048576, 8)])
@pytest.mark.parametrize("bm", [16, 32, 64])
def test_sets_share_the_grid_of_the_largest(plan, d, f, bm):
    I = ctypes.c_int * 3
    got = plan.set_grid_tiles(I(d, f, f), I(f, d, d), 3, bm, 64)
    assert got == max(-(-d // bm) * -(-f // 64), -(-f // bm) * -(-d // 64))


@pytest.mark.parametrize("full,mean,most,small", [
    (1, 1, 1, 1), (128, 16384, 16384, 1),                    # CUs without a full tile, at any contraction length
    (129, 512, 512, 1), (129, 513, 513, 0), (256, 513, 1026, 0), (256, 513, 1027, 1), (240, 16384, 16384, 0),   # one round of them
    (257, 16384, 16384, 1), (320, 16384, 16384, 1),          # a second one that is nearly empty
    (321, 64, 64, 0), (1536, 64, 512, 0),
])
def test_weight_gradient_tiles(plan, full, mean, most, small):
    assert plan.wgrad_small_tiles(full, mean, most) == small
