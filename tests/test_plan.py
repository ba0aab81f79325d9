"""The host's choices of tiles and grids (csrc/plan.h), checked without a GPU through a small C++ shim."""
import ctypes
import os
import subprocess

import pytest

from test_gpu_gemm_f32 import CASES as F32_CASES
from test_gpu_gemm_loop import FULL_HEIGHT
from test_gpu_result_bits import MASKS, POSITIONS
from test_gpu_large_f32 import BEYOND
from test_gpu_row_tiles import CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
#include "plan.h"
using namespace spes;
extern "C" {
long set_grid_tiles(const int* m, const int* n, int sets, int bm, int bn) { return plan::set_grid_tiles(m, n, sets, bm, bn); }
int wgrad_small_tiles(long full, long small, int mean, int most) { return plan::wgrad_small_tiles(full, small, mean, most); }
int row_tile(long rows, int experts, int d, int f) { return plan::row_tile(rows, experts, d, f); }
int rowdot_parts(int n, int row_tile, int est) { return plan::rowdot_parts(n, row_tile, est); }
unsigned tiles_cut(unsigned full, unsigned half_height) { return plan::tiles_cut(full, half_height); }
int column_tail(int n) { return plan::column_tail(n); }
int few_tiles_narrow(int n, int est) { return plan::few_tiles_narrow(n, est); }
int f32_row_tile(long rows, int experts, int d, int f) { return plan::f32_row_tile(rows, experts, d, f); }
int f32_on_matrix_cores(long tokens, long rows, long d, long f) { return plan::f32_on_matrix_cores(tokens, rows, d, f); }
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
    p.row_tile.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    p.f32_row_tile.argtypes = p.row_tile.argtypes
    p.f32_on_matrix_cores.argtypes = [ctypes.c_long] * 4
    p.wgrad_small_tiles.argtypes = [ctypes.c_long, ctypes.c_long, ctypes.c_int, ctypes.c_int]
    return p


@pytest.mark.parametrize("d,f", [(512, 512), (8192, 64), (8, 65536), (72, 24), (1, 1), (1048576, 8)])
@pytest.mark.parametrize("bm", [16, 32, 64])
def test_sets_share_the_grid_of_the_largest(plan, d, f, bm):
    I = ctypes.c_int * 3
    got = plan.set_grid_tiles(I(d, f, f), I(f, d, d), 3, bm, 64)
    assert got == max(-(-d // bm) * -(-f // 64), -(-f // bm) * -(-d // 64))


@pytest.mark.parametrize("full,small,mean,most,want", [
    (1, 1, 1, 1, 1), (128, 512, 16384, 16384, 1), (162, 510, 13797, 27593, 1),     # one round of small tiles, at any contraction length
    (162, 513, 512, 512, 1), (162, 513, 513, 513, 0), (256, 1024, 513, 1026, 0), (256, 1024, 513, 1027, 1), (240, 960, 16384, 16384, 0),   # one of full ones
    (257, 1028, 16384, 16384, 1), (320, 1280, 16384, 16384, 1),                    # a second one that is nearly empty
    (321, 1284, 64, 64, 0), (1536, 6144, 64, 512, 0),
])
def test_weight_gradient_tiles(plan, full, small, mean, most, want):
    assert plan.wgrad_small_tiles(full, small, mean, most) == want


def test_row_tile_lines(plan):
    rt = lambda mean, M, d, f, more=0: plan.row_tile(mean * M + more, M, d, f)
    # long contractions: 48 and 96 rows a head, whatever the width
    for d, f in ((2048, 2048), (897, 512), (904, 3616), (768, 3080)):
        assert [rt(48, 16, d, f), rt(48, 16, d, f, 1), rt(96, 16, d, f), rt(96, 16, d, f, 1), rt(2000, 16, d, f)] == [64, 128, 128, 256, 256]
    # narrow layers with few tiles: 256 rows, 512 up to 640 columns
    assert [rt(256, 4, 896, 512), rt(256, 4, 896, 512, 1), rt(512, 4, 640, 512), rt(512, 4, 640, 512, 1)] == [64, 256, 64, 256]
    assert rt(100, 8, 136, 544) == 64 and rt(100, 8, 136, 552) == 256           # d_ff up to 4 d_model
    # many full tiles: 128-row ones (d_model times their number beyond 448 K), then full ones (beyond 688 K, but not for a
    # width with a column tail)
    assert [rt(100, 64, 768, f) for f in (1280, 1408, 2048, 2304)] == [64, 128, 128, 256]   # 570, 627, 912, 1026 tiles; 597, 917
    assert [rt(n, 64, 704, 2560) for n in (48, 64, 65, 96, 97, 224)] == [64, 64, 128, 128, 256, 256]
    assert [rt(n, 64, 640, 2560) for n in (64, 65, 97, 224, 512)] == [64, 128, 128, 128, 128]
    assert rt(192, 48, 384, 1536) == 64                                         # 720 tiles of a short contraction
    # two or three rounds of full tiles, the last one partly and at most 0.6 full
    rounds = lambda M, d, f, mean: ((mean * M // 256 + (M + 1) // 2) * -(-f // 128), rt(mean, M, d, f))
    assert rounds(16, 768, 2048, 320) == (448, 256)
    assert rounds(16, 768, 2048, 384) == (512, 256)                             # two rounds, both full
    assert rounds(16, 768, 2048, 400) == (528, 128)
    assert rounds(16, 768, 2048, 512) == (640, 128)
    assert rounds(16, 768, 2048, 688) == (816, 256)                             # more than three rounds
    assert rounds(8, 512, 2048, 900) == (512, 128)                              # full rounds of the shortest contractions


def test_gate_gradient_partials(plan):
    """Two per column tile; the layout reserves ceil(f/64) + 1 of them, which every height and width has to stay within."""
    for f in range(8, 6145, 8):
        for rows in (64, 128, 256):
            for est in (0, 1, 16, 100, 2000):
                n = plan.rowdot_parts(f, rows, est)
                halves = rows < 256 or plan.few_tiles_narrow(f, est)
                assert n == 2 * -(-f // (128 if halves else 256)) and n <= -(-f // 64) + 1
        tail = plan.column_tail(f)
        assert tail == (f % 256 if f > 256 and f % 256 <= 128 else 0)


@pytest.mark.parametrize("kw,rows,down", CASES)
def test_the_layer_cases_take_the_tiles_they_are_for(plan, kw, rows, down):
    """What the GPU cases say of themselves: row tile, and how the down projection's columns are cut."""
    M, d, f = kw["M"], kw["d"], kw["f"]
    R = kw["T"] * kw["k"]
    assert plan.row_tile(R, M, d, f) == rows
    if rows < 256:
        got = "short"
    elif plan.column_tail(d):
        got = plan.column_tail(d)
    else:
        got = "half" if plan.few_tiles_narrow(d, R // 256 + (M + 1) // 2) else "full"
    assert got == down


@pytest.mark.parametrize("kw,n_base,rows", POSITIONS)
def test_the_position_cases_take_the_tiles_they_are_for(plan, kw, n_base, rows):
    rule = plan.row_tile if kw.get("dtype") == "bf16" else plan.f32_row_tile
    assert rule(kw["T"] * kw["k"], kw["M"], kw["d"], kw["f"]) == rows


def test_tiles_cut(plan):
    for full, half, want in ((0, 9, 0), (1, 0, 1), (128, 0, 128), (129, 0, 0), (128, 1, 0), (100, 56, 100), (100, 57, 0), (256, 0, 0),
                             (257, 254, 1), (257, 255, 0), (384, 0, 128), (385, 0, 0)):
        assert plan.tiles_cut(full, half) == want, (full, half)


def _whole(plan, rows, cols, width):
    """Tiles of one expert's `rows` rows and of `cols` columns that are left at full height."""
    gx, full, half = -(-cols // width), rows // 256 + (rows % 256 > 128), int(0 < rows % 256 <= 128)
    return full * gx - plan.tiles_cut(full * gx, half * gx)


@pytest.mark.parametrize("T,d,f,whole,tails", FULL_HEIGHT)
def test_the_full_height_cases_have_whole_tiles(plan, T, d, f, whole, tails):
    assert plan.row_tile(T, 1, d, f) == 256
    got, got_tails = [_whole(plan, T, f, 128)], []
    for n in (f, d):
        tail = plan.column_tail(n)
        got.append(_whole(plan, T, n - tail, 128 if not tail and plan.few_tiles_narrow(n, T // 256 + 1) else 256))
        got_tails.append(_whole(plan, T, tail, 128) if tail else 0)
    assert (tuple(got), tuple(got_tails)) == (whole, tails)


def test_a_position_case_has_both_heights_in_one_launch(plan):
    both = [kw for kw, _, rows in POSITIONS if rows == 256 and kw["M"] == 1]
    assert both
    for kw in both:
        T, f = kw["T"], kw["f"]
        for width in (128, 256):          # gate + up, SwiGLU backward
            full = (T // 256 + (T % 256 > 128)) * -(-f // width)
            assert 0 < _whole(plan, T, f, width) < full and not plan.column_tail(f) and not plan.few_tiles_narrow(f, T // 256 + 1)


@pytest.mark.parametrize("kw,numbers", MASKS)
def test_the_mask_cases_lie_on_either_side_of_the_line(plan, kw, numbers):
    T, d, M, f, k = (kw[n] for n in "TdMfk")
    tiles = lambda n, side: 3 * n * -(-d // side) * -(-f // side)
    if "dtype" not in kw:        # fp32: 64 x 64 tiles from 256 of them on
        assert [tiles(n, 64) >= 256 for n in numbers] == [False, True]
        return
    assert [plan.wgrad_small_tiles(tiles(n, 256), tiles(n, 128), -(-T * k // M), T) for n in numbers] == [1, 0]


def test_f32_tiles(plan):
    # 64-row tiles once the GEMM with fewest columns has 512 blocks of them
    assert [plan.f32_row_tile(r, 8, 512, 512) for r in (59 * 64, 60 * 64)] == [32, 64]        # (60 + 4) * 8
    assert [plan.f32_row_tile(16384, 16, 8, f) for f in (8, 512)] == [32, 32]
    for kw, rows in F32_CASES:
        assert plan.f32_row_tile(kw["T"] * kw["k"], kw["M"], kw["d"], kw["f"]) == rows
    # 32-bit byte offsets: four bytes an element, less the last 32 bytes
    lim = (1 << 30) - 8
    assert plan.f32_on_matrix_cores(1, 1, lim - 8, 1) and not plan.f32_on_matrix_cores(1, 1, lim, 1)
    assert not plan.f32_on_matrix_cores(lim // 8 + 1, 1, 8, 8) and not plan.f32_on_matrix_cores(1, lim // 8 + 1, 8, 8)
    assert not plan.f32_on_matrix_cores(1, 1, 1 << 15, 1 << 15)


def test_grids_of_the_longest_fp32_layers(plan):
    """T * top_k up to 2^22 - 4224.  A launch has 2^32 work-items along x and 65535 blocks along y and z."""
    rows, one = 2**22 - 4224, ctypes.c_int * 3
    for M in (1, 4, 32, 33, 64):
        # router scores, 64 x 64 and 32 x 32 tiles, the 131000 row tiles of the latter along x
        for side in (64, 32):
            tiles = plan.set_grid_tiles(one(rows), one(M), 1, side, side)
            assert tiles == -(-rows // side) * -(-M // side) and tiles * 256 < 2**32
        # expert GEMMs: row tiles along y
        for d, f in ((8, 8), (128, 8), (8, 256), (248, 248)):
            assert rows // plan.f32_row_tile(rows, M, d, f) + M + 1 <= 65535


@pytest.mark.parametrize("kw,heights", BEYOND)
def test_the_cases_beyond_32_bit_offsets_take_the_tiles_they_are_for(plan, kw, heights):
    T, d, M, f, n = (kw[k] for k in ("T", "d", "M", "f", "n_trainable"))
    assert not plan.f32_on_matrix_cores(T, T, d, f)
    up = lambda a, b: -(-a // b)
    height = lambda blocks: 4 if blocks >= 512 else 2 if blocks >= 256 else 1        # of 64 x 64
    rows = T // 64 + M + 1
    assert (height(rows * up(f, 64)), height(rows * up(d, 64)), height(3 * n * up(d, 64) * up(f, 64))) == heights
