"""The grid of the one-tile-per-workgroup kernels past 2^31 threads, run on the
host: the functions that the launches and kernels use (csrc/tc_grid.h),
compiled with the host compiler, at sizes that need no buffers.

A grid that goes on along y is made of whole rows, so its last row can hold
almost 2^31 / threads workgroups past the last tile; none of them may find
anything to do, however far beyond the items its tile lies.
"""

import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1801_03855_amd", "csrc")

SOURCE = r"""
#include "tc_grid.h"
extern "C" void grid(int64_t tiles, int threads, int64_t* x, int64_t* y) {
    const tc::GridXY g = tc::grid_of(tiles, threads);
    *x = g.x;
    *y = g.y;
}
extern "C" int items(int64_t total, int64_t tile, int per) { return tc::tile_items(total, tile, per); }
"""


@pytest.fixture(scope="module")
def native(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "grid.cpp").write_text(SOURCE)
    out = str(d / "libgrid.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, "-o", out,
                    str(d / "grid.cpp")], check=True)
    L = ctypes.CDLL(out)
    L.grid.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int64)]
    L.grid.restype = None
    L.items.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    L.items.restype = ctypes.c_int

    class Native:
        items = staticmethod(L.items)

        @staticmethod
        def grid(tiles, threads):
            x, y = ctypes.c_int64(), ctypes.c_int64()
            L.grid(tiles, threads, ctypes.byref(x), ctypes.byref(y))
            return x.value, y.value

    return Native


# Threads of a workgroup: one to 16 waves, and the half waves of the tiles of
# 16 and 32 lanes.
THREADS = [16, 32, 48, 64, 96, 128, 192, 256, 288, 416, 512, 768, 1024]
# Items of a full tile: 16 to 128 lanes of one slot or two, and the waves' 256
# and 512 elements.
PER = [16, 32, 64, 128, 256, 512]


@pytest.mark.parametrize("per", PER)
@pytest.mark.parametrize("threads", THREADS)
def test_rows_past_the_last_tile_are_empty(native, threads, per):
    rng = random.Random(threads * 1000 + per)
    most = 2 ** 31 // threads
    for rows in (1, 2, 3, 5):
        for tiles in (1, 2, most - 1, rows * most, rows * most + 1, rows * most + rng.randrange(2, most)):
            for total in (tiles * per, tiles * per - rng.randrange(per), (tiles - 1) * per + 1):
                x, y = native.grid(tiles, threads)
                assert x * threads <= 2 ** 31 and y < 65536
                assert x * y >= tiles and x * (y - 1) < tiles
                what = f"threads={threads} per={per} total={total}"
                # the last tile has the rest, those before it are full
                last = total - (tiles - 1) * per
                assert native.items(total, tiles - 1, per) == last, what
                for t in {0, tiles // 2, tiles - 2} - {-1, tiles - 1}:
                    assert native.items(total, t, per) == per, f"{what} tile={t}"
                # past it: nothing, at the near end, the far end and between
                spare = range(tiles, x * y)
                past = [spare[0], spare[-1], *(rng.choice(spare) for _ in range(20))] if spare else []
                for t in past:
                    assert native.items(total, t, per) == 0, f"{what} tile={t}"


def test_no_items(native):
    assert native.grid(0, 256) == (1, 1)
    assert native.items(0, 0, 64) == 0
