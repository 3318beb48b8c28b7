"""Search tilings and the scratch limit of the allocation-free query: the
host arithmetic of csrc/inpaint_dev.h, compiled here for the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1403_4238_amd", "csrc")
AUTO, SIMT, MFMA = 0, 1, 2
LIMIT = 32768   # partial minima the static scratch holds

SHIM = r"""
#include "inpaint_dev.h"
using namespace inpaint;
extern "C" void route(int path, int mfma, int tile_rows, int r, const int *k, int64_t *out) {
    const StaticRoute s = static_route(path, mfma != 0, tile_rows, r, k[0], k[1], k[2], k[3]);
    out[0] = s.ok;
    out[1] = s.mfma;
    out[2] = s.tile_rows;
    out[3] = s.t.count();
    out[4] = (kStaticScratchBytes - kStaticPartialsOff) / 8;
}
"""


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs g++ and the HIP headers")
    d = tmp_path_factory.mktemp("tiling")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + CSRC, "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))

    def call(path, mfma, tile_rows, r, rect):
        out = (ctypes.c_int64 * 5)()
        lib.route(path, int(mfma), tile_rows, r, (ctypes.c_int * 4)(*rect), out)
        return bool(out[0]), bool(out[1]), out[2], out[3], out[4]

    return call


def _simt_tiles(rect, rows):
    x0, y0, x1, y1 = rect
    return -(-(x1 - x0) // 64) * -(-(y1 - y0) // (4 * rows))


def _mfma_tiles(rect, r):
    x0, y0, x1, y1 = rect
    first = x0 - ((x0 - r + 8) & 7)
    return -(-(x1 - first) // 64) * -(-(y1 - y0) // 64)


def test_auto_query_one_column_past_the_scratch(route):
    # 32768 SIMT tiles, accepted; the aligned MFMA tiling needs 32769
    rect = (11, 4, 2097163, 5)
    assert _simt_tiles(rect, 8) == LIMIT and _mfma_tiles(rect, 4) == LIMIT + 1
    assert route(AUTO, True, 8, 4, rect) == (True, False, 8, LIMIT, LIMIT)


# Widths around the limit from every residue of the first column, one tile row
# and several: what is launched fits the scratch, and what is accepted is what
# the path's own tiling accepts.
@pytest.mark.parametrize("r", range(1, 9))
@pytest.mark.parametrize("rows", [1, 16, 32, 33, 64, 65, 130])
def test_static_route_fits_the_scratch(route, r, rows):
    for res in range(9):
        for tiles in (1, 2, LIMIT // 5, LIMIT // 3, LIMIT // 2, LIMIT - 1, LIMIT, LIMIT + 1):
            for extra in (-7, -1, 0, 1, 63):
                rect = (r + res, r, r + res + max(64 * tiles + extra, 1), r + rows)
                for path, mfma, tile_rows in ((AUTO, True, 8), (AUTO, False, 8), (SIMT, False, 4), (SIMT, False, 16),
                                              (MFMA, True, 16)):
                    ok, on_mfma, used, n, room = route(path, mfma, tile_rows, r, rect)
                    if path == MFMA and r <= 6:
                        want = _mfma_tiles(rect, r) <= LIMIT
                    else:
                        want = _simt_tiles(rect, 8 if path == AUTO else tile_rows) <= LIMIT
                    assert ok == want, (path, rect)
                    if ok:
                        assert n <= room and n == (_mfma_tiles(rect, r) if on_mfma else _simt_tiles(rect, used))
                        assert on_mfma == (mfma and _mfma_tiles(rect, r) <= LIMIT), (path, rect)
