"""Row tiles and tile heights of a group, as the kernels compute them (gemm_kernel.h, compiled for the host): right for groups of
up to 2^31 - 1 rows, where a sum of rows and tile height, or of rows and tile count, leaves 32 bits."""
import ctypes
import os
import subprocess

import pytest

from paper_2508_16584_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = '''#include <hip/hip_runtime.h>
#include "gemm_kernel.h"
extern "C" int row_tiles(int rows, int BM) { return gg::row_tiles(rows, BM); }
extern "C" int even_height(int rows, int tiles) { return gg::even_height(rows, tiles); }
'''


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_tiles")
    (d / "host.hip").write_text(SOURCE)
    subprocess.run(["hipcc", *binding.HIPCC_FLAGS, "-I", os.path.join(ROOT, "paper_2508_16584_amd", "csrc"), "-o", str(d / "host.so"), str(d / "host.hip")],
                   check=True, capture_output=True)
    return ctypes.CDLL(str(d / "host.so"))


ROWS = [1, 31, 32, 33, 160, 161, 321, 8191, 2 ** 30 + 1, 2080000001, 2130706433, 2134221211, 2 ** 31 - 257, 2 ** 31 - 128, 2 ** 31 - 2, 2 ** 31 - 1]


@pytest.mark.parametrize("BM", [16, 32, 64, 96, 128, 160, 192, 224, 256])
def test_tiles_of_a_group(host, BM):
    for rows in [0] + ROWS:
        assert host.row_tiles(rows, BM) == -(-rows // BM), (rows, BM)


@pytest.mark.parametrize("bm", [32, 64, 96, 128, 160])
def test_height_of_a_groups_tiles(host, bm):
    for rows in ROWS:
        tiles = -(-rows // bm)
        h = host.even_height(rows, tiles)
        assert h == -(-(-(-rows // tiles)) // 32) * 32, (rows, bm)
        assert h <= bm and h * tiles >= rows and (tiles - 1) * h < rows
