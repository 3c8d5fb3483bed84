"""Index arithmetic of the Helmholtz column tiles, run on the host: the header's
own functions are compiled for the CPU and every address a wavefront forms is
compared with the extent of what it reads."""
import ctypes
import os
import subprocess

import pytest

from paper_2511_21535_amd import build as B

SRC = """
#include "helm_columns.h"
// The largest and the smallest right-hand side that the lanes of any wavefront of
// 16 columns address in a tile of `cols` columns from column c0 of an instance
// with cnt columns left.
extern "C" void rhs_range(int32_t nrhs, int64_t c0, int32_t cnt, int32_t cols, int32_t *lo, int32_t *hi) {
    p2p::ColTile t{};
    t.c0 = c0;
    t.cnt = cnt;
    *lo = nrhs;
    *hi = -1;
    for (int w = 0; w < cols / 16; ++w) {
        const int32_t rhs0 = p2p::uni_first_rhs(p2p::col_lane<false>(t, nrhs, 16 * w).rhs);
        for (int col = 0; col < 16; ++col) {
            const int32_t r = rhs0 + col;
            *lo = r < *lo ? r : *lo;
            *hi = r > *hi ? r : *hi;
            // a column of the tile is read at its own right-hand side
            if (16 * w + col < cnt && r != p2p::col_lane<false>(t, nrhs, 16 * w + col).rhs) *hi = INT32_MAX;
        }
    }
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    src, out = d / "host.hip", d / "libhost.so"
    src.write_text(SRC)
    subprocess.run([B.HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wno-unused-function",
                    "-I", B.INC, "-I", B.CSRC, str(src), "-o", str(out)], check=True)
    return ctypes.CDLL(os.fspath(out))


@pytest.mark.parametrize("cols", [64, 128])
@pytest.mark.parametrize("nrhs", [16, 48, 64, 272, 560, 1 << 20])
def test_wavefronts_past_the_last_column_stay_inside_the_box(host, nrhs, cols):
    """side 12 and 272 right-hand sides: the last tile of 128 columns holds 48, five of its wavefronts none."""
    lo, hi = ctypes.c_int32(), ctypes.c_int32()
    for boxes in (1, 2, 27):
        total = boxes * nrhs
        for c0 in {0, (total - 1) // cols * cols, (total // 2) // cols * cols}:
            cnt = min(cols, total - c0)
            host.rhs_range(nrhs, ctypes.c_int64(c0), cnt, cols, ctypes.byref(lo), ctypes.byref(hi))
            assert 0 <= lo.value and hi.value < nrhs, (boxes, c0, cnt)
