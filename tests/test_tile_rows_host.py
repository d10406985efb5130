"""Arithmetic of the distance launches, on the host.  The row ranges of the matrix-core distance workgroups (csrc/tile_rows.h), compiled for the host: every row a
workgroup loads lies inside its set, and the passes of the fused select take every row once."""
import ctypes
import os
import subprocess

import pytest

from paper_2405_19325_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "tile_rows.h"
extern "C" {
void rows_of(int fm, int64_t tile, int64_t rpt, int64_t sr, int64_t se, int64_t n, int64_t *out) {
    const knnlm::RowRange r = knnlm::mfma_rows(fm, tile, rpt, sr, se, n);
    out[0] = r.first;
    out[1] = r.end;
}
void sample_of(int rpt, int *out) {
    const knnlm::FusedSample s = knnlm::fused_sample(rpt);
    out[0] = s.rows;
    out[1] = s.every;
}
uint32_t load_row(uint32_t row, uint32_t nrows) { return knnlm::mfma_load_row(row, nrows); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_rows")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2405_19325_amd", "csrc"), str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.rows_of.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 5 + [ctypes.c_void_p]
    lib.load_row.argtypes = [ctypes.c_uint32] * 2
    lib.load_row.restype = ctypes.c_uint32
    return lib


def _ranges(lib, fm, rpt, sr, se, n):
    """(tile, first, end) of every workgroup of a pass that has rows."""
    out = (ctypes.c_int64 * 2)()
    tiles = (n + rpt - 1) // rpt
    for t in range(0, tiles, se if fm == 1 else 1):
        lib.rows_of(fm, t, rpt, sr, se, n, out)
        if out[0] < out[1]:
            yield t, out[0], out[1]


# rows per tile, sample rows, sampled every: whole tiles sampled (256 of 256) and pieces of them
@pytest.mark.parametrize("rpt,sr,se", [(256, 256, 64), (512, 256, 32), (1024, 256, 16), (4096, 512, 8)])
def test_rows_loaded_lie_in_the_set(lib, rpt, sr, se):
    period = rpt * se
    for n in (1, sr - 1, sr, sr + 1, rpt, rpt + 1, rpt + 120, period - 1, period + 1, period + sr, period + sr + 1,
              period + rpt + 8, 4 * period + rpt + 8, 65800, 70000):
        for fm in (0, 1, 2):
            for t, first, end in _ranges(lib, fm, rpt, sr, se, n):
                assert 0 <= first and end <= n
                rows = end - first
                for row in (0, rows - 1, rows, rows + 127, 4 * rpt):  # passes past the end and padding steps
                    assert first <= first + lib.load_row(row, rows) < end
        whole = [(a, b) for _, a, b in _ranges(lib, 0, rpt, sr, se, n)]
        parts = sorted((a, b) for fm in (1, 2) for _, a, b in _ranges(lib, fm, rpt, sr, se, n))
        for spans in (whole, parts):  # every row once
            assert spans[0][0] == 0 and spans[-1][1] == n
            assert all(x[1] == y[0] for x, y in zip(spans, spans[1:]))


def test_a_wholly_sampled_tile_leaves_no_rows(lib):
    out = (ctypes.c_int64 * 2)()
    lib.rows_of(2, 256, 256, 256, 64, 65800, out)
    assert out[0] >= out[1]


def test_sample_of_every_width(lib):
    """Every width's tiles have a sample that both matrix-core launchers take: whole passes (of at most 256 rows;
    the packed kernel asks for whole blocks of 16), inside the tile, about 1/64 of the keys."""
    tile_rows = _lib.load()["_ZN5knnlm14mfma_tile_rowsEl"]
    tile_rows.argtypes, tile_rows.restype = [ctypes.c_int64], ctypes.c_int
    out = (ctypes.c_int * 2)()
    for d in range(128, 65536 + 1, 128):
        rpt = tile_rows(d)
        lib.sample_of(rpt, out)
        rows, every = out
        assert rows % 256 == 0 and 256 <= rows <= rpt and every >= 1, (d, rpt, rows, every)
        assert 1 / 72 < rows / (rpt * every) < 1 / 48, (d, rpt, rows, every)


def test_shares_of_several_queries_fit_every_xcd_at_once():
    """The several-queries kernel runs one workgroup a CU, and the shares go to the 8 XCDs of 32 CUs in turn: those of
    all query groups are at most 32 an XCD, and no fewer than leave less than one more share's room."""
    shares = _lib.load()["_ZN5knnlm12multi_rangesEl"]
    shares.argtypes, shares.restype = [ctypes.c_int64], ctypes.c_int64
    for groups in range(1, 33):
        assert shares(groups) % 8 == 0
        assert 32 - groups < shares(groups) // 8 * groups <= 32
    assert shares(4096) == 8
