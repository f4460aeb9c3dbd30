"""The block kernel's scale staging (csrc/scale_stage.h), walked on the CPU for every block shape of its tables: each
dword in the LDS has one writer and holds the scales of the row and the steps that the operand reads expect there,
for row-major and for tile-major weights."""
import ctypes
import glob
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_13565_amd", "csrc")

WALK = r"""
#include "scale_stage.h"
using namespace mxfp4::wide;
extern "C" int walk(int tiled, int bn, int wk, int row0, int n, int k, int pair, int* lds, int* from)
{
    const int nblk = k / 32, steps = (k + 127) / 128, n_tiles = (n + 15) / 16, n_items = (steps + 3) / 4;
    int count = 0;
    for (int i = 0; i < scale_rounds(bn, wk); ++i)
        for (int tid = 0; tid < kThreads; ++tid) {
            if (!scale_owned(bn, wk, tid, i))
                continue;
            const int step = pair * wk * 2 + scale_step(wk, tid, i);
            lds[count] = scale_lds(wk, tid, i);
            from[count++] = step >= steps ? -1 : scale_row_offset(tiled, row0 + scale_row(wk, tid, i), n, nblk, n_tiles,
                                                                  n_items) + scale_step_offset(tiled, step);
        }
    return count;
}
"""


def shapes():
    found = set()
    for path in glob.glob(os.path.join(CSRC, "gemm_wide*.hip")):
        for wm, wn, wk, mf, nf in re.findall(r"\{(\d), (\d), (\d), (\d), (\d), [\d.]+f", open(path).read()):
            found.add((int(wn) * int(nf) * 16, int(wk)))
    return sorted(found)


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("scale_stage")
    (d / "walk.cpp").write_text(WALK)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "walk.cpp"),
                           "-o", str(d / "walk.so")])
    return ctypes.CDLL(str(d / "walk.so")).walk


def test_every_shape_is_known():
    assert len(shapes()) >= 13                              # different (weight rows, steps a phase) of the tables


@pytest.mark.parametrize("bn,wk", shapes())
@pytest.mark.parametrize("tiled", [False, True])
def test_one_writer_of_the_right_scales(walk, bn, wk, tiled):
    n = 2 * bn + 5                                          # the third block repeats the last row, or its tile
    room = (ctypes.c_int * (2 * 1024 * 8))
    for k in (128, 128 * 5, 128 * (2 * wk + 3), 4096):
        steps = k // 128
        for row0 in (0, bn, 2 * bn):
            for pair in range((steps + 2 * wk - 1) // (2 * wk)):
                lds, where = room(), room()
                count = walk(int(tiled), bn, wk, row0, n, k, pair, lds, where)
                got = dict(zip(lds[:count], where[:count]))
                assert len(got) == count == bn * 2 * wk     # nobody shares a dword
                for r in range(bn):
                    for c in range(2 * wk):
                        step = pair * 2 * wk + c
                        if tiled:
                            tile = min((row0 + r) // 16, (n + 15) // 16 - 1)
                            want = (tile * ((steps + 3) // 4) + step // 4) * 256 + r % 16 * 16 + step % 4 * 4
                        else:
                            want = min(row0 + r, n - 1) * (k // 32) + 4 * step
                        assert got[r * (8 * wk + 4) + 4 * c] == (want if step < steps else -1)
