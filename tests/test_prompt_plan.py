"""Tile and K split of the prompt projections, asked without a GPU: the split decides the order of the sums, so the sizes where other
step times chose other splits (and were slower) are pinned, as are sizes around them."""
import ctypes as C
import os

import pytest

from paper_2307_02628_amd import _build, skd

SKINNY, MID, TILE, CHUNKS = range(4)


class RowsGemm(C.Structure):
    _fields_ = [("kind", C.c_int), ("B_pad", C.c_int), ("R", C.c_int), ("split", C.c_int), ("wr", C.c_int), ("ar", C.c_int), ("partial", C.c_bool)]


@pytest.fixture(scope="module")
def plan():
    if not os.path.exists(skd.LIB_PATH):
        _build.build(force=True)
    f = getattr(skd.lib(), "_Z9plan_rowsiiib")
    f.argtypes, f.restype = [C.c_int, C.c_int, C.c_int, C.c_bool], RowsGemm
    return f


@pytest.mark.parametrize("N,K,rows,tile", [
    (512, 1536, 8208, (128, 256, 1)), (512, 1536, 8640, (128, 256, 1)), (512, 1536, 9104, (128, 256, 1)),
    (2048, 2048, 2464, (128, 256, 1)), (2048, 2048, 2816, (128, 256, 1)),
    (2048, 8192, 672, (128, 256, 4)), (2048, 8192, 912, (128, 256, 4)), (2048, 8192, 1088, (128, 256, 3)),
    (2048, 8192, 4192, (256, 256, 3)), (2048, 8192, 4320, (256, 256, 3)), (2048, 8192, 4800, (256, 256, 3)), (2048, 8192, 5120, (256, 256, 3)),
    (4096, 4096, 672, (128, 256, 2)), (4096, 16384, 144, (128, 256, 8))])
def test_splits(plan, N, K, rows, tile):
    p = plan(N, K, rows, True)
    assert (p.wr, p.ar, p.split) == tile and p.partial == (p.split > 1)
    assert p.kind == (TILE if tile[:2] == (256, 256) else MID)


def test_every_plan_can_be_launched(plan):
    for N, K in ((768, 256), (256, 1024), (1152, 384), (512, 1536), (6144, 2048), (2048, 8192), (12288, 4096), (4096, 16384)):
        for split_ok in (False, True):
            for rows in [*range(16, 1200, 16), *range(1200, 70000, 1008)]:
                p = plan(N, K, rows, split_ok)
                if rows <= 64:
                    assert p.kind == SKINNY and p.B_pad >= rows and p.partial == split_ok
                    continue
                assert p.kind in (MID, TILE) and N % p.wr == 0 and (p.split == 1 or split_ok)
                assert p.split * rows * N <= 32 << 20 or p.split == 1
                assert K // 32 // p.split >= 8 or p.split == 1
