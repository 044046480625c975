"""Which columns of narrow models take the one-launch kernel, asked without a GPU: points measured on both sides of the line."""
import ctypes as C
import os

import pytest

from paper_2307_02628_amd import _build, skd
from tests.helpers import internal


@pytest.fixture(scope="module")
def team_keys():
    if not os.path.exists(skd.LIB_PATH):
        _build.build(force=True)
    f = internal("bf16_team_keys")
    f.argtypes, f.restype = [C.c_int, C.c_int, C.c_long, C.c_long], C.c_bool
    return lambda d, B, keys: f(d, B, keys, B * keys)


# (width, rows, keys): the separate kernels were faster
@pytest.mark.parametrize("d,B,keys", [(64, 32, 4000), (64, 64, 1500), (64, 64, 2000), (64, 96, 1500), (64, 128, 1000), (64, 128, 2000), (128, 32, 4000),
                                      (128, 64, 2000), (128, 96, 1500), (128, 128, 2000), (192, 128, 1000), (192, 64, 3000), (192, 128, 2000),
                                      (256, 96, 3000), (320, 96, 3000), (384, 128, 2100), (512, 128, 2100), (512, 1, 6000), (512, 2, 6000), (512, 1, 8000)])
def test_slower_points_take_separate_kernels(team_keys, d, B, keys):
    assert not team_keys(d, B, keys)


@pytest.mark.parametrize("d,B,keys", [(64, 1, 8000), (64, 8, 8000), (64, 32, 2000), (64, 64, 1000), (64, 128, 500), (128, 64, 1500), (128, 96, 1000),
                                      (192, 32, 3000), (256, 64, 2000), (256, 128, 1000), (320, 64, 2000), (384, 64, 2000), (512, 64, 3000), (384, 128, 2000),
                                      (512, 128, 1500), (512, 1, 4000), (512, 4, 8000), (384, 1, 8000), (256, 2, 16), (512, 128, 16)])
def test_faster_points_take_one_launch(team_keys, d, B, keys):
    assert team_keys(d, B, keys)
