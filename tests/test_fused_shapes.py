"""What the projections with the row reducer, or the merge of the attention's splits, in their prologue accept, asked without a
launch (CPU only): everything the engine plans for one to four rows, nothing beyond what the kernel was written for."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2307_02628_amd import _build, skd
from tests.helpers import internal

EPI_PARTIAL, EPI_QKV, EPI_RELU, EPI_LOGITS = range(4)
P, I = C.c_void_p, C.c_int


class RowMap(C.Structure):
    _fields_ = [("seq", P), ("first_row", P), ("start", P), ("P", I)]


class KvGeom(C.Structure):
    _fields_ = [("page_tokens", I), ("max_pages", I), ("H", I), ("dh", I), ("page_elems", C.c_long)]


class GemmArgs(C.Structure):
    _fields_ = [("W", P), ("G", I), ("A", P), ("bias", P), ("N", I), ("K", I), ("B", I), ("B_pad", I), ("t0", I), ("split", I),
                ("ws_rot", I), ("rows", I), ("rm", RowMap), ("x", P), ("partial", P), ("q_out", P), ("kv_new", P), ("kv_pool", P),
                ("bt_layer", P), ("d", I), ("kv", KvGeom), ("act_out", P), ("ln_x", P), ("ln_partial", P), ("ln_bias", P),
                ("ln_g", P), ("ln_b", P), ("ln_x_out", P), ("ln_split", I), ("logits", P), ("attn_part", P), ("attn_splits", I),
                ("head_full", I), ("head_mid", I), ("head_mid_r", I), ("pmax", P), ("pidx", P)]


def test_mirror_of_the_arguments(tmp_path):
    """The structures above are the library's, field by field."""
    lines = ['#include <cstddef>', '#include "skd_kernels.h"']
    for s in (RowMap, KvGeom, GemmArgs):
        lines.append(f"static_assert(sizeof(skd::{s.__name__}) == {C.sizeof(s)}, \"size of {s.__name__}\");")
        lines += [f"static_assert(offsetof(skd::{s.__name__}, {f}) == {getattr(s, f).offset}, \"{s.__name__}::{f}\");" for f, _ in s._fields_]
    src = tmp_path / "mirror.hip"
    src.write_text("\n".join(lines) + "\n")
    res = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "--cuda-host-only", "-fsyntax-only",
                          "-std=c++17", "-Wno-invalid-offsetof", "-x", "hip", "-I", _build.CSRC, str(src)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]


@pytest.fixture(scope="module")
def check():
    if not os.path.exists(skd.LIB_PATH):
        _build.build(force=True)
    f = internal("bf16_gemm_ln_check")

    def call(N, K, B, R=2, epi=EPI_QKV, **other):
        a = GemmArgs(N=N, K=K, B=B, B_pad=16, G=R, split=1, ln_split=1)
        for k, v in other.items():
            setattr(a, k, v)
        return f(C.byref(a), epi, R)
    return call


def test_planned_shapes_are_accepted(check):
    for B in (1, 2, 3, 4):
        for d in range(64, (4096 if B <= 2 else 2048) + 1, 64):
            for R in (1, 2, 3, 4):
                for ln_split in (1, 2, 8, 32):
                    assert check(3 * d, d, B, R, EPI_QKV, ln_split=ln_split) == -(-3 * d // (16 * R))
                    assert check(4 * d + 32, d, B, R, EPI_RELU, ln_split=ln_split) == -(-(4 * d + 32) // (16 * R))


@pytest.mark.parametrize("B,K,R,epi,other", [
    (5, 256, 2, EPI_QKV, {}), (0, 256, 2, EPI_QKV, {}), (1, 4160, 2, EPI_QKV, {}), (3, 2112, 2, EPI_RELU, {}), (1, 48, 2, EPI_QKV, {}),
    (1, 256, 5, EPI_QKV, {}), (1, 256, 0, EPI_QKV, {}), (1, 256, 2, EPI_PARTIAL, {}), (1, 256, 2, EPI_LOGITS, {}),
    (1, 256, 2, EPI_QKV, {"split": 2}), (1, 256, 2, EPI_QKV, {"rows": 16}), (1, 256, 2, EPI_QKV, {"B_pad": 32}),
    (1, 256, 2, EPI_QKV, {"ln_split": 0}), (1, 256, 2, EPI_QKV, {"G": 5})])
def test_others_are_refused(check, B, K, R, epi, other):
    assert check(768, K, B, R, epi, **other) == -1


@pytest.fixture(scope="module")
def merge_check():
    if not os.path.exists(skd.LIB_PATH):
        _build.build(force=True)
    f = internal("bf16_gemm_merge_check")

    def call(N, K, B, R=2, waves=8, dh=128, splits=4, **other):
        a = GemmArgs(N=N, K=K, B=B, B_pad=16, G=R, split=1, attn_splits=splits, kv=KvGeom(64, 4, K // dh, dh, 0))
        for k, v in other.items():
            setattr(a, k, v)
        return f(C.byref(a), R, waves)
    return call


def test_merged_shapes_are_accepted(merge_check):
    for B in (1, 2):
        for dh in (64, 128):
            for d in range(dh, 4096 + 1, dh):
                for R in (1, 2):
                    for splits in (2, 3, 8):
                        assert merge_check(d, d, B, R, dh=dh, splits=splits) == -(-d // (16 * R))
    assert merge_check(2048, 2048, 2, split=4) == 64


@pytest.mark.parametrize("B,K,other", [
    (3, 256, {}), (0, 256, {}), (1, 4224, {}), (1, 4128, {"dh": 64}), (1, 48, {"dh": 64}), (1, 192, {}), (1, 256, {"dh": 32}),
    (1, 256, {"splits": 1}), (1, 256, {"splits": 9}), (1, 256, {"R": 3}), (1, 256, {"R": 0}), (1, 256, {"waves": 4}),
    (1, 256, {"B_pad": 32}), (1, 256, {"rows": 16}), (1, 256, {"split": 3}), (1, 256, {"split": 0}), (1, 256, {"G": 5})])
def test_others_are_not_merged(merge_check, B, K, other):
    assert merge_check(256, K, B, **other) == -1
