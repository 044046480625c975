"""Every kernel and launch shape a prompt projection can take, against the column-by-column path (the decode kernels).

Bars as for the batched prompt path elsewhere: both sides round to bf16 between kernels (8 mantissa bits) and differ in
summation order only, so logits agree within 5e-3 of their range and cached keys and values within 2e-2."""
import os

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu

WIDE = S.ModelShape(L=2, d=512, H=4, f=1536, V=600, max_pos=320)       # every tile divides every N
NARROW = S.ModelShape(L=2, d=384, H=6, f=1088, V=333, max_pos=320)     # 384 and 1152: no 256 tiles; 1088 = 17 x 64


def prompt(shape, w, tokens, mask, env):
    B, P = tokens.shape
    os.environ.update(env)
    try:
        with skd.Decoder(skd.make_config(shape, B, P, P + 2, 1, shape.L, page_tokens=32), w) as dec:
            for _ in range(2):  # the second pass starts from what the first left in the workspace
                dec.prefill(tokens, mask)
                lg = dec.logits_argmax()[1].copy()
            return lg, [dec.kv_read(l, b) for l in range(shape.L) for b in range(B)]
    finally:
        for k in env:
            os.environ.pop(k, None)


def check(shape, B, P, shortest, env, seed):
    w = S.weights_to_bf16_values(S.make_weights(shape, seed))
    tokens = S.make_prompts(B, P, shape.V, seed + 1)
    mask = S.make_ragged_mask(B, P, shortest, P, seed=seed + 2) if shortest else None
    got, want = prompt(shape, w, tokens, mask, env), prompt(shape, w, tokens, mask, {"SKD_PREFILL_BATCHED": "0"})
    assert np.abs(got[0] - want[0]).max() <= 5e-3 * (want[0].max() - want[0].min())
    start = (mask == 0).sum(axis=1) if shortest else np.zeros(B, dtype=int)
    for i, ((ka, va), (kb, vb)) in enumerate(zip(got[1], want[1])):
        real = slice(int(start[i % B]), P)
        np.testing.assert_allclose(ka[real], kb[real], rtol=2e-2, atol=2e-2)
        np.testing.assert_allclose(va[real], vb[real], rtol=2e-2, atol=2e-2)


@pytest.mark.parametrize("shape", [WIDE, NARROW])
@pytest.mark.parametrize("tile", ["256x256x1", "256x256x3", "256x128x3", "128x256x1", "128x128x1", "128x128x4", "64x128x2", "128x64x3", "64x64x1", "64x64x5"])
def test_forced_tiles(shape, tile):
    check(shape, 7, 83, 9, {"SKD_PREFILL_TILE": tile}, 40)      # rows: no multiple of 64; K parts of unequal length


@pytest.mark.parametrize("shape,B,P,shortest", [
    (WIDE, 1, 1, 0), (NARROW, 1, 16, 0), (WIDE, 2, 16, 0), (NARROW, 1, 33, 0),     # 16, 16, 32, 48 rows: decode kernels
    (WIDE, 4, 13, 1), (WIDE, 1, 65, 0), (NARROW, 5, 47, 20), (WIDE, 3, 301, 0),     # 64 rows; 80, ragged, 912: tiles
    (WIDE, 13, 97, 20), (NARROW, 40, 31, 1)])                                      # ragged, more than 512 rows: top layer as a column
def test_planned_shapes(shape, B, P, shortest):
    check(shape, B, P, shortest, {}, 50)


# more than 512 rows, no multiple of 256: the top layer computes only k and v, from the weight tile behind q's
@pytest.mark.parametrize("shape", [WIDE, NARROW])
@pytest.mark.parametrize("tile", ["256x256x1", "256x128x2", "128x256x1", "128x128x1", "64x128x1", "128x64x1", "64x64x2"])
def test_forced_tiles_behind_q(shape, tile):
    check(shape, 9, 83, 50, {"SKD_PREFILL_TILE": tile}, 60)


# K parts of 1 to 9 k-steps (512 and 1536 columns over 16, 12, 8 and 5 parts), even and odd: fewer than, as many as and
# more than the stages of the rings of the kernels of eight waves
@pytest.mark.parametrize("tile", ["256x256", "256x128", "128x256"])
@pytest.mark.parametrize("split", [16, 12, 8, 5])
def test_short_k_parts(split, tile):
    check(WIDE, 7, 83, 9, {"SKD_PREFILL_TILE": f"{tile}x{split}"}, 70)


# 256 x 256 tiles: 12 workgroups (no multiple of 8: some XCDs have one more), 270 of 1 to 4 k-steps (more than CUs), and 294 to
# 882 of 16 and 48 k-steps with every epilogue
@pytest.mark.parametrize("split,B,P,shortest", [(1, 13, 97, 0), (15, 24, 96, 80), (1, 128, 300, 270)])
def test_several_tiles_per_workgroup(split, B, P, shortest):
    check(WIDE, B, P, shortest, {"SKD_PREFILL_TILE": f"256x256x{split}"}, 80)
