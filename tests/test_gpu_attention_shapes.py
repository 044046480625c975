"""Decode attention while its launch shape changes with the position: contexts growing through the limits at which waves
are added (2, 4, 8, 16 blocks of 32 keys) and the key range is split (17 blocks), few (row, head) pairs, ragged rows.
Every step against a state whose shape is fixed at its largest; the two differ in the order of fp32 sums and in bf16
roundings of the result (8 mantissa bits), hence the bar of the other kernel-against-kernel tests, 5e-3 of the range."""
import os

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H", [(256, 4), (256, 2)])
@pytest.mark.parametrize("B,P,steps,ragged", [(1, 28, 40, False), (3, 250, 12, True), (2, 505, 14, False), (1, 540, 10, False)])
def test_shape_follows_position(d, H, B, P, steps, ragged):
    shape = S.ModelShape(L=2, d=d, H=H, f=512, V=400, max_pos=600)
    w = S.weights_to_bf16_values(S.make_weights(shape, 3))
    tokens = S.make_prompts(B, P, shape.V, 4)
    mask = S.make_ragged_mask(B, P, P - 40, P, seed=5) if ragged else None
    tape = S.make_token_tape(B, steps, shape.V, 6)

    def run():
        out = []
        with skd.Decoder(skd.make_config(shape, B, P, P + steps, 2, 2, page_tokens=32), w) as dec:
            dec.prefill(tokens, mask)
            for k in range(steps):
                dec.decode_step(P + k, tape[k])
                out.append(dec.logits_argmax()[1].copy())
        return np.stack(out)

    got = run()
    os.environ.update(SKD_ATTN_WAVES="16", SKD_ATTN_SPLITS="8")
    try:
        want = run()
    finally:
        for k in ("SKD_ATTN_WAVES", "SKD_ATTN_SPLITS"):
            os.environ.pop(k)
    assert np.abs(got - want).max() <= 5e-3 * (want.max() - want.min())
