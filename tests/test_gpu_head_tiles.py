"""LM heads whose workgroups own four tiles, fewer and one (rounds that the vocabulary does not fill) against equal
workgroups: a logit is the same sum whatever group its tile is in, so logits and tokens are the same bits."""
import os

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


# tiles (16 words): 1024 equal groups of 4 and no rest; one more tile, partly filled; 3 tiles over; half a round over (rounds
# of two), a little less than that and more (a round of two or three that is not full), nearly a whole round
@pytest.mark.parametrize("B", [2, 19, 47, 64, 90, 128])
@pytest.mark.parametrize("V", [16384, 16390, 16384 + 48, 16384 + 16 * 300, 16384 + 16 * 520, 16384 + 16 * 700 + 5, 16384 + 16 * 1023])
def test_mixed_groups(B, V):
    shape = S.ModelShape(L=1, d=128, H=2, f=64, V=V, max_pos=8)
    w = S.weights_to_bf16_values(S.make_weights(shape, 5))
    tokens = S.make_prompts(B, 3, V, 6)

    def run(env):
        os.environ.update(env)
        try:
            with skd.Decoder(skd.make_config(shape, B, 3, 6, 1, 1), w) as dec:
                dec.prefill(tokens)
                return [x.copy() for x in dec.logits_argmax()]
        finally:
            for k in env:
                os.environ.pop(k, None)
    tok, lg = run({})
    tok1, lg1 = run({"SKD_R_HEAD": "1"})  # one tile per workgroup
    np.testing.assert_array_equal(lg, lg1)
    np.testing.assert_array_equal(tok, tok1)
    np.testing.assert_array_equal(tok, lg.argmax(-1))
