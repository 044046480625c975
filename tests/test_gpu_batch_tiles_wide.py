"""Batches of 33 to 64 rows of models from 2048 columns on, against the oracle and, bit by bit, against the general kernel alone
(SKD_GEMM_WS=0): the kernel with separate weight-streaming and activation-loading waves, which adds up in another order, begins
at 65 rows."""
import os

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd
from tests.helpers import compare

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2     # of the logit range: the bar of the bf16 path
# FFN2's K range of 10 stages of 4 k-steps; of 36 k-steps, no whole stages per part; more than a round of LM head workgroups
# (tiles of 4 rows and smaller ones)
SHAPES = [S.ModelShape(L=2, d=2048, H=16, f=1280, V=301, max_pos=32), S.ModelShape(L=1, d=2048, H=32, f=1152, V=4099, max_pos=32),
          S.ModelShape(L=1, d=2048, H=32, f=2048, V=17000, max_pos=32)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"f{s.f}_V{s.V}")
@pytest.mark.parametrize("B", [33, 48, 49, 64])
def test_batch(shape, B):
    w = S.weights_to_bf16_values(S.make_weights(shape, 41))
    P, N = 5, 8
    prompts, mask, tape = S.make_prompts(B, P, shape.V, 42), S.make_ragged_mask(B, P, 2, P, seed=43), S.make_token_tape(B, N - P, shape.V, 44)
    got, _, _ = compare(shape, w, prompts, P, N, 1, shape.L, BF16_TOL, dtype=skd.BF16, mask=mask, tape=tape, min_decided=0.1)
    os.environ["SKD_GEMM_WS"] = "0"
    try:
        general, _, _ = compare(shape, w, prompts, P, N, 1, shape.L, BF16_TOL, dtype=skd.BF16, mask=mask, tape=tape, min_decided=0.1)
    finally:
        os.environ.pop("SKD_GEMM_WS", None)
    for z, y in zip(got["logits"], general["logits"]):
        np.testing.assert_array_equal(z, y)
