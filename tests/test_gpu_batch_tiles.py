"""Batches around the limits of the padded batch sizes (32, 48, 64, 96, 128 rows) against the oracle, on the separate decode
kernels and on the one-launch columns."""
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd
from tests.helpers import compare

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("narrow_columns")]

BF16_TOL = 2e-2     # of the logit range: the bar of the bf16 path
WIDE = S.ModelShape(L=2, d=512, H=4, f=1536, V=1000, max_pos=64)      # 96 and 128 rows on the wave-specialised kernel
NARROW = S.ModelShape(L=2, d=384, H=6, f=1088, V=333, max_pos=64)     # 34 k-steps: FFN2 on the general one


@pytest.mark.parametrize("shape", [WIDE, NARROW])
@pytest.mark.parametrize("B", [33, 47, 48, 49, 65, 96, 97])
def test_batch(shape, B):
    w = S.weights_to_bf16_values(S.make_weights(shape, 21))
    P, N = 9, 13
    compare(shape, w, S.make_prompts(B, P, shape.V, 22), P, N, 1, 2, BF16_TOL, dtype=skd.BF16,
            mask=S.make_ragged_mask(B, P, 2, P, seed=23), tape=S.make_token_tape(B, N - P, shape.V, 24), min_decided=0.0)
