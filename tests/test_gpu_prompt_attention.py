"""Prompt attention at the edges of its blocks (32 keys), waves (32 queries), workgroups (128 queries) and page-table
windows (64 pages), with scores spread widely enough that the softmax reference moves and with equal ones, against the
column-by-column path.  Bars as in test_gpu_prompt_shapes."""
import numpy as np
import pytest

import synth_inputs as S
from tests.test_gpu_prompt_shapes import check, prompt

pytestmark = pytest.mark.gpu

H128 = S.ModelShape(L=2, d=256, H=2, f=256, V=300, max_pos=2200)
H64 = S.ModelShape(L=2, d=128, H=2, f=256, V=300, max_pos=2200)


@pytest.mark.parametrize("shape", [H128, H64])
@pytest.mark.parametrize("B,P,shortest", [(1, 31, 0), (2, 32, 0), (1, 33, 0), (2, 127, 0), (1, 128, 0), (3, 129, 1), (4, 300, 97)])
def test_lengths(shape, B, P, shortest):
    check(shape, B, P, shortest, {}, 70)


def test_second_window_of_pages():
    check(H64, 1, 2100, 0, {}, 80)      # 66 pages of 32 positions


@pytest.mark.parametrize("gain", [0.0, 40.0])
def test_equal_and_spread_scores(gain):
    # LayerNorm gain 0: all scores equal; 40: scores of hundreds, one key takes nearly all the weight.  With hidden states
    # this large the two paths' bf16 roundings decide near-ties between keys differently: only that nothing overflows and
    # that most positions agree is asked of the spread case, and the usual bar of the equal one.
    w = S.make_weights(H128, 90)
    w["ln1_g"] = [g * gain for g in w["ln1_g"]]
    w = S.weights_to_bf16_values(w)
    tokens = S.make_prompts(2, 150, H128.V, 91)
    got, want = prompt(H128, w, tokens, None, {}), prompt(H128, w, tokens, None, {"SKD_PREFILL_BATCHED": "0"})
    assert np.isfinite(got[0]).all() and all(np.isfinite(x).all() for kv in got[1] for x in kv)
    scale = want[0].max() - want[0].min()
    if gain == 0.0:
        assert np.abs(got[0] - want[0]).max() <= 5e-3 * scale
    else:
        for (ka, _), (kb, _) in zip(got[1][2:], want[1][2:]):       # layer 1: behind one attention
            off = np.abs(ka - kb).max(axis=1) > 5e-2 * np.abs(kb).max()
            assert off.mean() <= 0.05
