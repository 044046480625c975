"""Few rows at long contexts: the output projection of one or two rows that merges the attention's splits in its prologue against separate
kernels (SKD_FUSE_LN=0: merge kernel, row reducers).  Same sums in another order, rounded to bf16 (8 mantissa bits) between
kernels: 5e-3 of the logit range and 2e-2 of the residual stream's, the bars of the other kernel-against-kernel tests."""
import os

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


# both head widths; K ranges of one chunk per thread, fewer and more (4096 without a split along K: two); a K range of an odd
# number of k-steps (320 / 32 = 10, in 2 parts); 2, 3 and 8 splits (9: merged by the kernel), some without keys
@pytest.mark.parametrize("B", [1, 2, 3])  # (three rows keep separate kernels)
@pytest.mark.parametrize("d,H,env", [(512, 8, {}), (320, 5, {"SKD_S_OUT": "2"}), (2048, 16, {}), (2048, 32, {"SKD_S_OUT": "1", "SKD_R_OUT": "1"}),
                                     (4096, 32, {"SKD_S_OUT": "1"}), (1024, 8, {"SKD_U_OUT": "1"})])
@pytest.mark.parametrize("splits", [2, 3, 8, 9])
def test_against_separate_kernels(B, d, H, env, splits):
    shape = S.ModelShape(L=2, d=d, H=H, f=256, V=200, max_pos=160)
    w = S.weights_to_bf16_values(S.make_weights(shape, 21))
    P, N = 150, 153
    tokens = S.make_prompts(B, P, shape.V, 22)
    mask = S.make_ragged_mask(B, P, 3, P, seed=23) if B > 1 else None
    tape = S.make_token_tape(B, N - P, shape.V, 24)
    out = {}
    for fuse in ("1", "0"):
        os.environ.update(env, SKD_FUSE_LN=fuse, SKD_ATTN_SPLITS=str(splits))
        try:
            with skd.Decoder(skd.make_config(shape, B, P, N, 2, 2), w) as dec:
                dec.prefill(tokens, mask)
                logits, hidden = [], []
                for k in range(N - P):
                    dec.decode_step(P + k, tape[k])
                    hidden.append(dec.read_hidden())
                    logits.append(dec.logits_argmax()[1].copy())
                out[fuse] = np.stack(logits), np.stack(hidden)
        finally:
            for k in (*env, "SKD_FUSE_LN", "SKD_ATTN_SPLITS"):
                os.environ.pop(k, None)
    for got, want, tol in zip(out["1"], out["0"], (5e-3, 2e-2)):
        assert np.abs(got - want).max() <= tol * (want.max() - want.min())
