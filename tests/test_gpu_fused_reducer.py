"""Few rows: the row reducers as prologues of the projections against separate reducers (SKD_FUSE_LN=0).  Same sums in
another order, rounded to bf16 (8 mantissa bits) between kernels: 5e-3 of the logit range, the bar of the other
kernel-against-kernel tests; the residual stream (fp32, read back) to 2e-2 of its range."""
import os

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


# widths whose float4 chunks fill a wave partly (384), one chunk per thread (512, 2048), and one and a part (2304 for 512
# threads); partial sums of more than the four that are requested together; the widest rows that one to two and three to
# four rows may have (four rows of 2048 need a split of 2: 96 KiB of rows and partial sums of the 128 allowed)
@pytest.mark.parametrize("B,d,H,f,env", [
    (B, *shape) for B in (1, 2, 3, 4)
    for shape in [(384, 6, 512, {}), (512, 4, 1536, {"SKD_S_FFN2": "8", "SKD_S_OUT": "2"}), (2048, 16, 256, {"SKD_S_OUT": "2"}),
                  (2304, 18, 256, {}), (4096, 32, 512, {"SKD_S_OUT": "2"})] if B <= 2 or shape[0] <= 2048])
def test_fused_against_separate(B, d, H, f, env):
    shape = S.ModelShape(L=3, d=d, H=H, f=f, V=200, max_pos=64)
    w = S.weights_to_bf16_values(S.make_weights(shape, 11))
    P, N = 5, 12
    tokens = S.make_prompts(B, P, shape.V, 12)
    tape = S.make_token_tape(B, N - P, shape.V, 13)
    out, reducers = {}, {}
    for fuse in ("1", "0"):
        os.environ.update(env, SKD_FUSE_LN=fuse)
        try:
            with skd.Decoder(skd.make_config(shape, B, P, N, 1, 3), w) as dec:
                dec.prefill(tokens)
                dec.profile_enable(1)
                logits, hidden = [], []
                for k in range(N - P):
                    dec.decode_step(P + k, tape[k])
                    hidden.append(dec.read_hidden())
                    logits.append(dec.logits_argmax()[1].copy())
                reducers[fuse] = dec.profile_read()["reduce_ln"]["launches"]
                out[fuse] = np.stack(logits), np.stack(hidden)
        finally:
            for k in (*env, "SKD_FUSE_LN"):
                os.environ.pop(k, None)
    # the fused state launches one reducer a step, behind the last layer; the other two a layer
    layers = sum(skd.skd_schedule(P + k, P, N, 1, 3, shape.L) for k in range(N - P))
    assert (reducers["1"], reducers["0"]) == (N - P, 2 * layers)
    for got, want, tol in zip(out["1"], out["0"], (5e-3, 2e-2)):
        assert np.abs(got - want).max() <= tol * (want.max() - want.min())
