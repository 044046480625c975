"""The threshold search of the sampling head on few candidates (up to 64: all their masses in one round) and on up to 1024 (interval divided
by 17), with many equal logits: identical vocabulary rows give identical logits, and a nucleus takes all tokens tied with
its last one.  Tokens equal the oracle's wherever its decision margins exceed fp32 rounding (1e-5 of the mass, the bar of
the other sampling tests)."""
import numpy as np
import pytest

import synth_inputs as S
from oracle import oracle as O
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


# (50272 equal tokens are left out: half a token's mass, the largest margin of a draw, is 1e-5)
@pytest.mark.parametrize("V,levels", [(V, n) for V in (40, 64, 65, 256, 257, 1000, 1025, 9000, 50272) for n in (1, 3, 40) if (V, n) != (50272, 1)])
def test_ties(V, levels):
    shape = S.ModelShape(L=1, d=128, H=2, f=128, V=V, max_pos=8)
    w = S.make_weights(shape, 5)
    g = np.random.Generator(np.random.Philox(key=[V, levels]))
    kinds = g.standard_normal(size=(levels, 128), dtype=np.float32) * np.float32(0.2)
    w["lm_head"] = kinds[g.integers(0, levels, size=V)]
    w = S.weights_to_bf16_values(w)
    B = 5
    rng = np.random.default_rng(9)
    checked = total = 0
    with skd.Decoder(skd.make_config(shape, B, 2, 4, 1, 1), w) as dec:
        dec.prefill(S.make_prompts(B, 2, V, 6))
        lg = dec.logits_argmax()[1].copy()
        assert len(np.unique(lg[0])) <= levels
        for temperature in (0.1, 0.5, 1.0, 2.0):
            for top_p in (0.05, 0.5, 0.9, 0.99, 1.0):
                u = rng.random(B).astype(np.float32)
                tok, _ = dec.logits_sample(u, temperature, top_p, want_logits=False)
                for b in range(B):
                    ref, m_set, m_run = O.op_sample(lg[b], temperature, top_p, float(u[b]))
                    total += 1
                    if m_set > 1e-5 and m_run > 1e-5:
                        assert tok[b] == ref, (temperature, top_p, b)
                        checked += 1
    assert checked >= total // 4
