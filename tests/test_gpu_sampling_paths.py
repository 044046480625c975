"""The sampling head where the number of tokens that can be in the nucleus passes the limits of its paths (256 and 1024
for one wave, 4096 for four, beyond: the whole workgroup), over vocabularies of every register tile.  Tokens equal the
oracle's wherever its decision margins exceed fp32 rounding (1e-5 of the mass, the bar of the other sampling tests)."""
import numpy as np
import pytest

import synth_inputs as S
from oracle import oracle as O
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [300, 16385, 32768, 50272, 65536])
def test_candidate_counts(V):
    shape = S.ModelShape(L=1, d=128, H=2, f=128, V=V, max_pos=8)
    w = S.make_weights(shape, 5)
    g = np.random.Generator(np.random.Philox(key=[5, 98]))
    w["lm_head"] = g.standard_normal(size=(V, shape.d), dtype=np.float32) * np.float32(0.09)
    w = S.weights_to_bf16_values(w)
    B = 4
    rng = np.random.default_rng(8)
    checked, counts = 0, []
    with skd.Decoder(skd.make_config(shape, B, 2, 4, 1, 1), w) as dec:
        dec.prefill(S.make_prompts(B, 2, V, 6))
        _, lg = dec.logits_argmax()
        for temperature in (0.05, 0.2, 0.3, 0.4, 0.5, 0.7, 1.0, 3.0):
            for top_p in (0.3, 0.9, 1.0):
                u = rng.random(B).astype(np.float32)
                tok, _ = dec.logits_sample(u, temperature, top_p, want_logits=False)
                for b in range(B):
                    p = np.exp((lg[b].astype(np.float64) - lg[b].max()) / temperature)
                    total = p.sum()
                    lower = max([t for t in (2.0 ** -5, 2.0 ** -10) if p[p >= t].sum() >= top_p * total],
                                default=(1 - top_p) * total / (2 * V))
                    counts.append(int((p >= lower).sum()))
                    ref, m_set, m_run = O.op_sample(lg[b], temperature, top_p, float(u[b]))
                    if m_set > 1e-5 and m_run > 1e-5:
                        assert tok[b] == ref, (temperature, top_p, b, counts[-1])
                        checked += 1
    assert checked >= 30
    if V >= 32768:  # all four paths were taken
        assert np.unique(np.digitize(counts, [257, 1025, 4097])).tolist() == [0, 1, 2, 3], sorted(counts)
