"""LM heads of few tiles, whose K range is split over workgroups, against whole K in a workgroup (SKD_S_HEAD=1)."""
import os

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


# one tile; three, partly filled; rows of logits that do not start at 16 bytes; the most tiles that are split and one more
# token; 2, 4 and 8 parts, on the wave-specialised kernel too
@pytest.mark.parametrize("d,H,V,B", [(1024, 8, 16, 1), (1024, 8, 777, 2), (2048, 16, 33, 16), (1024, 8, 2048, 17), (1024, 8, 2049, 3),
                                     (2048, 16, 1000, 47), (2048, 16, 501, 64), (1024, 8, 1001, 90), (1024, 8, 1000, 128),
                                     (4096, 32, 250, 5), (2048, 32, 2046, 97)])
def test_head_parts(d, H, V, B):
    shape = S.ModelShape(L=1, d=d, H=H, f=64, V=V, max_pos=8)
    w = S.weights_to_bf16_values(S.make_weights(shape, 5))
    tokens = S.make_prompts(B, 3, V, 6)

    def run(env):
        os.environ.update(env)
        try:
            with skd.Decoder(skd.make_config(shape, B, 3, 6, 1, 1), w) as dec:
                dec.prefill(tokens)
                tok, lg = (x.copy() for x in dec.logits_argmax())
                u = np.full(B, 0.5, dtype=np.float32)
                return tok, lg, dec.logits_sample(u, 1.0, 0.9)[1].copy()
        finally:
            for k in env:
                os.environ.pop(k, None)
    tok, lg, lg_sampled = run({})
    _, lg1, _ = run({"SKD_S_HEAD": "1"})
    # both are fp32 sums of the same d products, in another order: each within d 2^-24 sum |w a| <= d 2^-24 |w| |a|
    a = np.sqrt(d) * np.abs(np.asarray(w["lnf_g"], dtype=np.float64)).max() + np.linalg.norm(w["lnf_b"])
    rows = np.linalg.norm(np.asarray(w.get("lm_head", w["tok_emb"]), dtype=np.float64), axis=1)
    assert (np.abs(lg.astype(np.float64) - lg1) <= 2 * d * 2.0 ** -24 * a * rows[None, :]).all()
    np.testing.assert_array_equal(tok, lg.argmax(-1))
    np.testing.assert_array_equal(lg_sampled, lg)


def test_identical_rows_give_identical_logits():
    """... and the lowest index wins, as without parts."""
    shape = S.ModelShape(L=1, d=1024, H=8, f=64, V=1000, max_pos=8)
    w = S.weights_to_bf16_values(S.make_weights(shape, 7))
    emb = np.asarray(w["tok_emb"]).copy()
    emb[[990, 517, 18]] = emb[400] * 8  # far above the others in size: one of the four, or none, is the largest
    w["tok_emb"] = emb
    with skd.Decoder(skd.make_config(shape, 20, 3, 6, 1, 1), w) as dec:
        dec.prefill(S.make_prompts(20, 3, 1000, 8))
        tok, lg = (x.copy() for x in dec.logits_argmax())
    for i in (517, 990):
        np.testing.assert_array_equal(lg[:, i], lg[:, 18])
    np.testing.assert_array_equal(tok, lg.argmax(-1))


def test_overrides_out_of_range_are_ignored(monkeypatch):
    shape = S.ModelShape(L=1, d=1024, H=8, f=64, V=1000, max_pos=8)
    w = S.weights_to_bf16_values(S.make_weights(shape, 9))
    tokens = S.make_prompts(5, 3, 1000, 10)

    def logits(name=None, value=None):
        with monkeypatch.context() as m:
            if name:
                m.setenv(name, value)
            with skd.Decoder(skd.make_config(shape, 5, 3, 6, 1, 1), w) as dec:
                dec.prefill(tokens)
                return dec.logits_argmax()[1].copy()
    parts, whole = logits(), logits("SKD_S_HEAD", "1")
    assert (parts != whole).any()  # another order of the sums
    for name, value in (("SKD_R_HEAD", "9"), ("SKD_R_HEAD", ""), ("SKD_U_HEAD", "0"), ("SKD_W_HEAD", "16"), ("SKD_S_HEAD", "9")):
        np.testing.assert_array_equal(logits(name, value), parts)
    for name, value in (("SKD_R_HEAD", "2"), ("SKD_U_HEAD", "1"), ("SKD_W_HEAD", "8")):
        np.testing.assert_array_equal(logits(name, value), whole)
