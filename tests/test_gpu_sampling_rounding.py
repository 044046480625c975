"""Draws that rounding decides: with top_p 1 the nucleus ends where float sums stop growing, and u at the ends of [0, 1) picks its
first and last members, so these tokens change with the order in which masses are added.  They are recorded
(golden/sampling_rounding.json): the order is part of what a seed reproduces."""
import json
import os

import numpy as np
import pytest

from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "sampling_rounding.json")
B, D = 128, 64
# vocabulary, spread of the LM head, temperature: up to 64, 256, 1024 candidates and more in one pass, and the chunked first pass
CASES = [(60, 1.0, 1.0), (200, 1.0, 0.7), (1000, 0.25, 0.3), (1000, 1.5, 1.0), (3000, 0.3, 0.4), (50272, 1.5, 0.7), (50272, 0.7, 0.3)]


def tokens(V, spread, temperature):
    import torch
    rng = np.random.default_rng([V, int(100 * spread)])
    put = lambda a: torch.from_numpy(np.asarray(a, dtype=np.float32)).to(torch.bfloat16).cuda()  # noqa: E731
    zero = {"ln1_g": D, "ln1_b": D, "wqkv": (3 * D, D), "bqkv": 3 * D, "wo": (D, D), "bo": D, "ln2_g": D, "ln2_b": D, "w1": (64, D), "b1": 64,
            "w2": (D, 64), "b2": D}
    w = {"tok_emb": put(rng.normal(0, 1, (V, D))), "pos_emb": put(np.zeros((8, D))), "lnf_g": put(np.ones(D)), "lnf_b": put(np.zeros(D)),
         "lm_head": put(rng.normal(0, spread, (V, D))), **{k: [put(np.zeros(s))] for k, s in zero.items()}}
    torch.cuda.synchronize()
    shape = type("Shape", (), dict(L=1, d=D, H=1, f=64, V=V, max_pos=8))
    u = np.where(np.arange(B) % 2, np.float32(0.99999994), np.float32(0)).astype(np.float32)
    with skd.Decoder(skd.make_config(shape, B, 2, 6, 1, 1), w, location=skd.DEVICE, elem=skd.W_BF16) as dec:
        dec.prefill(rng.integers(0, V, (B, 2)).astype(np.int32))
        return dec.logits_sample(u, temperature, 1.0)[0].tolist()


@pytest.mark.parametrize("case", CASES)
def test_recorded_tokens(case):
    with open(GOLDEN) as f:
        want = json.load(f)["%d %g %g" % case]
    assert tokens(*case) == want
