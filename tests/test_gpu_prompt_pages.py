"""Where the tiled q | k | v projections of a prompt put keys and values: pages of one and of an odd number of 32-key blocks, tiles
that begin in either half of a block, last tiles with 1 to 15 real positions, padding tiles; heads of 64 and 128."""
import os

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads", [4, 8])
@pytest.mark.parametrize("page_tokens", [32, 96, 160])
@pytest.mark.parametrize("tile", ["256x256x1", "128x256x1", "128x128x1", "64x64x1"])
def test_pages(tile, page_tokens, heads):
    B, P = 7, 171
    shape = S.ModelShape(L=2, d=512, H=heads, f=512, V=300, max_pos=P + 2)
    w = S.weights_to_bf16_values(S.make_weights(shape, 31))
    tokens = S.make_prompts(B, P, shape.V, 32)
    lens = [171, 1, 16, 95, 97, 160, 30]
    mask = (np.arange(P)[None, :] >= P - np.array(lens)[:, None]).astype(np.uint8)

    def cached(env, page):
        os.environ.update(env)
        try:
            with skd.Decoder(skd.make_config(shape, B, P, P + 2, 1, 2, page_tokens=page), w) as dec:
                dec.prefill(tokens, mask)
                lg = dec.logits_argmax()[1].copy()
                dec.decode_step(P, tokens[:, 0])  # reads the pages as the decode attention does
                return lg, dec.logits_argmax()[1].copy(), [dec.kv_read(l, b) for l in range(2) for b in range(B)]
        finally:
            for k in env:
                os.environ.pop(k, None)
    got, want = cached({"SKD_PREFILL_TILE": tile}, page_tokens), cached({"SKD_PREFILL_TILE": tile}, 64)
    # the same sums, in other places
    for g, r in zip(got[2], want[2]):
        for x, y in zip(g, r):
            np.testing.assert_array_equal(x, y)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])
    # and the column by column path puts the same rows there (bars as in test_gpu_prompt_shapes)
    ref = cached({"SKD_PREFILL_BATCHED": "0"}, page_tokens)
    for n, (g, r) in enumerate(zip(got[2], ref[2])):
        for x, y in zip(g, r):
            real = slice(P - lens[n % B], P)
            np.testing.assert_allclose(x[real], y[real], rtol=2e-2, atol=2e-2)
