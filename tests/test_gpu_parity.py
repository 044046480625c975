"""GPU parity: the HIP path through the C ABI against the CPU oracle on the
same seeded random-init weights and inputs, teacher-forced.

Tolerances (max |delta logit| relative to the logit range of the step):
  bf16 path  2e-2   -- weights/KV/activations rounded to bf16 (8 mantissa
                       bits) between kernels, fp32 accumulation
  fp32 path  1e-4   -- same arithmetic as the oracle up to summation order
Schedule, layer indices and cache lengths must match exactly.
"""
import numpy as np
import pytest

import synth_inputs as S
from oracle import oracle as O
from paper_2307_02628_amd import skd
from tests.helpers import compare, rel_err, run_hip

pytestmark = pytest.mark.gpu

BF16_TOL, FP32_TOL = 2e-2, 1e-4


def bf16_weights(shape, seed):
    return S.weights_to_bf16_values(S.make_weights(shape, seed))


def test_config1_fp32():
    # contract configuration 1 on the fp32 debug build of the path
    w = S.make_weights(S.TINY, 0)
    pr = S.make_prompts(2, 16, S.TINY.V, 1)
    got, ref, err = compare(S.TINY, w, pr, 16, 32, 2, 4, FP32_TOL, dtype=skd.FP32)
    assert [len(a) for a in got["layers"]] == [4] * 5 + [3] * 8 + [2] * 3
    print("fp32 config-1 per-step error:", err.max())


@pytest.mark.usefixtures("narrow_columns")
def test_config1_bf16():
    w = bf16_weights(S.TINY, 0)
    pr = S.make_prompts(2, 16, S.TINY.V, 1)
    got, ref, err = compare(S.TINY, w, pr, 16, 32, 2, 4, BF16_TOL, dtype=skd.BF16)
    assert got["pages"][0] < got["pages"][1] or got["pages"][0] == got["pages"][1]
    print("bf16 config-1 per-step error:", err.max())


def test_config1_full_depth_both():
    # n(t) = L everywhere: ordinary decoding
    for dtype, tol, w in ((skd.FP32, FP32_TOL, S.make_weights(S.TINY, 0)), (skd.BF16, BF16_TOL, bf16_weights(S.TINY, 0))):
        pr = S.make_prompts(2, 16, S.TINY.V, 1)
        compare(S.TINY, w, pr, 16, 32, 4, 4, tol, dtype=dtype)


MID = S.ModelShape(L=3, d=512, H=4, f=1536, V=1000, max_pos=128)      # head_dim 128, vocab tail (1000 % 16 != 0)
MID64 = S.ModelShape(L=5, d=384, H=6, f=1024, V=777, max_pos=160)     # head_dim 64


@pytest.mark.usefixtures("narrow_columns")
@pytest.mark.parametrize("dtype,tol", [(skd.FP32, FP32_TOL), (skd.BF16, BF16_TOL)])
def test_mid_ragged_left_padded(dtype, tol):
    # several KV pages and 32-key blocks, ragged batch (5 rows), left padding, page size 32
    w = S.make_weights(MID, 2)
    if dtype == skd.BF16:
        w = S.weights_to_bf16_values(w)
    B, P, N = 5, 40, 90
    pr = S.make_prompts(B, P, MID.V, 3)
    mask = S.make_ragged_mask(B, P, 1, 40, seed=4)
    mask[0] = 1
    mask[1] = 0
    mask[1, -1] = 1                                                    # a row with a single real prompt token
    compare(MID, w, pr, P, N, 1, 3, tol, mask=mask, dtype=dtype, page_tokens=32)


@pytest.mark.usefixtures("narrow_columns")
@pytest.mark.parametrize("B", [1, 16, 17, 33, 64, 100])     # activation tiles 1, 1, 2, 4, 4, 8 (batch padded to 16/32/64/128)
def test_batch_tiles_bf16(B):
    w = bf16_weights(MID64, 5)
    P, N = 9, 30
    pr = S.make_prompts(B, P, MID64.V, 6)
    compare(MID64, w, pr, P, N, 2, 5, BF16_TOL, dtype=skd.BF16)


@pytest.mark.parametrize("ws", ["1", "0"])
@pytest.mark.parametrize("B", [113, 128])
@pytest.mark.parametrize("small", [False, True])
def test_batch_128_projection_kernels(B, ws, small):
    # 8 activation tiles (batch padded to 128): the projections run on the kernel with separate weight-streaming
    # and activation-loading waves (K ranges of 4, 12 and 16 stages per workgroup here: a ring that never fills,
    # and one that wraps), or, switched off, on the general skinny kernel; ragged left padding
    import os
    shape = S.ModelShape(L=3, d=512, H=4, f=1536, V=1000, max_pos=64)
    if small:   # K ranges of one and two stages: a ring that is never ahead, weight prefetches past the end
        shape = S.ModelShape(L=2, d=128, H=2, f=256, V=300, max_pos=64)
    w = bf16_weights(shape, 91)
    P, N = 11, 24
    pr = S.make_prompts(B, P, shape.V, 92)
    mask = S.make_ragged_mask(B, P, 2, P, seed=93)
    old = os.environ.get("SKD_GEMM_WS")
    os.environ["SKD_GEMM_WS"] = ws
    try:
        compare(shape, w, pr, P, N, 1, shape.L, BF16_TOL, mask=mask, dtype=skd.BF16, page_tokens=32, min_decided=0.0)
    finally:
        if old is None:
            os.environ.pop("SKD_GEMM_WS", None)
        else:
            os.environ["SKD_GEMM_WS"] = old


@pytest.mark.usefixtures("narrow_columns")
@pytest.mark.parametrize("dtype,tol", [(skd.FP32, FP32_TOL), (skd.BF16, BF16_TOL)])
def test_warmup_layer(dtype, tol):
    # one warm-up layer at the bottom + top window (the setting of every Table 2 row)
    w = S.make_weights(MID64, 7)
    if dtype == skd.BF16:
        w = S.weights_to_bf16_values(w)
    pr = S.make_prompts(3, 12, MID64.V, 8)
    got, ref, _ = compare(MID64, w, pr, 12, 40, 2, 4, tol, warmup=1, dtype=dtype)
    assert all(a[0] == 0 and a[1] >= 2 for a in got["layers"][4:])


def test_free_running_equals_teacher_forced():
    w = bf16_weights(S.TINY, 0)
    pr = S.make_prompts(2, 16, S.TINY.V, 1)
    free = run_hip(S.TINY, w, pr, 16, 32, 2, 4, dtype=skd.BF16)
    forced = run_hip(S.TINY, w, pr, 16, 32, 2, 4, tape=free["fed"], dtype=skd.BF16)
    np.testing.assert_array_equal(free["logits"], forced["logits"])    # deterministic kernels
    for k in range(16):
        np.testing.assert_array_equal(free["fed"][k], free["logits"][k].argmax(-1))


def test_kv_bookkeeping_and_pages():
    w = bf16_weights(S.TINY, 0)
    cfg = skd.make_config(S.TINY, 2, 16, 32, 2, 4, page_tokens=32)
    pr = S.make_prompts(2, 16, S.TINY.V, 1)
    with skd.Decoder(cfg, w) as dec:
        res, dense = dec.kv_pages()
        assert dense == 4 * 2 * 1 and res == dense          # 32 tokens = one page per (layer,row) either way
        dec.prefill(pr)
        assert [dec.kv_len(l) for l in range(4)] == [16] * 4
        total = 16 * 4
        for k in range(16):
            t = 16 + k
            act = skd.skd_active_layers(t, cfg)
            for l in act:
                assert dec.kv_len(l) == t                    # every earlier key exists: nothing to recompute
            dec.decode_step(t, pr[:, k])
            total += len(act)
            assert sum(dec.kv_len(l) for l in range(4)) == total
    cfg2 = skd.make_config(S.TINY, 2, 32, 64, 1, 2, page_tokens=32)   # bottom layers stop after the prompt
    with skd.Decoder(cfg2, w) as dec:
        res, dense = dec.kv_pages()
        assert dense == 4 * 2 * 2 and res == 2 * (1 + 1 + 2 + 2)


def test_call_order_and_range_errors():
    w = bf16_weights(S.TINY, 0)
    cfg = skd.make_config(S.TINY, 2, 16, 32, 2, 4)
    pr = S.make_prompts(2, 16, S.TINY.V, 1)
    tok = np.array([1, 2], np.int32)
    with skd.Decoder(cfg, w) as dec:
        assert dec.decode_step_rc(16, tok) == skd.ERR_ORDER          # no prefill yet
        assert dec._lib.skd_logits_argmax(dec._h, None, None) == skd.ERR_ORDER
        bad = pr.copy()
        bad[0, 3] = S.TINY.V
        assert dec.prefill_rc(bad) == skd.ERR_RANGE
        m = np.ones((2, 16), np.uint8)
        m[0, 5] = 0                                                   # hole: not left padding
        assert dec.prefill_rc(pr, m) == skd.ERR_SHAPE
        m = np.ones((2, 16), np.uint8)
        m[1] = 0                                                      # empty row
        assert dec.prefill_rc(pr, m) == skd.ERR_SHAPE
        dec.prefill(pr)
        assert dec.decode_step_rc(17, tok) == skd.ERR_ORDER          # wrong position
        assert dec.decode_step_rc(16, None) == skd.ERR_ORDER         # no argmax to continue from
        assert dec.decode_step_rc(16, np.array([1, -1], np.int32)) == skd.ERR_RANGE
        assert dec.decode_step_rc(32, tok) == skd.ERR_RANGE          # t >= N
        dec.decode_step(16, tok)
        assert dec.decode_step_rc(16, tok) == skd.ERR_ORDER          # same column twice
        dec.logits_argmax()
        dec.decode_step(17, None)
        # a second prefill restarts the generation
        dec.prefill(pr)
        assert [dec.kv_len(l) for l in range(4)] == [16] * 4
        dec.decode_step(16, tok)


def test_device_io_mode_matches_host_io():
    import torch
    w = bf16_weights(S.TINY, 0)
    pr = S.make_prompts(2, 16, S.TINY.V, 1)
    tape = S.make_token_tape(2, 16, S.TINY.V, 9)
    host = run_hip(S.TINY, w, pr, 16, 32, 2, 4, tape=tape, dtype=skd.BF16)
    cfg = skd.make_config(S.TINY, 2, 16, 32, 2, 4, io_on_device=1)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        pr_dev = torch.from_numpy(np.ascontiguousarray(pr.T)).cuda()           # [P][B]
        tape_dev = torch.from_numpy(tape).cuda()
        logits = torch.zeros(17, 2, S.TINY.V, dtype=torch.float32, device="cuda")
        toks = torch.zeros(17, 2, dtype=torch.int32, device="cuda")
        stream.synchronize()
        with skd.Decoder(cfg, w, stream=stream.cuda_stream) as dec:
            dec.prefill(pr_dev)
            dec.logits_argmax_device(toks[0], logits[0])
            for k in range(16):
                dec.decode_step(16 + k, tape_dev[k])
                dec.logits_argmax_device(toks[k + 1], logits[k + 1])
            dec.synchronize()
        np.testing.assert_array_equal(logits.cpu().numpy(), host["logits"])
        np.testing.assert_array_equal(toks.cpu().numpy(), host["logits"].argmax(-1))


@pytest.mark.usefixtures("narrow_columns")
@pytest.mark.parametrize("dtype,tol", [(skd.FP32, FP32_TOL), (skd.BF16, BF16_TOL)])
@pytest.mark.parametrize("warm", [0, 1])
def test_custom_monotone_schedule_table(dtype, tol, warm):
    # Section 2.3 / Section 5: other decay functions (power law here) and decay that already starts inside the
    # prompt.  The library takes the per-position layer counts; the oracle is driven with the same layer sets.
    shape = MID64
    w = S.make_weights(shape, 11)
    if dtype == skd.BF16:
        w = S.weights_to_bf16_values(w)
    B, P, N = 3, 12, 44
    table = []
    for i in range(N):
        n = shape.L if i < 8 else max(1 + warm, int(round(shape.L * (i - 7) ** -0.55)))
        table.append(min(n, table[-1]) if table else n)
    assert table[P - 1] < shape.L and table[-1] == 1 + warm and sorted(table, reverse=True) == table
    tok = S.make_prompts(B, N, shape.V, 12)
    cfg = skd.make_config(shape, B, P, N, 1 + warm, shape.L, warm, dtype)
    ref_dec = O.Decoder(shape, w, B, N)
    with skd.Decoder(cfg, w, n_table=table) as dec:
        sets = [dec.active_layers(i) for i in range(N)]
        for i, A in enumerate(sets):
            assert len(A) == table[i] and A[:warm] == list(range(warm)) and A[warm:] == list(range(shape.L - (table[i] - warm), shape.L))
        dec.prefill(tok[:, :P])
        for i in range(P):
            ref, _ = ref_dec.column(i, tok[:, i], sets[i], want_logits=(i == P - 1))
        errs = []
        for i in range(P - 1, N):
            if i >= P:
                dec.decode_step(i, tok[:, i])
                ref, _ = ref_dec.column(i, tok[:, i], sets[i])
            _, got = dec.logits_argmax()
            errs.append(np.abs(got - ref).max() / (ref.max() - ref.min()))
        assert [dec.kv_len(l) for l in range(shape.L)] == [ref_dec.kv_len(l) for l in range(shape.L)]
        assert sum(dec.kv_len(l) for l in range(shape.L)) == sum(table)
    ref_dec.close()
    assert max(errs) <= tol, errs


@pytest.mark.parametrize("dtype", [skd.FP32, skd.BF16])
def test_sampling_head_matches_oracle(dtype):
    # Temperature / top-p sampling (Section 3.2).  The HIP sampler and the oracle's sampler are given the same
    # logits (the HIP path's own, read back) and the same uniform numbers; tokens must agree wherever the
    # oracle's decision margins are above fp32 rounding.  Then greedy-free generation continues from the samples.
    shape = S.TINY
    w = S.make_weights(shape, 0)
    if dtype == skd.BF16:
        w = S.weights_to_bf16_values(w)
    B, P, N = 2, 16, 32
    pr = S.make_prompts(B, P, shape.V, 1)
    cfg = skd.make_config(shape, B, P, N, 2, 4, dtype=dtype)
    rng = np.random.default_rng(5)
    checked = 0
    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr)
        for temperature, top_p in ((0.3, 0.7), (1.0, 0.9), (2.0, 1.0), (0.05, 0.5)):
            for _ in range(25):
                u = rng.random(B).astype(np.float32)
                tok, lg = dec.logits_sample(u, temperature, top_p)
                _, lg2 = dec.logits_argmax()
                np.testing.assert_array_equal(lg, lg2)                       # same logits as the argmax head
                for b in range(B):
                    ref, m_set, m_run = O.op_sample(lg[b], temperature, top_p, float(u[b]))
                    if m_set > 1e-5 and m_run > 1e-5:
                        assert tok[b] == ref, (temperature, top_p, u[b], m_set, m_run)
                        checked += 1
        assert checked > 180
        # invalid arguments
        assert dec.logits_sample_rc(np.array([0.5, 1.0], np.float32), 0.3, 0.7)[0] == skd.ERR_RANGE
        assert dec.logits_sample_rc(np.array([0.5, 0.5], np.float32), 0.0, 0.7)[0] == skd.ERR_RANGE
        assert dec.logits_sample_rc(np.array([0.5, 0.5], np.float32), 0.3, 1.5)[0] == skd.ERR_RANGE
        # free-running from sampled tokens: the next column's input is the sample
        u = rng.random(B).astype(np.float32)
        tok, _ = dec.logits_sample(u, 0.3, 0.7)
        dec.decode_step(P, None)
        _, lg_free = dec.logits_argmax()
        dec.rewind(P)
        dec.decode_step(P, tok)
        _, lg_forced = dec.logits_argmax()
        np.testing.assert_array_equal(lg_free, lg_forced)


def test_sampling_head_full_vocab_distribution():
    # vocabulary 50272 (49.1 tokens per thread, ragged tail): frequencies over a grid of uniform numbers follow the
    # renormalised nucleus probabilities, and every sample lies in the nucleus
    shape = S.ModelShape(L=1, d=128, H=2, f=128, V=50272, max_pos=8)
    w = S.make_weights(shape, 3)
    g = np.random.Generator(np.random.Philox(key=[3, 99]))
    # an untied LM head with a wider spread, so that the nucleus at temperature 0.3 is a few hundred tokens
    w["lm_head"] = (g.standard_normal(size=(shape.V, shape.d), dtype=np.float32) * np.float32(0.09))
    w = S.weights_to_bf16_values(w)
    B, P, N = 64, 2, 4
    pr = np.tile(S.make_prompts(1, P, shape.V, 4), (B, 1))   # identical rows: identical logits in every row
    cfg = skd.make_config(shape, B, P, N, 1, 1, dtype=skd.BF16)
    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr)
        toks = []
        for r in range(16):
            u = ((np.arange(B) + r * B + 0.5) / (16 * B)).astype(np.float32)
            tok, lg = dec.logits_sample(u, 0.3, 0.7, want_logits=(r == 0))
            if r == 0:
                logits = lg[0].astype(np.float64)
                assert np.abs(lg - lg[0]).max() == 0
            toks.append(tok)
    toks = np.concatenate(toks)
    p = np.exp((logits - logits.max()) / 0.3)
    p /= p.sum()
    order = np.argsort(-p, kind="stable")
    k = int(np.searchsorted(np.cumsum(p[order]), 0.7, side="left")) + 1
    nucleus = order[:k]
    assert 20 < k < 20000
    assert set(toks.tolist()) <= set(nucleus.tolist())
    mass = p[nucleus].sum()
    top = nucleus[:5]
    for i in top:
        assert abs((toks == i).mean() - p[i] / mass) < 2.5 / len(toks) + 1e-3


def test_sampling_head_full_vocab_both_paths():
    # vocabulary 50272, rows with different logits.  After the exponent rounds of the threshold search the tokens
    # that can still be in the nucleus are few at low temperature (one wave then finishes the row alone on the
    # compacted candidates) and thousands at high temperature or top-p 1 (the whole workgroup searches on).  Both
    # paths against the oracle's sampler on the same logits and uniform numbers.
    shape = S.ModelShape(L=1, d=128, H=2, f=128, V=50272, max_pos=8)
    w = S.make_weights(shape, 5)
    g = np.random.Generator(np.random.Philox(key=[5, 99]))
    w["lm_head"] = (g.standard_normal(size=(shape.V, shape.d), dtype=np.float32) * np.float32(0.09))
    w = S.weights_to_bf16_values(w)
    B, P, N = 8, 2, 4
    pr = S.make_prompts(B, P, shape.V, 6)
    cfg = skd.make_config(shape, B, P, N, 1, 1, dtype=skd.BF16)
    rng = np.random.default_rng(7)

    def candidates(z, temperature, top_p):
        # tokens at or above the largest power of two whose upper set reaches the target mass
        pz = np.exp((z - z.max()) / temperature)
        for e in range(0, -127, -1):
            if pz[pz >= 2.0 ** e].sum() >= top_p * pz.sum():
                return int((pz >= 2.0 ** e).sum())
        return z.size

    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr)
        _, lg = dec.logits_argmax()
        for temperature, top_p, few in ((0.3, 0.7, True), (0.2, 0.9, True), (0.5, 0.7, False), (3.0, 0.7, False),
                                        (1.0, 1.0, False)):
            cand = np.array([candidates(lg[b].astype(np.float64), temperature, top_p) for b in range(B)])
            assert (cand <= 600).all() if few else (cand >= 2000).all(), (temperature, top_p, cand)   # limit: 1024
            checked = 0
            for _ in range(6):
                u = rng.random(B).astype(np.float32)
                tok, _ = dec.logits_sample(u, temperature, top_p, want_logits=False)
                for b in range(B):
                    ref, m_set, m_run = O.op_sample(lg[b], temperature, top_p, float(u[b]))
                    if m_set > 1e-5 and m_run > 1e-5:
                        assert tok[b] == ref, (temperature, top_p, b, u[b], m_set, m_run)
                        checked += 1
            if temperature <= 0.5:
                assert checked >= 24, (temperature, top_p, checked)
            else:
                # nearly flat over tens of thousands of tokens: the oracle's decision margins are below fp32 rounding
                # almost everywhere, so check membership instead: every sample lies in the nucleus
                for b in range(B):
                    pz = np.exp((lg[b].astype(np.float64) - lg[b].max()) / temperature)
                    srt = np.sort(pz)[::-1]
                    k = int(np.searchsorted(np.cumsum(srt), top_p * pz.sum(), side="left"))
                    assert pz[tok[b]] >= srt[min(k, srt.size - 1)] * (1 - 1e-4), (temperature, top_p, b)


@pytest.mark.usefixtures("narrow_columns")
@pytest.mark.parametrize("dtype,tol", [(skd.FP32, FP32_TOL), (skd.BF16, BF16_TOL)])
def test_minimal_sizes(dtype, tol):
    # one row, one prompt token, two decode steps; and a prompt that ends exactly on a page boundary
    w = S.make_weights(MID64, 13)
    if dtype == skd.BF16:
        w = S.weights_to_bf16_values(w)
    compare(MID64, w, S.make_prompts(1, 1, MID64.V, 14), 1, 3, 1, 5, tol, dtype=dtype)
    compare(MID64, w, S.make_prompts(2, 32, MID64.V, 15), 32, 66, 2, 5, tol, dtype=dtype, page_tokens=32)


def test_rewind_regenerates_identically():
    w = bf16_weights(S.TINY, 0)
    pr = S.make_prompts(2, 16, S.TINY.V, 1)
    tape = S.make_token_tape(2, 16, S.TINY.V, 17)
    cfg = skd.make_config(S.TINY, 2, 16, 32, 2, 4)
    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr)
        first = []
        for k in range(10):
            dec.decode_step(16 + k, tape[k])
            first.append(dec.logits_argmax()[1])
        lens = [dec.kv_len(l) for l in range(4)]
        assert dec._lib.skd_rewind(dec._h, 27) == skd.ERR_RANGE      # beyond the current position
        assert dec._lib.skd_rewind(dec._h, 15) == skd.ERR_RANGE      # inside the prompt
        dec.rewind(20)
        assert [dec.kv_len(l) for l in range(4)] == [min(x, 20) for x in lens]
        assert dec._lib.skd_logits_argmax(dec._h, None, None) == skd.ERR_ORDER   # no hidden state after a rewind
        for k in range(4, 10):
            dec.decode_step(16 + k, tape[k])
            np.testing.assert_array_equal(dec.logits_argmax()[1], first[k])
        assert [dec.kv_len(l) for l in range(4)] == lens


@pytest.mark.usefixtures("narrow_columns")
@pytest.mark.parametrize("shape,batched", [(MID, "1"), (MID, "0"), (MID64, "0")])
def test_kv_page_contents_match_oracle(shape, batched):
    # every key and value the cache holds after prefill + decode against the oracle's cache, element by element:
    # covers the page addressing, the 32-key block boundaries (columns 32, 64, 96), page boundaries (page = 32
    # tokens here) and the rule that a layer holds exactly the columns at which it ran (Section 2.2)
    import os
    w = bf16_weights(shape, 6)
    B, P, N = 3, 20, 100
    pr = S.make_prompts(B, P, shape.V, 7)
    mask = S.make_ragged_mask(B, P, 3, 20, seed=8)
    mask[1] = 1
    tape = S.make_token_tape(B, N - P, shape.V, 9)
    n_min, n_max = 1, shape.L
    odec = O.Decoder(shape, w, B, N)
    for i in range(P):
        odec.column(i, pr[:, i], list(range(shape.L)), mask[:, i], want_logits=False)
    os.environ["SKD_PREFILL_BATCHED"] = batched
    try:
        cfg = skd.make_config(shape, B, P, N, n_min, n_max, page_tokens=32)
        with skd.Decoder(cfg, w) as dec:
            dec.prefill(pr, mask)
            for k in range(N - P):
                t = P + k
                odec.column(t, tape[k], O.active_layers(t, P, N, n_min, n_max, 0, shape.L), want_logits=False)
                dec.decode_step(t, tape[k])
            start = (mask == 0).sum(axis=1)
            for l in range(shape.L):
                assert dec.kv_len(l) == odec.kv_len(l)
                for b in range(B):
                    K, V = dec.kv_read(l, b)
                    Ko, Vo = odec.kv_read(l, b)
                    assert K.shape == Ko.shape and K.shape[0] == dec.kv_len(l)
                    sl = slice(int(start[b]), None)      # padded columns are never read: not compared
                    scale = max(np.abs(Ko[sl]).max(), np.abs(Vo[sl]).max())
                    assert np.abs(K[sl] - Ko[sl]).max() <= 2e-2 * scale, (l, b)
                    assert np.abs(V[sl] - Vo[sl]).max() <= 2e-2 * scale, (l, b)
    finally:
        os.environ.pop("SKD_PREFILL_BATCHED", None)
        odec.close()


def test_prompt_tiles_in_xcd_order_page_contents():
    # 1024 prompt rows (16 sequences x 64 positions) at d = 512, ffn = 1536: the tiled prompt GEMM launches
    # 6 x 4 (q,k,v and FFN1) and 2 x 4 (output projection, FFN2) workgroups, i.e. grids whose size is a multiple
    # of 8 with 4 activation tiles, which it walks in its XCD-aware order.  Logits per step and every cached key
    # and value against the oracle.
    shape = MID
    B, P, N = 16, 64, 70
    for n_out in (3 * shape.d, shape.d, shape.f):
        gx, gy = n_out // 256, (B * P) // 256
        assert n_out % 256 == 0 and (gx * gy) % 8 == 0 and gy % 4 == 0
    w = bf16_weights(shape, 81)
    pr = S.make_prompts(B, P, shape.V, 82)
    tape = S.make_token_tape(B, N - P, shape.V, 83)
    compare(shape, w, pr, P, N, 1, 3, BF16_TOL, dtype=skd.BF16, page_tokens=32, tape=tape,
            min_decided=0.0)   # near-flat logits at this width: the logit bar and the cache contents are the check
    odec = O.Decoder(shape, w, B, N)
    for i in range(P):
        odec.column(i, pr[:, i], list(range(shape.L)), want_logits=False)
    cfg = skd.make_config(shape, B, P, N, 1, 3, page_tokens=32)
    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr)
        for l in range(shape.L):
            assert dec.kv_len(l) == odec.kv_len(l) == P
            for b in range(B):
                K, V = dec.kv_read(l, b)
                Ko, Vo = odec.kv_read(l, b)
                scale = max(np.abs(Ko).max(), np.abs(Vo).max())
                assert np.abs(K - Ko).max() <= 2e-2 * scale and np.abs(V - Vo).max() <= 2e-2 * scale, (l, b)
    odec.close()


@pytest.mark.parametrize("B", [20, 28])
def test_prompt_tiles_partial_band(B):
    # 1280 and 1792 prompt rows: 5 and 7 activation tiles, i.e. one full band of 4 and a last band of 1 or 3 in the
    # tile order of the prompt GEMM, with grid sizes (30, 10; 42, 14) that are no multiple of the 8 XCDs.  Every tile
    # must still be computed exactly once: logits per step and every cached key and value against the oracle.
    shape = MID
    P, N = 64, 67
    assert (B * P) % 256 == 0 and ((B * P) // 256) % 4 != 0
    w = bf16_weights(shape, 71)
    pr = S.make_prompts(B, P, shape.V, 72)
    tape = S.make_token_tape(B, N - P, shape.V, 73)
    compare(shape, w, pr, P, N, 1, 3, BF16_TOL, dtype=skd.BF16, page_tokens=32, tape=tape, min_decided=0.0)
    odec = O.Decoder(shape, w, B, N)
    for i in range(P):
        odec.column(i, pr[:, i], list(range(shape.L)), want_logits=False)
    cfg = skd.make_config(shape, B, P, N, 1, 3, page_tokens=32)
    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr)
        for l in range(shape.L):
            for b in range(B):
                K, V = dec.kv_read(l, b)
                Ko, Vo = odec.kv_read(l, b)
                scale = max(np.abs(Ko).max(), np.abs(Vo).max())
                assert np.abs(K - Ko).max() <= 2e-2 * scale and np.abs(V - Vo).max() <= 2e-2 * scale, (l, b)
    odec.close()


def test_prompt_tiles_ragged_head_dim_64():
    # The tiled prompt path on a ragged batch with 64-wide heads: 22 sequences whose real positions, padded to whole
    # 16-row tiles, make exactly 1024 rows (grids 6 x 4, 2 x 4, 4 x 4: the XCD-aware order).  Lengths leave 1, 2 and 3
    # valid positions in the last group of four (values are filed four positions at a time), sequences of 1 and 3
    # tiles put the tile pairs of the prompt attention across sequence boundaries.  Logits per step and every cached
    # key and value of the real positions against the oracle.
    shape = S.ModelShape(L=2, d=512, H=8, f=1024, V=1000, max_pos=96)
    lens = [61, 47, 33, 18, 64, 50, 35, 3, 62, 21, 64, 49, 31, 17, 63, 45, 2, 29, 57, 13, 64, 46]
    B, P, N = len(lens), 64, 68
    assert sum((n + 15) // 16 * 16 for n in lens) == 1024
    assert {n % 4 for n in lens} == {0, 1, 2, 3}
    mask = np.zeros((B, P), dtype=np.uint8)
    for b, n in enumerate(lens):
        mask[b, P - n:] = 1
    w = bf16_weights(shape, 61)
    pr = S.make_prompts(B, P, shape.V, 62)
    tape = S.make_token_tape(B, N - P, shape.V, 63)
    compare(shape, w, pr, P, N, 1, 2, BF16_TOL, mask=mask, dtype=skd.BF16, page_tokens=32, tape=tape, min_decided=0.0)
    odec = O.Decoder(shape, w, B, N)
    for i in range(P):
        odec.column(i, pr[:, i], list(range(shape.L)), mask[:, i], want_logits=False)
    cfg = skd.make_config(shape, B, P, N, 1, 2, page_tokens=32)
    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr, mask)
        for l in range(shape.L):
            assert dec.kv_len(l) == odec.kv_len(l) == P
            for b in range(B):
                K, V = dec.kv_read(l, b)
                Ko, Vo = odec.kv_read(l, b)
                sl = slice(P - lens[b], P)                   # padded columns are never read: not compared
                scale = max(np.abs(Ko[sl]).max(), np.abs(Vo[sl]).max())
                assert np.abs(K[sl] - Ko[sl]).max() <= 2e-2 * scale, (l, b)
                assert np.abs(V[sl] - Vo[sl]).max() <= 2e-2 * scale, (l, b)
    odec.close()


@pytest.mark.parametrize("env", [
    {"SKD_R_QKV": "1", "SKD_R_FFN1": "2", "SKD_R_HEAD": "3", "SKD_R_OUT": "1", "SKD_R_FFN2": "2"},
    {"SKD_U_QKV": "2", "SKD_U_FFN1": "4", "SKD_U_HEAD": "2", "SKD_U_OUT": "2", "SKD_U_FFN2": "4"},
    {"SKD_W_QKV": "4", "SKD_W_FFN1": "4", "SKD_W_HEAD": "4", "SKD_W_OUT": "4", "SKD_W_FFN2": "4"},
    {"SKD_S_OUT": "1", "SKD_S_FFN2": "8", "SKD_R_OUT": "4", "SKD_R_FFN2": "4"},
    {"SKD_ATTN_SPLITS": "1"}, {"SKD_ATTN_SPLITS": "4"}, {"SKD_PREFILL_BATCHED": "0", "SKD_ATTN_SPLITS": "8"},
    {"SKD_ATTN_WAVES": "4", "SKD_ATTN_SPLITS": "2"}, {"SKD_ATTN_WAVES": "8", "SKD_ATTN_SPLITS": "1"},
    {"SKD_ATTN_WAVES": "16", "SKD_ATTN_SPLITS": "3"}, {"SKD_ATTN_WAVES": "2"},
    {"SKD_ATTN_WAVES": "1"}, {"SKD_ATTN_WAVES": "1", "SKD_ATTN_SPLITS": "2"},
])
def test_launch_shape_overrides(env):
    # every launch shape the planner can choose (tile rows per workgroup, k-steps per buffer, waves, split-K,
    # attention waves and splits) computes the same function: forced through the environment overrides on one workload
    import os
    shape = MID
    w = bf16_weights(shape, 51)
    B, P, N = 20, 37, 70
    pr = S.make_prompts(B, P, shape.V, 52)
    mask = S.make_ragged_mask(B, P, 5, P, seed=53)
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        compare(shape, w, pr, P, N, 1, 3, BF16_TOL, mask=mask, dtype=skd.BF16, page_tokens=32)
    finally:
        for k, v in old.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v


@pytest.mark.parametrize("dtype,B", [(skd.FP32, 5), (skd.BF16, 5), (skd.BF16, 128)])
@pytest.mark.parametrize("far", [False, True])
def test_argmax_exact_ties_take_lowest_index(dtype, far, B):
    # greedy head: the LOWEST index attaining the maximum.  An untied LM head with duplicated rows makes every
    # logit tie exactly with its twin: 500 rows away (another workgroup of the LM-head projection, merged by the
    # final reduction) or in the next row (same 16-row tile, merged inside the projection's epilogue).  Batch 128 runs
    # the LM head on the wave-specialised kernel, which keeps one summation order for all vocabulary rows.
    shape = S.TINY
    w = S.make_weights(shape, 0)
    lm = np.array(w["tok_emb"], copy=True)
    if far:
        lm[shape.V // 2:] = lm[:shape.V // 2]
    else:
        lm[1::2] = lm[0::2]
    w["lm_head"] = lm
    if dtype == skd.BF16:
        w = S.weights_to_bf16_values(w)
    P, N = 6, 12
    pr = S.make_prompts(B, P, shape.V, 44)
    tape = S.make_token_tape(B, N - P, shape.V, 45)
    cfg = skd.make_config(shape, B, P, N, 2, 4, dtype=dtype)
    odec = O.Decoder(shape, w, B, N)
    for i in range(P):
        _, otok = odec.column(i, pr[:, i], list(range(shape.L)), want_logits=(i == P - 1))
    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr)
        for k in range(N - P + 1):
            tok, lg = dec.logits_argmax()
            twin = tok + shape.V // 2 if far else tok + 1
            assert (tok < shape.V // 2).all() if far else (tok % 2 == 0).all()
            rows = np.arange(B)
            np.testing.assert_array_equal(lg[rows, tok], lg[rows, twin])        # the tie is exact
            np.testing.assert_array_equal(lg[rows, tok], lg.max(axis=1))
            np.testing.assert_array_equal(tok, lg.argmax(axis=1))
            assert (otok < shape.V // 2).all() if far else (otok % 2 == 0).all()  # the oracle breaks ties the same way
            if k == N - P:
                break
            dec.decode_step(P + k, tape[k])
            _, otok = odec.column(P + k, tape[k], O.active_layers(P + k, P, N, 2, 4, 0, shape.L))
    odec.close()


def test_one_wave_attention_head_dim_64():
    # one wave per (row, head) is what batches of 128 rows x 32 heads get; forced here on 64-wide heads (one element
    # of the head per thread; 128-wide heads, two per thread, are covered by the launch-shape walk above)
    import os
    w = bf16_weights(MID64, 95)
    pr = S.make_prompts(7, 45, MID64.V, 96)
    mask = S.make_ragged_mask(7, 45, 3, 45, seed=97)
    os.environ["SKD_ATTN_WAVES"] = "1"
    try:
        compare(MID64, w, pr, 45, 110, 2, 5, BF16_TOL, mask=mask, dtype=skd.BF16, page_tokens=32, min_decided=0.0)
    finally:
        os.environ.pop("SKD_ATTN_WAVES", None)


def test_unlaunchable_override_is_refused_at_create():
    # a launch-shape override the kernels cannot run (K = 1536 = 48 k-steps does not split 7 ways) is caught when the
    # state is created, not in the middle of a column: skd_create returns SKD_ERR_SHAPE and no state exists
    import os
    w = bf16_weights(MID, 2)
    cfg = skd.make_config(MID, 2, 4, 8, 1, 3, dtype=skd.BF16)
    os.environ["SKD_S_FFN2"] = "7"
    try:
        with pytest.raises(skd.SkdError) as e:
            skd.Decoder(cfg, w)
        assert e.value.code == skd.ERR_SHAPE
    finally:
        os.environ.pop("SKD_S_FFN2", None)
    with skd.Decoder(cfg, w) as dec:                      # the same configuration without the override is fine
        dec.prefill(S.make_prompts(2, 4, MID.V, 3))


def test_vocabulary_above_sampler_limit():
    # the sampling head keeps a row of probabilities in registers: vocabularies above 65536 are refused with
    # SKD_ERR_SHAPE, while the LM head and greedy argmax have no such limit
    shape = S.ModelShape(L=1, d=128, H=2, f=64, V=70001, max_pos=8)
    w = bf16_weights(shape, 41)
    pr = S.make_prompts(2, 2, shape.V, 42)
    cfg = skd.make_config(shape, 2, 2, 4, 1, 1, dtype=skd.BF16)
    ref = O.generate(shape, w, pr, 2, 4, 1, 1, steps=0)
    with skd.Decoder(cfg, w) as dec:
        dec.prefill(pr, None)
        rc, _, _ = dec.logits_sample_rc(np.array([0.5, 0.5], dtype=np.float32), 0.3, 0.7)
        assert rc == skd.ERR_SHAPE
        tok, lg = dec.logits_argmax()
        assert rel_err(lg[None], ref["logits"][:1]).max() <= BF16_TOL


@pytest.mark.parametrize("d", [8192, 16384])
def test_wide_model_bf16(d):
    # d_model 8192 and the maximum, 16384: the row kernels (embedding, split-K reduce, LayerNorm) hold two and four
    # register chunks per thread, the projections run 256 and 512 k-steps, 64 and 128 heads
    shape = S.ModelShape(L=1, d=d, H=d // 128, f=128, V=100, max_pos=16)
    w = bf16_weights(shape, 31)
    pr = S.make_prompts(2, 3, shape.V, 32)
    compare(shape, w, pr, 3, 6, 1, 1, BF16_TOL, dtype=skd.BF16, min_decided=0.0)


@pytest.mark.usefixtures("narrow_columns")
@pytest.mark.parametrize("seed", range(8))
def test_random_small_configurations(seed):
    # seeded draw over the knobs that change code paths: head size, batch tile count, prompt length against the
    # 16-position tiles and 32-key blocks, page size, warm-up layers, ragged left padding, schedule window
    g = np.random.Generator(np.random.Philox(key=[77, seed]))
    dh = int(g.choice([64, 128]))
    H = int(g.choice([2, 3, 4]))
    d = dh * H
    L = int(g.integers(2, 6))
    shape = S.ModelShape(L=L, d=d, H=H, f=int(g.choice([256, 512, 768])), V=int(g.integers(300, 1200)), max_pos=256)
    B = int(g.choice([1, 2, 5, 18, 35]))
    P = int(g.integers(1, 80))
    T = int(g.integers(2, 50))
    n_max = int(g.integers(1, L + 1))
    n_min = int(g.integers(1, n_max + 1))
    warm = int(g.integers(0, n_min + 1)) if g.random() < 0.4 else 0
    page = int(g.choice([0, 32, 64, 128]))
    w = bf16_weights(shape, 100 + seed)
    pr = S.make_prompts(B, P, shape.V, 200 + seed)
    mask = None
    if g.random() < 0.6:
        mask = S.make_ragged_mask(B, P, 1, P, seed=300 + seed)
    tape = S.make_token_tape(B, T, shape.V, 400 + seed)
    compare(shape, w, pr, P, P + T, n_min, n_max, BF16_TOL, warmup=warm, mask=mask, dtype=skd.BF16, page_tokens=page,
            tape=tape, min_decided=0.0)     # tiny random models may have near-flat logits: the logit bar is the check


def test_batched_prefill_matches_column_prefill():
    # the whole-prompt path (row-chunked projections + causal prompt attention) against the column-by-column path:
    # same cache contents up to bf16 rounding of differently ordered sums, same logits within the parity tolerance
    import os
    shape = MID
    w = bf16_weights(shape, 2)
    B, P, N = 5, 40, 60
    pr = S.make_prompts(B, P, shape.V, 3)
    mask = S.make_ragged_mask(B, P, 1, 40, seed=4)
    mask[0] = 1
    tape = S.make_token_tape(B, N - P, shape.V, 5)
    outs = {}
    for mode in ("1", "0"):
        os.environ["SKD_PREFILL_BATCHED"] = mode
        try:
            cfg = skd.make_config(shape, B, P, N, 1, 3, page_tokens=32)
            with skd.Decoder(cfg, w) as dec:
                dec.prefill(pr, mask)
                lg = [dec.logits_argmax()[1]]
                kv = [dec.kv_read(l, b) for l in range(shape.L) for b in range(B)]
                for k in range(N - P):
                    dec.decode_step(P + k, tape[k])
                    lg.append(dec.logits_argmax()[1])
                outs[mode] = (np.stack(lg), kv, [dec.kv_len(l) for l in range(shape.L)])
        finally:
            os.environ.pop("SKD_PREFILL_BATCHED", None)
    a, b = outs["1"], outs["0"]
    assert a[2] == b[2]
    rng = b[0].max() - b[0].min()
    assert np.abs(a[0] - b[0]).max() / rng < 5e-3
    start = (mask == 0).sum(axis=1)
    for i, ((ka, va), (kb, vb)) in enumerate(zip(a[1], b[1])):
        r = i % B
        sl = slice(int(start[r]), P)                      # padded columns are never read: not compared
        np.testing.assert_allclose(ka[sl], kb[sl], rtol=2e-2, atol=2e-2)
        np.testing.assert_allclose(va[sl], vb[sl], rtol=2e-2, atol=2e-2)


@pytest.mark.parametrize("f", [32, 64, 96, 288])
def test_prompt_tiles_short_and_odd_k(f):
    # the tiled prompt GEMM keeps a ring of k-steps in flight: FFN widths of 1, 2, 3 and 9 k-steps exercise a ring
    # that never fills, fills exactly, and wraps at an odd count (FFN2 runs on the tile kernel with K = f; FFN1, whose
    # N = f does not tile, falls back to the weight-streaming kernel)
    shape = S.ModelShape(L=2, d=256, H=4, f=f, V=500, max_pos=64)
    w = bf16_weights(shape, 61 + f)
    B, P, N = 6, 33, 40
    pr = S.make_prompts(B, P, shape.V, 62)
    mask = S.make_ragged_mask(B, P, 7, P, seed=63)
    compare(shape, w, pr, P, N, 1, 2, BF16_TOL, mask=mask, dtype=skd.BF16, page_tokens=32, min_decided=0.0)


def test_batched_prefill_is_deterministic():
    # the prompt pass (tile GEMM with its ring of in-flight operand stages, prompt attention, row kernels) has no
    # atomics and a fixed summation order: three runs give bit-identical logits and cache contents
    shape = MID
    w = bf16_weights(shape, 71)
    B, P, N = 9, 48, 52
    pr = S.make_prompts(B, P, shape.V, 72)
    mask = S.make_ragged_mask(B, P, 30, P, seed=73)
    runs = []
    for _ in range(3):
        cfg = skd.make_config(shape, B, P, N, 1, 3, page_tokens=32)
        with skd.Decoder(cfg, w) as dec:
            dec.prefill(pr, mask)
            lg = dec.logits_argmax()[1].copy()
            kv = [dec.kv_read(l, b) for l in range(shape.L) for b in (0, B - 1)]
            runs.append((lg, kv))
    for lg, kv in runs[1:]:
        assert np.array_equal(lg, runs[0][0])
        for (k1, v1), (k0, v0) in zip(kv, runs[0][1]):
            assert np.array_equal(k1, k0) and np.array_equal(v1, v0)
