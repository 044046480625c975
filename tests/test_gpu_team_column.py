"""Decode columns of narrow models in one launch (a team of workgroups per XCD) against the separate decode kernels
(SKD_TEAM=0).  Same products, other summation orders, rounded to bf16 (8 mantissa bits) between phases: 5e-3 of the logit
range and 2e-2 of the hidden and cached values' range, the bars of the other kernel-against-kernel tests."""
import os
import re
import subprocess

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import _build, skd


def columns(shape, w, B, P, N, n_min, warmup, mask, tokens, tape, env):
    os.environ.update(env)
    try:
        with skd.Decoder(skd.make_config(shape, B, P, N, n_min, shape.L, warmup), w) as dec:
            dec.prefill(tokens, mask)
            logits, hidden = [], []
            for k in range(N - P):
                dec.decode_step(P + k, tape[k])
                hidden.append(dec.read_hidden())
                logits.append(dec.logits_argmax()[1].copy())
            kv = [np.stack(dec.kv_read(l, b)) for l in range(shape.L) for b in sorted({0, B // 2, B - 1})]
        return np.stack(logits), np.stack(hidden), kv
    finally:
        for k in env:
            os.environ.pop(k, None)


def compare(L, d, H, f, B, P, steps, warmup=0, shortest=0, env=None, n_min=1):
    shape = S.ModelShape(L=L, d=d, H=H, f=f, V=301, max_pos=P + steps)
    w = S.weights_to_bf16_values(S.make_weights(shape, 3))
    tokens, tape = S.make_prompts(B, P, shape.V, 4), S.make_token_tape(B, steps, shape.V, 5)
    mask = S.make_ragged_mask(B, P, shortest, P, seed=6) if shortest else None
    run = lambda e: columns(shape, w, B, P, P + steps, max(n_min, warmup), warmup, mask, tokens, tape, e)  # noqa: E731
    got, want = run(env or {}), run({"SKD_TEAM": "0"})
    for g, r, tol in zip(got[:2], want[:2], (5e-3, 2e-2)):
        assert np.abs(g - r).max() <= tol * (r.max() - r.min())
    for g, r in zip(got[2], want[2]):
        np.testing.assert_allclose(g, r, rtol=2e-2, atol=2e-2)
    again = run(env or {})  # the control words are as the first state's launches found theirs; sums in a fixed order
    np.testing.assert_array_equal(got[0], again[0])


@pytest.mark.gpu
# every width compiled; fewer rows than XCDs, one more, a full tile each; ffn that fills the last k-steps of the waves partly
@pytest.mark.parametrize("d,H,f,B", [(64, 1, 32, 3), (128, 2, 96, 9), (192, 3, 544, 1), (256, 4, 1024, 2), (320, 5, 64, 17),
                                     (384, 6, 1024, 11), (448, 7, 160, 77), (512, 8, 2048, 16), (128, 1, 256, 8), (256, 2, 2048, 5),
                                     (384, 3, 512, 128), (512, 4, 1536, 33)])
def test_widths(d, H, f, B):
    compare(3, d, H, f, B, 35, 4, warmup=1, shortest=3 if B > 2 else 0)


@pytest.mark.gpu
# keys: none cached for some rows' blocks, the edges of a block and a page, one block per wave and one more, several per
# wave; the keys of a (row, head) pair shared out over two and four workgroups
@pytest.mark.parametrize("d,H,B,P", [(256, 4, 1, 1), (256, 4, 3, 31), (256, 4, 3, 32), (256, 2, 8, 63), (512, 4, 2, 256), (512, 4, 2, 257),
                                     (256, 4, 1, 700), (512, 4, 9, 1100), (384, 6, 16, 900), (256, 4, 128, 130)])
def test_contexts(d, H, B, P):
    compare(2, d, H, 256, B, P, 3, shortest=max(1, P // 9) if B > 2 else 0)


@pytest.mark.gpu
@pytest.mark.parametrize("members", [1, 2, 5, 15])  # small teams: several rounds of tiles and of (row, head) pairs
def test_small_teams(members):
    compare(3, 256, 4, 1024, 20, 40, 4, shortest=5, env={"SKD_TEAM_WGS": str(members)})


@pytest.mark.gpu
def test_two_states_at_once():
    """Two states on two streams, enqueued in turn without waiting: their teams share the CUs, each finishes its rows."""
    import torch
    shape = S.ModelShape(L=4, d=256, H=4, f=1024, V=301, max_pos=128)
    w = S.weights_to_bf16_values(S.make_weights(shape, 8))
    B, P, T = 24, 20, 30
    tape = torch.from_numpy(S.make_token_tape(B, T, shape.V, 9)).cuda()
    pr = torch.from_numpy(np.ascontiguousarray(S.make_prompts(B, P, shape.V, 10).T)).cuda()
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    decs = [skd.Decoder(skd.make_config(shape, B, P, P + T, 1, 4, dtype=skd.BF16, io_on_device=1), w, stream=s.cuda_stream) for s in streams]
    out = torch.zeros(2, T, B, shape.V, device="cuda")
    for dec in decs:
        dec.prefill(pr)
    torch.cuda.synchronize()

    def steps(which):
        for k in range(T):
            for i in which:
                decs[i].decode_step(P + k, tape[k])
                decs[i].logits_argmax_device(None, out[i, k])
        torch.cuda.synchronize()
    steps((0, 1))
    both = out.cpu().numpy()
    decs[0].rewind(P)
    steps((0,))
    np.testing.assert_array_equal(both[0], both[1])
    np.testing.assert_array_equal(out[0].cpu().numpy(), both[0])
    for dec in decs:
        dec.close()


def test_no_registers_in_memory():
    """The team kernel keeps its vector registers (scalar ones may move to lanes of a vector register)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "--cuda-device-only", "-O3", "-std=c++17", "-Xclang", "-target-feature",
                          "-Xclang", "-packed-fp32-ops", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
                          os.path.join(_build.CSRC, "team_column.hip"), "-o", os.devnull], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found = re.findall(r"(ScratchSize \[bytes/lane\]|VGPRs Spill): (\d+)", res.stderr)
    assert len(found) >= 24 and all(v == "0" for _, v in found), found
