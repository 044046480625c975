"""Decode columns of narrow models in one launch (a team of workgroups per XCD) against the separate decode kernels
(SKD_TEAM=0): the same sums in the same order, so the same bits in logits, hidden rows, keys and values, whatever the size of
the team that formed."""
import os
import re
import subprocess

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import _build, skd


def columns(shape, w, B, P, N, n_min, warmup, mask, tokens, tape, env, page_tokens=0):
    os.environ.update(env)
    try:
        with skd.Decoder(skd.make_config(shape, B, P, N, n_min, shape.L, warmup, page_tokens=page_tokens), w) as dec:
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


def compare(L, d, H, f, B, P, steps, warmup=0, shortest=0, env=None, n_min=1, page_tokens=0):
    shape = S.ModelShape(L=L, d=d, H=H, f=f, V=301, max_pos=P + steps)
    w = S.weights_to_bf16_values(S.make_weights(shape, 3))
    tokens, tape = S.make_prompts(B, P, shape.V, 4), S.make_token_tape(B, steps, shape.V, 5)
    mask = S.make_ragged_mask(B, P, shortest, P, seed=6) if shortest else None
    run = lambda e: columns(shape, w, B, P, P + steps, max(n_min, warmup), warmup, mask, tokens, tape, e, page_tokens)  # noqa: E731
    got, want = run(env or {}), run({"SKD_TEAM": "0"})
    for g, r in zip((*got[:2], *got[2]), (*want[:2], *want[2])):
        np.testing.assert_array_equal(g, r)


@pytest.mark.gpu
# every width compiled; fewer rows than XCDs, one more, a full tile each; ffn that fills the last k-steps of the waves partly
@pytest.mark.parametrize("d,H,f,B", [(64, 1, 32, 3), (128, 2, 96, 9), (192, 3, 544, 1), (256, 4, 1024, 2), (320, 5, 64, 17),
                                     (384, 6, 1024, 11), (448, 7, 160, 77), (512, 8, 2048, 16), (128, 1, 256, 8), (256, 2, 2048, 5),
                                     (384, 3, 512, 128), (512, 4, 1536, 33),
                                     # sums of the four-wave projections, in rotated order and not (k-steps of a part
                                     # no multiple of four, an odd number of them)
                                     (64, 1, 1056, 66), (128, 2, 512, 96), (256, 4, 1024, 97), (320, 5, 992, 128), (512, 8, 2048, 128),
                                     # one to four rows, and two k-steps in a row with a part that they do not divide
                                     (512, 8, 1984, 4), (256, 4, 960, 3), (448, 7, 1600, 16), (512, 4, 2016, 64)])
def test_widths(d, H, f, B):
    compare(3, d, H, f, B, 35, 4, warmup=1, shortest=3 if B > 2 else 0)


@pytest.mark.gpu
# keys: none cached for some rows' blocks, the edges of a block and a page, one block per wave and one more, several per
# wave; the keys of a (row, head) pair shared out over two and four workgroups
@pytest.mark.parametrize("d,H,B,P", [(256, 4, 1, 1), (256, 4, 3, 31), (256, 4, 3, 32), (256, 2, 8, 63), (512, 4, 2, 256), (512, 4, 2, 257),
                                     (256, 4, 1, 700), (512, 4, 9, 1100), (384, 6, 16, 900), (256, 4, 128, 130),
                                     (512, 8, 5, 1300), (256, 2, 33, 600), (64, 1, 128, 500), (128, 1, 1, 900)])
def test_contexts(d, H, B, P):
    compare(2, d, H, 256, B, P, 3, shortest=max(1, P // 9) if B > 2 else 0)


@pytest.mark.gpu
def test_route_changes_within_a_generation():
    """128 rows of 64 columns take separate kernels from 600 cached keys on: the state goes on with the same bits."""
    compare(3, 64, 1, 256, 128, 598, 5)


@pytest.mark.gpu
@pytest.mark.parametrize("d,H,B,P", [(64, 1, 128, 1100), (128, 2, 97, 1500), (512, 8, 1, 4500)])
def test_more_keys_than_pay(d, H, B, P):
    compare(2, d, H, 256, B, P, 2, env={"SKD_TEAM": "2"})


@pytest.mark.gpu
@pytest.mark.parametrize("page_tokens", [32, 96, 416])  # 1, 3 and 13 blocks to a page
def test_pages(page_tokens):
    compare(2, 256, 4, 256, 3, 900, 3, shortest=50, page_tokens=page_tokens)


@pytest.mark.gpu
# small teams: several rounds of tiles, of (row, head) pairs and of their keys' shares, several of these to a wave
@pytest.mark.parametrize("members", [1, 2, 5, 15])
@pytest.mark.parametrize("d,H,B,P", [(256, 4, 20, 40), (256, 4, 1, 700), (512, 4, 9, 1100), (512, 8, 16, 600), (256, 2, 66, 300)])
def test_small_teams(members, d, H, B, P):
    compare(3, d, H, 1024, B, P, 4, shortest=5 if B > 2 else 0, env={"SKD_TEAM_WGS": str(members)})


@pytest.mark.gpu
@pytest.mark.parametrize("B,P", [(24, 20), (3, 600)])
def test_two_states_at_once(B, P):
    """Two states on two streams, enqueued in turn without waiting: their teams share the CUs, each finishes its rows."""
    import torch
    T = 30
    shape = S.ModelShape(L=4, d=256, H=4, f=1024, V=301, max_pos=P + T)
    w = S.weights_to_bf16_values(S.make_weights(shape, 8))
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
