"""A generation of a narrow model beside long prompts on another stream: the prompt tiles hold every CU's LDS, so a step waits until
one of them is done, and no longer."""
import time

import numpy as np
import pytest

from paper_2307_02628_amd import skd

pytestmark = pytest.mark.gpu


class Shape:
    def __init__(self, L, d, H, f, V, max_pos):
        self.L, self.d, self.H, self.f, self.V, self.max_pos = L, d, H, f, V, max_pos


def _state(torch, s, B, P, N, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def n(*size, mean=0.0):
        return torch.empty(*size, device="cuda").normal_(mean, 0.02, generator=g).to(torch.bfloat16)
    w = {"tok_emb": n(s.V, s.d), "pos_emb": n(s.max_pos, s.d), "lnf_g": n(s.d, mean=1.0), "lnf_b": n(s.d)}
    sizes = {"ln1_g": (s.d,), "ln1_b": (s.d,), "wqkv": (3 * s.d, s.d), "bqkv": (3 * s.d,), "wo": (s.d, s.d), "bo": (s.d,),
             "ln2_g": (s.d,), "ln2_b": (s.d,), "w1": (s.f, s.d), "b1": (s.f,), "w2": (s.d, s.f), "b2": (s.d,)}
    for name in skd.PER_LAYER:
        w[name] = [n(*sizes[name]) for _ in range(s.L)]
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    cfg = skd.make_config(s, B, P, N, s.L, s.L, dtype=skd.BF16, io_on_device=1)
    dec = skd.Decoder(cfg, w, location=skd.DEVICE, elem=skd.W_BF16, stream=stream.cuda_stream)
    tokens = torch.randint(0, s.V, (N, B), dtype=torch.int32, device="cuda", generator=g)
    torch.cuda.synchronize()
    return dec, tokens, stream


def test_a_step_waits_for_one_tile():
    """8192 rows of 4096: two thirds of a prompt pass are in tiles of K = 4096, a third in tiles of 16384, which take 3 and 12 % of
    it, so a step that begins at any time waits for (2/3 3 + 1/3 12) / 2 = 3 % of a pass if a workgroup gives its CU back after
    one tile (measured 3.3), and for half of each launch, 10 %, if it keeps it to the launch's end."""
    import torch
    steps, prompts = 100, 24
    narrow, tn, _ = _state(torch, Shape(4, 256, 4, 1024, 1000, 256), 16, 64, 64 + steps, 1)
    wide, tw, _ = _state(torch, Shape(2, 4096, 32, 16384, 1000, 2304), 4, 2048, 2049, 2)

    def decode():
        narrow.rewind(64)
        took = []
        for k in range(steps):
            t = time.perf_counter()
            narrow.decode_step(64 + k, tn[64 + k])
            narrow.synchronize()
            took.append(time.perf_counter() - t)
        return float(np.mean(took))

    narrow.prefill(tn[:64])
    for _ in range(3):
        wide.prefill(tw[:2048])
    wide.synchronize()
    t = time.perf_counter()
    for _ in range(10):
        wide.prefill(tw[:2048])
    wide.synchronize()
    prompt = (time.perf_counter() - t) / 10
    alone = min(decode() for _ in range(3))
    beside = []
    for _ in range(3):
        for _ in range(prompts):
            wide.prefill(tw[:2048])
        beside.append(decode())
        wide.synchronize()
    print(f"prompt {prompt * 1e6:.0f} us, step alone {alone * 1e6:.0f}, beside {[round(b * 1e6) for b in beside]}")
    assert min(beside) - alone < 0.06 * prompt
    for dec in (narrow, wide):
        dec.close()
