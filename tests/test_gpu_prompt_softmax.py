"""The prompt's attention kernel by itself against a float64 softmax over the same bf16 queries, keys and values: lengths at
the edges of its tiles (16), waves and blocks (32) and workgroups (32, 64 and 128 positions, by the longest sequence), and
scores for which the softmax reference stays where the first block put it, is raised by later blocks (more than 8 in
log2), now and then or in every block, or is far above everything that follows.

Bound: a weight is rounded to bf16 (relative 2^-9) in the numerator and in the denominator, the result once more; with
values up to vmax that is at most 3 * 2^-9 * vmax.  Scores are fp32 sums: their error (a few 2^-24 of scores up to 200)
moves a weight by less than 2^-14."""
import ctypes as C

import numpy as np
import pytest

from tests.helpers import internal
from tests.test_gpu_prompt_rows import RowMap

pytestmark = pytest.mark.gpu


class KvGeom(C.Structure):
    _fields_ = [("page_tokens", C.c_int), ("max_pages", C.c_int), ("H", C.c_int), ("dh", C.c_int), ("page_elems", C.c_long)]


class Args(C.Structure):
    _fields_ = [("q", C.c_void_p), ("pool", C.c_void_p), ("bt_layer", C.c_void_p), ("rm", RowMap), ("B", C.c_int),
                ("max_len", C.c_int), ("kv", KvGeom), ("o", C.c_void_p)]


class Attention:
    def __init__(self, lens, H, dh, page_tokens=64, seed=1, q=None, k=None):
        """lens: real positions of each sequence; q, k: [len, H, dh] of each sequence, None = N(0, 1)."""
        import torch
        self.torch, self.lens, self.H, self.dh = torch, lens, H, dh
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        bf = lambda x: x.to(torch.bfloat16)
        r = lambda n: torch.randn(n, H, dh, generator=g, device="cuda")
        self.q = [bf(r(n) if q is None else q(n, r)) for n in lens]
        self.k = [bf(r(n) if k is None else k(n, r)) for n in lens]
        self.v = [bf(r(n)) for n in lens]
        d, B, P, pt = H * dh, len(lens), max(lens), page_tokens
        first, rows = [], 0
        for n in lens:
            first.append(rows)
            rows += -(-n // 16) * 16
        self.d, self.rows = d, rows
        i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
        pages = [-(-n // pt) for n in lens]
        max_pages = max(pages)
        bt, at = np.full((B, max_pages), -1, dtype=np.int32), 0
        for b in range(B):
            bt[b, :pages[b]] = at + np.random.default_rng(b).permutation(pages[b])
            at += pages[b]
        page = 2 * pt * d
        pool = torch.zeros(at, page, dtype=torch.bfloat16, device="cuda")
        qt = torch.zeros(rows // 16, d // 32, 16, 32, dtype=torch.bfloat16, device="cuda")
        hh, ee = torch.arange(H, device="cuda")[None, :, None], torch.arange(dh, device="cuda")[None, None, :]
        for b, n in enumerate(lens):
            pos = torch.arange(n, device="cuda")
            tt = (pos % pt)[:, None, None]
            kk = tt % 32
            base = hh * (pt * dh * 2) + tt // 32 * (64 * dh)
            k_off = base + (((kk // 16) * (dh // 32) + ee // 32) * 64 + kk % 16 + 16 * (ee % 32 // 8)) * 8 + ee % 8
            v_off = base + 32 * dh + (ee // 16 * 64 + 16 * (kk % 16 // 4) + ee % 16) * 8 + 4 * (kk // 16) + kk % 4
            pg = torch.tensor(bt[b], device="cuda").long()[pos // pt][:, None, None].expand(n, H, dh)
            pool[pg, k_off] = self.k[b]
            pool[pg, v_off] = self.v[b]
            padded = torch.zeros(-(-n // 16) * 16, d, dtype=torch.bfloat16, device="cuda")
            padded[:n] = self.q[b].reshape(n, d)
            qt[first[b] // 16:first[b] // 16 + len(padded) // 16] = padded.view(-1, 16, d // 32, 32).permute(0, 2, 1, 3)
        self.first = first
        self.out = torch.zeros_like(qt)
        seq = i32([b for b, n in enumerate(lens) for _ in range(-(-n // 16) * 16)])
        first_t, start, bt_t = i32(first), i32([P - n for n in lens]), torch.tensor(bt, device="cuda")
        self.keep = (pool, qt, seq, first_t, start, bt_t)
        self.args = Args(qt.data_ptr(), pool.data_ptr(), bt_t.data_ptr(), RowMap(seq.data_ptr(), first_t.data_ptr(), start.data_ptr(), P),
                         B, P, KvGeom(pt, max_pages, H, dh, page), self.out.data_ptr())
        self.fn = internal("bf16_attention_rows")

    def run(self):
        self.fn(C.c_void_p(0), C.byref(self.args))

    def worst(self):
        """Largest difference from float64, in units of the largest value."""
        torch = self.torch
        torch.cuda.synchronize()
        rows = self.out.permute(0, 2, 1, 3).reshape(self.rows, self.d)
        worst = 0.0
        for b, n in enumerate(self.lens):
            q, k, v = (t[b].double().cpu().permute(1, 0, 2).contiguous() for t in (self.q, self.k, self.v))
            s = q @ k.transpose(1, 2).contiguous() / np.sqrt(self.dh)
            s.masked_fill_(torch.ones(n, n, dtype=torch.bool).triu(1), -np.inf)
            want = (torch.softmax(s, -1) @ v).permute(1, 0, 2).reshape(n, self.d)
            got = rows[self.first[b]:self.first[b] + n].double().cpu()
            worst = max(worst, float((got - want).abs().max() / v.abs().max()))
        return worst


BOUND = 3 * 2.0 ** -9


@pytest.mark.parametrize("H,dh", [(2, 64), (2, 128)])
@pytest.mark.parametrize("lens", [[1], [16, 3], [17, 31], [32] * 5, [33, 1, 16], [64, 40, 32], [63], [65, 20], [128, 127], [129, 5, 96], [300]])
def test_lengths(lens, H, dh):
    for pt in (32, 64):
        a = Attention(lens, H, dh, pt)
        a.run()
        assert a.worst() <= BOUND


def grow(n, r):        # keys that count for more and more: most blocks raise the reference
    x = r(n)
    return x * (0.3 + 3.0 * x.new_tensor(range(n))[:, None, None] / n)


SCORES = {
    # deviation of the scores in log2: below 1.5 (no raise after the first block), 6 (now and then), 23 (often)
    "flat": (lambda n, r: 0.5 * r(n), None),
    "moderate": (lambda n, r: 4.0 * r(n), None),
    "spread": (lambda n, r: 16.0 * r(n), None),
    "growing": (lambda n, r: 8.0 * r(n), grow),
    # one huge first key: what follows stays far below the reference; one huge last key: everything before counts for nothing
    "first": (lambda n, r: r(n).abs() + 1, lambda n, r: r(n).index_fill_(0, r(1).new_zeros(1).long(), 12.0)),
    "last": (lambda n, r: r(n).abs() + 1, lambda n, r: r(n).index_fill_(0, r(1).new_full((1,), n - 1).long(), 12.0)),
}


@pytest.mark.parametrize("H,dh", [(3, 64), (2, 128)])
@pytest.mark.parametrize("scores", SCORES)
@pytest.mark.parametrize("lens", [[30, 23], [61, 33], [333, 200, 41]])
def test_scores(lens, scores, H, dh):
    q, k = SCORES[scores]
    a = Attention(lens, H, dh, seed=5, q=q, k=k)
    a.run()
    assert a.worst() <= BOUND


def test_cost_of_short_sequences():
    # 2048 rows as 128 sequences of 8 (padded to 16) and as 32 of 64: about 1.05 times as long, 1.45 times when every
    # sequence had a workgroup of four waves
    import torch
    us = {}
    for B, n in ((128, 8), (32, 64)):
        a, t = Attention([n] * B, 32, 128), []
        for _ in range(9):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                a.run()
            e1.record()
            e1.synchronize()
            t.append(e0.elapsed_time(e1) * 50)
        us[n] = min(t)
    print("attention us", us)
    assert us[8] <= 1.3 * us[64]
