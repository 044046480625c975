"""The row kernels of the prompt pass, called by themselves: LayerNorm, and embedding + LayerNorm, over every width that one
wave keeps a row of (multiples of 256 up to 4096, each compiled by itself) and the row counts at which the rows of a
workgroup change, and their cost where one wave per row once lost time."""
import ctypes as C

import numpy as np
import pytest

from tests.helpers import internal

pytestmark = pytest.mark.gpu


class RowMap(C.Structure):
    _fields_ = [("seq", C.c_void_p), ("first_row", C.c_void_p), ("start", C.c_void_p), ("P", C.c_int)]


class Rows:
    def __init__(self, rows, d, lens=None, seed=3):
        import torch
        self.torch, self.rows, self.d = torch, rows, d
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        r = lambda *s: torch.randn(*s, generator=g, device="cuda")
        self.V, P = 500, min(rows, 2048)
        lens = lens or [P] * (rows // P)
        self.B, self.P = len(lens), P
        first, seq, at = [], [], 0
        for b, n in enumerate(lens):
            first.append(at)
            seq += [b] * (-(-n // 16) * 16)
            at += -(-n // 16) * 16
        assert at == rows
        i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
        self.first, self.seq, self.start = i32(first), i32(seq), i32([P - n for n in lens])
        self.tokens = torch.randint(0, self.V, (P, self.B), generator=g, device="cuda", dtype=torch.int32)
        self.tok_emb, self.pos_emb = r(self.V, d).to(torch.bfloat16), r(P, d).to(torch.bfloat16)
        self.x, self.g, self.b = r(rows, d), 1 + 0.1 * r(d), 0.1 * r(d)
        self.out = torch.zeros(rows, d, dtype=torch.bfloat16, device="cuda")
        self.ln_fn, self.embed_fn = internal("bf16_ln_rows"), internal("bf16_embed_ln_rows")
        self.null = C.c_void_p(0)

    def p(self, t):
        return C.c_void_p(t.data_ptr())

    def ln(self):
        self.ln_fn(self.null, self.p(self.x), self.p(self.g), self.p(self.b), self.p(self.out), self.rows, self.d)

    def embed(self):
        rm = RowMap(self.seq.data_ptr(), self.first.data_ptr(), self.start.data_ptr(), self.P)
        self.embed_fn(self.null, self.p(self.tokens), rm, self.rows, self.p(self.tok_emb), self.p(self.pos_emb), self.p(self.g),
                      self.p(self.b), self.p(self.x), self.p(self.out), self.B, self.d, self.V)

    def result(self):  # the 16 x 32 tiles as rows
        self.torch.cuda.synchronize()
        return self.out.view(self.rows // 16, self.d // 32, 16, 32).permute(0, 2, 1, 3).reshape(self.rows, self.d).double().cpu()

    def reference(self, x):
        x = x.double().cpu()
        y = (x - x.mean(1, keepdim=True)) / (x.var(1, unbiased=False, keepdim=True) + 1e-5).sqrt()
        return y * self.g.double().cpu() + self.b.double().cpu()

    def microseconds(self, f, n=30):
        torch = self.torch
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(n):
                f()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 1e3 / n)
        return float(np.median(times))


def check(got, want):
    # bf16 keeps 8 bits (half a unit: 2^-9 of the value); the fp32 arithmetic before it adds far less
    assert (got - want).abs().max() <= 2.0 ** -8 * want.abs().max()
    assert ((got - want).abs() <= 2.0 ** -8 * want.abs() + 1e-4).all()


@pytest.mark.parametrize("d", [256 * n for n in range(1, 17)] + [64, 320, 4160])
@pytest.mark.parametrize("rows", [16, 1024, 1040])
def test_values(rows, d):
    r = Rows(rows, d)
    r.ln()
    check(r.result(), r.reference(r.x))
    lens = [rows - 16 - 7, 9] if rows > 16 else [11]        # padding rows in both last tiles
    r = Rows(rows, d, lens)
    r.embed()
    got, x = r.result(), r.x.cpu()
    want_x = r.torch.zeros(rows, d)
    for b, n in enumerate(lens):
        first = int(r.first[b])
        toks = r.tokens[r.P - n:, b].long()
        want_x[first:first + n] = (r.tok_emb[toks].float() + r.pos_emb[:n].float()).cpu()
        check(got[first:first + n], r.reference(want_x[first:first + n]))
        assert (got[first + n:-(-(first + n) // 16) * 16] == 0).all()
    assert r.torch.equal(x, want_x)


def test_cost():
    # 16384 rows of 2048, 201 MB, beside a copy that moves as much (both from the memory-side cache): 1.35 times as long,
    # and 2.2 times with gain and offset fetched behind the statistics and a chunk count that is not exact
    r = Rows(16384, 2048)
    n = 16384 * 2048 * 3 // 4
    a, b = r.torch.zeros(n, device="cuda"), r.torch.empty(n, device="cuda")
    ln, copy = r.microseconds(r.ln), r.microseconds(lambda: b.copy_(a))
    # 64 rows of 4096 with the embedding, beside the kernel of one workgroup per row at the next width
    r, wide = Rows(64, 4096), Rows(64, 4160)
    few, few_wide = r.microseconds(r.embed), wide.microseconds(wide.embed)
    print(f"LayerNorm {ln:.1f} us, copy {copy:.1f}; 64 rows with the embedding {few:.1f}, one workgroup per row {few_wide:.1f}")
    assert ln <= 1.75 * copy
    assert few <= 1.4 * few_wide
