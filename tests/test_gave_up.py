"""A wait inside the one-launch column that runs out is reported: every call that hands over results, or goes on from them,
returns SKD_ERR_HIP from then on.  The host's part of it on the CPU, and, on the GPU, with the word written by the host
before any kernel could (no kernel waits in vain here)."""
import ctypes as C
import subprocess

import numpy as np
import pytest

import synth_inputs as S
from paper_2307_02628_amd import _build, skd
from tests.helpers import internal

DRIVER = r"""
#include <cstdio>
#include "gave_up.h"
#define EXPECT(c) do { if (!(c)) { printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #c); return 1; } } while (0)
int main() {
  skd::GaveUp none;
  EXPECT(!none.seen());
  uint32_t word = 0, other = 0;
  skd::GaveUp a{&word}, b{&other};
  EXPECT(!a.seen() && !a.seen());
  word = 1;  // as a kernel does
  EXPECT(a.seen() && a.seen() && !b.seen());  // it stays, and belongs to one state
  EXPECT(word == 1);
  printf("all checks passed\n");
  return 0;
}
"""


def test_word(tmp_path):
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O2", "-I", _build.CSRC, str(src), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and "all checks passed" in res.stdout, res.stdout + res.stderr


def word_of(dec):
    f = internal("team_gave_up")
    f.argtypes, f.restype = [C.c_void_p], C.POINTER(C.c_uint32)
    return f(dec._h)


def refused(call):
    with pytest.raises(skd.SkdError) as e:
        call()
    assert e.value.code == skd.ERR_HIP
    assert skd.lib().skd_last_hip_error() == 702  # hipErrorLaunchTimeOut


@pytest.mark.gpu
@pytest.mark.parametrize("device", [0, 1])
def test_calls_report_it(device):
    import torch
    shape, B, P, N = S.TINY, 2, 16, 24
    w = S.weights_to_bf16_values(S.make_weights(shape, 0))
    pr, tape = S.make_prompts(B, P, shape.V, 1), S.make_token_tape(B, N - P, shape.V, 2)
    put = (lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()) if device else np.ascontiguousarray
    tokens, columns, u = put(pr.T if device else pr), [put(t) for t in tape], put(np.full(B, 0.5, dtype=np.float32))
    with skd.Decoder(skd.make_config(shape, B, P, N, 2, 4, io_on_device=device), w) as dec:
        head = dec.logits_argmax_device if device else dec.logits_argmax
        sample = (lambda: dec.logits_sample_device(u, 0.7, 0.9)) if device else (lambda: dec.logits_sample(u, 0.7, 0.9))
        dec.prefill(tokens)
        dec.decode_step(P, columns[0])
        head()
        sample()
        dec.synchronize()
        word = word_of(dec)
        assert word[0] == 0
        word[0] = 1
        for call in (dec.synchronize, head, sample, dec.read_hidden, lambda: dec.kv_read(0, 0), lambda: dec.decode_step(P + 1, columns[1]),
                     lambda: dec.prefill(tokens)):
            refused(call)
        if device:
            assert dec.logits_argmax_noalloc_rc(None, None) == skd.ERR_HIP
        assert dec.kv_len(shape.L - 1) == P + 1  # nothing was enqueued behind it
        word[0] = 0
        dec.synchronize()


@pytest.mark.gpu
def test_wide_models_have_no_such_word():
    shape = S.ModelShape(L=1, d=576, H=9, f=64, V=50, max_pos=8)
    with skd.Decoder(skd.make_config(shape, 1, 2, 6, 1, 1), S.weights_to_bf16_values(S.make_weights(shape, 0))) as dec:
        assert not word_of(dec)
