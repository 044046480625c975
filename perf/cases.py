"""The calls of the library whose speed is measured, with their inputs, their work and their reference results.

Three kinds of pass, each through the public binding (paper_2307_02628_amd.skd):
  decode  `steps` columns of a generation on a cache that a prompt has filled: skd_decode_step + a head per column
  prompt  one prompt: skd_prefill + the head that yields the first token
  head    the sampling head alone, `calls` times with other uniform numbers, as a sampler that redraws calls it
Shapes are the OPT-like ones that the benchmark and the tests use; where a case stands for the layers of a model and
not for the whole call, it has few layers of the full width (and mostly a vocabulary of 1000, as in the tests, so that
the LM head does not hide them).  The bf16 build is what is measured: the fp32 one is for debugging.

Weights follow the usual initialisation of such models (matrices N(0, 0.02), the two projections into the residual
stream scaled by 1 / sqrt(2 L)); token embeddings are wide enough, and the final LayerNorm gain small enough, that the
logits are as decided as a trained model's: with near-flat logits the greedy token would be a coin toss between
correct implementations.  The head cases want the opposite, a nucleus of dozens to hundreds of tokens, and get it from
an untied LM head over hidden states that are embeddings alone (the block's output projections are zero).
"""
import math

import numpy as np
import torch

from paper_2307_02628_amd import skd

# (d_model, heads, ffn) of the models the repository's configurations and tests name, and generic narrow ones
WIDTHS = {
    "tiny": (256, 4, 1024),
    "mid64": (384, 6, 1024),
    "mid": (512, 4, 1536),
    "opt1.3b": (2048, 32, 8192),
    "opt6.7b": (4096, 32, 16384),
}
MAX_POS = 3072
TEMPERATURE, TOP_P = 0.3, 0.7  # the paper's sampling setting


class Shape:
    def __init__(self, case):
        self.d, self.H, self.f = WIDTHS[case["width"]]
        self.L, self.V, self.max_pos = case["layers"], case["vocab"], MAX_POS


def _case(kind, width, layers, vocab, batch, prompt, n_max=0, n_min=0, warmup=0, steps=1, shortest=0, head="argmax",
          io="device", **name):
    """shortest: 0 = every row has `prompt` tokens; else real lengths uniform in [shortest, prompt], left-padded."""
    return dict(name, kind=kind, width=width, layers=layers, vocab=vocab, batch=batch, prompt=prompt,
                n_max=n_max or layers, n_min=n_min or layers, warmup=warmup, steps=steps, shortest=shortest, head=head, io=io)


def listed():
    return [
        # the smallest model of the test configurations, whole generation of 16 tokens with host buffers (the binding's
        # default): nothing but call latency and launches
        _case("decode", "tiny", 4, 1000, 2, 16, 4, 2, steps=16, io="host", name="generate_tiny_b2"),
        # one user at a long, odd context: weights stream for a single row
        _case("decode", "opt6.7b", 4, 1000, 1, 1999, 4, 2, steps=4, name="layers6.7b_b1_ctx1999"),
        # few rows at long contexts
        _case("decode", "opt6.7b", 2, 1000, 8, 2048, 2, 1, steps=4, name="layers6.7b_b8_ctx2048"),
        # an odd batch between the powers of two, with a warm-up layer
        _case("decode", "opt6.7b", 3, 1000, 47, 777, 3, 2, 1, steps=4, name="layers6.7b_b47_ctx777"),
        # the largest batch, ragged prompts
        _case("decode", "opt6.7b", 2, 1000, 128, 512, 2, 1, steps=4, shortest=64, name="layers6.7b_b128_ragged"),
        # whole models: the benchmark's two sizes, depth decaying over the pass as over a generation
        _case("decode", "opt1.3b", 24, 50272, 16, 256, 24, 12, steps=8, name="model1.3b_b16"),
        _case("decode", "opt6.7b", 32, 50272, 32, 512, 32, 6, steps=8, name="model6.7b_b32"),
        # prompts: one short request, a few odd ones at 64-wide heads, long ones, a large ragged batch
        _case("prompt", "opt6.7b", 2, 1000, 1, 60, name="prompt6.7b_b1_60"),
        _case("prompt", "opt1.3b", 4, 50272, 3, 301, name="prompt1.3b_b3_301"),
        _case("prompt", "opt6.7b", 2, 1000, 8, 2048, name="prompt6.7b_b8_2048"),
        _case("prompt", "opt6.7b", 2, 1000, 128, 512, shortest=64, name="prompt6.7b_b128_ragged"),
        # temperature + top-p over the whole vocabulary
        _case("head", "opt6.7b", 1, 50272, 32, 4, steps=8, head="sample", name="sample_b32"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prompt", "prompt", "prompt", "head"])
    width = rng.choice(["tiny", "mid64", "mid", "opt1.3b", "opt1.3b", "opt6.7b", "opt6.7b", "opt6.7b"])
    large = width.startswith("opt")
    vocab = rng.choice([1000, 50272]) if large else rng.choice([777, 1000])
    batch = _log(rng, 1, 128)
    if kind == "head":
        width = rng.choice(["opt1.3b", "opt6.7b"])
        batch = _log(rng, 16, 128)
        return _case("head", width, 1, rng.choice([32000, 50272]), batch, rng.randint(1, 8), steps=-(-256 // batch), head="sample")
    prompt = _log(rng, 8, 2048)
    prompt = max(1, min(prompt, 32768 // batch))
    layers = rng.randint(2, 6) if width != "opt6.7b" else rng.randint(1, 3)
    if batch * prompt > 16384:
        layers = min(layers, 2)
    shortest = rng.choice([0, 0, max(1, prompt // 8)]) if batch > 1 else 0
    if kind == "prompt":
        return _case("prompt", width, layers, vocab, batch, prompt, shortest=shortest)
    warmup = rng.choice([0, 0, 1])
    n_min = rng.randint(max(1, warmup), layers)
    return _case("decode", width, layers, vocab, batch, prompt, rng.randint(n_min, layers), n_min, warmup,
                 steps=rng.randint(2, 6), shortest=shortest, head=rng.choice(["argmax", "argmax", "sample"]),
                 io="device" if large else rng.choice(["device", "host"]))


# ---------------------------------------------------------------------------------------------- inputs
def _start(case, seed):
    """Left-padding columns of each row."""
    if not case["shortest"]:
        return np.zeros(case["batch"], dtype=np.int64)
    lens = np.random.default_rng([seed, 3]).integers(case["shortest"], case["prompt"] + 1, size=case["batch"])
    return case["prompt"] - lens


def _tokens(case, seed):
    """[columns][B] int32: the prompt and the column inputs of the pass (teacher-forced)."""
    g = np.random.default_rng([seed, 2])
    return g.integers(0, case["vocab"], size=(case["prompt"] + case["steps"], case["batch"]), dtype=np.int32)


def _uniforms(case, seed):
    return np.random.default_rng([seed, 4]).random((case["steps"], case["batch"]), dtype=np.float32).clip(0, 0.999999)


def _generator(seed, part):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1009 + part)
    return g


def _normal(g, std, *size, mean=0.0):
    return torch.empty(*size, dtype=torch.float32, device="cuda").normal_(mean, std, generator=g).to(torch.bfloat16)


def _global_weights(case, seed):
    s, g = Shape(case), _generator(seed, 0)
    flat = case["kind"] == "head"
    w = {"tok_emb": _normal(g, 0.02 if flat else 0.5, s.V, s.d), "pos_emb": _normal(g, 0.02, s.max_pos, s.d),
         "lnf_g": _normal(g, 0.02 if flat else 0.001, s.d, mean=1.0 if flat else 0.04), "lnf_b": _normal(g, 0.02 if flat else 0.001, s.d)}
    if flat:
        w["lm_head"] = _normal(g, 0.02 * math.sqrt(4096 / s.d), s.V, s.d)
    return w


def _layer_weights(case, seed, layer):
    s, g = Shape(case), _generator(seed, 1 + layer)
    res = 0.0 if case["kind"] == "head" else 1.0 / math.sqrt(2 * s.L)  # scale of what enters the residual stream
    return {"ln1_g": _normal(g, 0.02, s.d, mean=1.0), "ln1_b": _normal(g, 0.02, s.d),
            "wqkv": _normal(g, 0.02, 3 * s.d, s.d), "bqkv": _normal(g, 0.02, 3 * s.d),
            "wo": _normal(g, 0.02 * res, s.d, s.d), "bo": _normal(g, 0.02 * res, s.d),
            "ln2_g": _normal(g, 0.02, s.d, mean=1.0), "ln2_b": _normal(g, 0.02, s.d),
            "w1": _normal(g, 0.02, s.f, s.d), "b1": _normal(g, 0.02, s.f),
            "w2": _normal(g, 0.02 * res, s.d, s.f), "b2": _normal(g, 0.02 * res, s.d)}


# ---------------------------------------------------------------------------------------------- the passes
def prepare(case, seed):
    s, B, P, T = Shape(case), case["batch"], case["prompt"], case["steps"]
    device = case["io"] == "device"
    weights = _global_weights(case, seed)
    layers = [_layer_weights(case, seed, l) for l in range(s.L)]
    for name in skd.PER_LAYER:
        weights[name] = [w[name] for w in layers]
    cfg = skd.make_config(s, B, P, P + T, case["n_min"], case["n_max"], case["warmup"], dtype=skd.BF16, io_on_device=int(device))
    # the default stream, as in a program with one generation at a time: passes follow each other, and do not overlap
    # those of another state
    dec = skd.Decoder(cfg, weights, location=skd.DEVICE, elem=skd.W_BF16)
    tokens, start, uniforms = _tokens(case, seed), _start(case, seed), _uniforms(case, seed)
    mask = (np.arange(P)[None, :] >= start[:, None]).astype(np.uint8) if case["shortest"] else None
    st = {"kind": case["kind"], "head": case["head"], "dec": dec, "P": P, "mask": mask}
    if device:
        st["prompt"] = torch.from_numpy(tokens[:P].copy()).cuda()
        st["tape"] = list(torch.from_numpy(tokens[P:].copy()).cuda().unbind(0))
        st["uniforms"] = list(torch.from_numpy(uniforms).cuda().unbind(0))
        st["tokens"] = torch.zeros(T, B, dtype=torch.int32, device="cuda")
        st["logits"] = torch.zeros(1 if case["kind"] == "head" else T, B, s.V, dtype=torch.float32, device="cuda")
        st["token_rows"] = list(st["tokens"].unbind(0))
        st["logit_rows"] = list(st["logits"].unbind(0)) * (T if case["kind"] == "head" else 1)
        torch.cuda.synchronize()
    else:
        st["prompt"] = np.ascontiguousarray(tokens[:P].T)
        st["tape"], st["uniforms"] = list(tokens[P:]), list(uniforms)
    if case["kind"] != "prompt":
        dec.prefill(st["prompt"], mask)
        dec.synchronize()
    return st


def run(st):
    dec, sample = st["dec"], st["head"] == "sample"
    if "tokens" not in st:  # host buffers
        tokens, logits = [], []

        def head(k):
            t, z = dec.logits_sample(st["uniforms"][k], TEMPERATURE, TOP_P) if sample else dec.logits_argmax()
            tokens.append(t)
            logits.append(z)
        out = {"tokens": tokens, "logits": logits}
    else:
        def head(k):
            if sample:
                dec.logits_sample_device(st["uniforms"][k], TEMPERATURE, TOP_P, st["token_rows"][k], st["logit_rows"][k])
            else:
                dec.logits_argmax_device(st["token_rows"][k], st["logit_rows"][k])
        out = {"tokens": st["tokens"], "logits": st["logits"]}
    if st["kind"] == "prompt":
        dec.prefill(st["prompt"], st["mask"])
        head(0)
    elif st["kind"] == "decode":
        dec.rewind(st["P"])
        for k, column in enumerate(st["tape"]):
            dec.decode_step(st["P"] + k, column)
            head(k)
    else:
        for k in range(len(st["tape"])):
            head(k)
    return out


# ---------------------------------------------------------------------------------------------- work, reference
def _depth(case, k):
    """Active layers of decode step k: linear from n_max towards n_min, nearest integer, halves up."""
    T, hi, lo = case["steps"], case["n_max"], case["n_min"]
    return (2 * (hi * T - (hi - lo) * k) + T) // (2 * T)


def _columns(case):
    """Columns 0 .. c-1 that each layer processes in prompt + pass: the prompt runs every layer, then the warm-up
    layers and the top of the stack stay."""
    P, L = case["prompt"], case["layers"]
    cols = [P] * L
    if case["kind"] == "decode":
        for k in range(case["steps"]):
            n = _depth(case, k) - case["warmup"]
            for l in list(range(case["warmup"])) + list(range(L - n, L)):
                cols[l] = P + k + 1
    return cols


def work(case):
    """Every column of a generation needs the token before it, so a step reads its weights, and the cached keys and
    values of its layers, once per column."""
    s, B, P = Shape(case), case["batch"], case["prompt"]
    d, f, V = s.d, s.f, s.V
    per_layer, mean = 4 * d * d + 2 * d * f, P - ((P - case["shortest"]) / 2 if case["shortest"] else 0)
    vectors = 4 * (9 * d + f)
    head_b, head_f = 2 * V * d + 4 * B * V + 4 * B, 2 * B * V * d
    if case["kind"] == "head":
        return {"bytes": case["steps"] * head_b, "flops": case["steps"] * head_f}
    if case["kind"] == "prompt":
        rows = B * mean
        return {"bytes": s.L * (2 * per_layer + vectors + 4 * d * rows) + 2 * 2 * d * rows + head_b,
                "flops": s.L * (2 * rows * per_layer + 2 * d * rows * (mean + 1)) + head_f}
    b = fl = 0
    for k in range(case["steps"]):
        n, cached = _depth(case, k), B * (mean + k)
        b += n * (2 * per_layer + vectors + 4 * d * (cached + B)) + 2 * 2 * d * B + head_b
        fl += n * (2 * B * per_layer + 4 * d * (cached + B)) + head_f
    return {"bytes": b, "flops": fl}


def tolerance(case):
    """About four times the distance from exact() that is seen: 0.0014 to 0.0038 through the layers (activations, keys
    and values are bf16 between kernels), 0.0017 through the head alone (its input is bf16).  A sampled token may
    change where the running mass passes u within rounding."""
    if case["kind"] == "head":
        return {"rel": 7e-3, "differ": 0.01}
    return {"rel": 1.5e-2}


def exact(case, seed):
    """The same weights and tokens in float64: every layer is an ordinary causal block over a prefix of the columns."""
    s, B, P = Shape(case), case["batch"], case["prompt"]
    steps = case["steps"] if case["kind"] == "decode" else 0
    d, H, N = s.d, s.H, P + steps
    dh, f64 = d // H, torch.float64
    w = _global_weights(case, seed)
    tok = torch.from_numpy(_tokens(case, seed)[:N].T.copy()).cuda().long()
    start = torch.from_numpy(_start(case, seed)).cuda()
    col = torch.arange(N, device="cuda")
    pos = (col[None, :] - start[:, None]).clamp_(min=0)
    x = w["tok_emb"][tok].to(f64) + w["pos_emb"][pos].to(f64)

    def norm(v, g, b):
        v = v - v.mean(-1, keepdim=True)
        return v / (v.square().mean(-1, keepdim=True) + 1e-5).sqrt() * g.to(f64) + b.to(f64)

    def linear(v, m, b):
        return torch.addmm(b.to(f64), v.reshape(-1, v.shape[-1]), m.to(f64).t()).reshape(*v.shape[:-1], -1)

    for l, c in enumerate(_columns(case)):
        m = _layer_weights(case, seed, l)
        y = x[:, :c]
        qkv = linear(norm(y, m["ln1_g"], m["ln1_b"]), m["wqkv"], m["bqkv"])
        o = torch.empty_like(y)
        causal = col[:c, None] >= col[None, :c]
        for b in range(B):
            q, k, v = (t.reshape(c, H, dh).transpose(0, 1).contiguous() for t in qkv[b].split(d, dim=-1))
            # padding columns see each other (their results are never used), real ones the real ones before them
            seen = causal & ((col[None, :c] >= start[b]) | (col[:c, None] < start[b]))
            p = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(dh)
            p = p.masked_fill_(~seen, -math.inf).softmax(-1)
            o[b] = torch.matmul(p, v).transpose(0, 1).reshape(c, d)
        del qkv
        y = y + linear(o, m["wo"], m["bo"])
        del o
        y = y + linear(linear(norm(y, m["ln2_g"], m["ln2_b"]), m["w1"], m["b1"]).relu_(), m["w2"], m["b2"])
        x[:, :c] = y
    last = x[:, P:] if steps else x[:, P - 1:P]
    z = linear(norm(last, w["lnf_g"], w["lnf_b"]).transpose(0, 1).contiguous(), w.get("lm_head", w["tok_emb"]),
               torch.zeros(1, dtype=f64, device="cuda"))
    return {"tokens": None, "logits": list(z) if case["io"] == "host" else z}
