"""The library's performance cases: what its users have it do, as calls of the public entry points.

`listed()` holds the fixed cases, `draw(rng)` gives further ones from the same ranges, `prepare(case,
seed)` makes what a program holds before the call, `run(state)` is the call itself, `work(case)` the
bytes and flops no implementation can do without, and `tolerance(case)` how far two correct
implementations may be apart.

A case is a dict of plain values. `op` names the entry point:
  gemm      mlt_gemm:              m, n, k, transb, dtype
  bias_act  mlt_gemm_bias_act:     the same plus act (0 none, 1 ReLU, 2 GELU), always with a bias
  acc       mlt_gemm_acc:          m, n, k, transb, dtype (C is fp32, read and written)
  mha       mlt_mha_fwd:           b, h, sq, sk, d, causal, dtype
  paged     mlt_paged_attn_decode: b, h, d, block, s (longest sequence), dtype; lengths s/4 .. s
All programs keep their output buffer, as a training or serving loop does.
"""
import math

import torch

from paper_2503_14985_amd import binding

_DTYPE = {"bf16": torch.bfloat16, "fp16": torch.float16}
_MAX_FLOPS = 2.0 * 8192 ** 3               # the largest listed case
_ODD_FLOPS = 2.0 * 1999 * 3001 * 1501      # the listed case of odd sizes


def listed():
    return [
        # ---- GEMM
        # The smallest of the square sweep: a small layer or an optimiser's product, where the call
        # itself, the launch and one short K loop are the whole cost.
        dict(name="gemm_512", op="gemm", m=512, n=512, k=512, transb=False, dtype="bf16"),
        # The benchmark's GEMM, the largest square: training-size layer products.
        dict(name="gemm_8192", op="gemm", m=8192, n=8192, k=8192, transb=False, dtype="bf16"),
        # Sizes nobody padded (vocabularies, feature counts, truncated batches): no dimension a
        # multiple of anything, so no row of A, B or C starts aligned.
        dict(name="gemm_odd", op="gemm", m=1999, n=3001, k=1501, transb=False, dtype="bf16"),
        # Prefill of a layer: a prompt of ragged length against a weight matrix stored N x K.
        dict(name="gemm_prefill", op="gemm", m=777, n=4096, k=14336, transb=True, dtype="bf16"),
        # Next-token decode, attention projections: a batch of 16 against a 4096 x 4096 weight.
        dict(name="gemm_decode", op="gemm", m=16, n=4096, k=4096, transb=True, dtype="bf16"),
        # Next-token decode, feed-forward layer with its bias and GELU fused, a batch that does not
        # fill its tile.
        dict(name="ffn_decode_gelu", op="bias_act", m=24, n=14336, k=4096, transb=True, act=2, dtype="bf16"),
        # The paper's own form, C += A * B in fp32: gradient accumulation into a weight's fp32 buffer.
        dict(name="gemm_acc", op="acc", m=4096, n=4096, k=2048, transb=False, dtype="fp16"),
        # ---- attention forward
        # The benchmark's attention: long unmasked sequences.
        dict(name="mha_4096", op="mha", b=4, h=32, sq=4096, sk=4096, d=128, causal=False, dtype="bf16"),
        # The short end of the paper's FlashAttention-2 sweep (32k tokens, hidden 2048, fp16), causal.
        dict(name="mha_causal_1024", op="mha", b=32, h=32, sq=1024, sk=1024, d=64, causal=True, dtype="fp16"),
        # A small batch with ragged lengths, queries and keys of different length (cross attention,
        # a chunk of queries against a longer context): few query tiles for the whole chip.
        dict(name="mha_ragged", op="mha", b=2, h=16, sq=333, sk=1501, d=128, causal=False, dtype="bf16"),
        # ---- paged decode
        # A serving batch: sequences of mixed length in a shuffled cache of 16-key blocks.
        dict(name="paged_batch", op="paged", b=64, h=32, d=128, block=16, s=4096, dtype="bf16"),
        # One long sequence with few heads: too few (sequence, head) pairs to fill the chip.
        dict(name="paged_long", op="paged", b=1, h=8, d=128, block=16, s=32768, dtype="bf16"),
    ]


def _log(rng, lo, hi, mult=1):
    """An integer of [lo, hi], even over its logarithm, a multiple of `mult`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 0.999)))
    return max(lo, min(hi, int(v) // mult * mult))


def draw(rng):
    dtype = rng.choice(["bf16", "bf16", "fp16"])
    kind = rng.choice(["layer", "odd", "decode", "decode", "acc", "mha", "mha", "mha_few", "paged", "paged"])
    if kind == "layer":                     # any number of rows, weights with rows of whole 16-byte pieces
        while True:
            m, n, k = _log(rng, 128, 8192), _log(rng, 512, 14336, 8), _log(rng, 512, 14336, 8)
            if 2.0 * m * n * k <= _MAX_FLOPS:
                break
        if rng.random() < 0.75:             # most layers' sizes are multiples of 64 (all of them >= 512)
            n, k = n // 64 * 64, k // 64 * 64
        if rng.random() < 0.3:
            return dict(op="bias_act", m=m, n=n, k=k, transb=rng.random() < 0.5, act=rng.choice([0, 1, 2]), dtype=dtype)
        return dict(op="gemm", m=m, n=n, k=k, transb=rng.random() < 0.5, dtype=dtype)
    if kind == "odd":
        while True:
            m, n, k = _log(rng, 33, 4001), _log(rng, 33, 4001), _log(rng, 33, 4001)
            if 2.0 * m * n * k <= _ODD_FLOPS:
                break
        return dict(op="gemm", m=m, n=n, k=k, transb=rng.random() < 0.5, dtype=dtype)
    if kind == "decode":
        m, n, k = _log(rng, 1, 64), _log(rng, 1024, 28672, 8), _log(rng, 1024, 28672, 64)
        if rng.random() < 0.35:
            return dict(op="bias_act", m=m, n=n, k=k, transb=True, act=rng.choice([0, 1, 2]), dtype=dtype)
        return dict(op="gemm", m=m, n=n, k=k, transb=True, dtype=dtype)
    if kind == "acc":
        while True:
            m, n, k = _log(rng, 256, 4096, 8), _log(rng, 256, 8192, 8), _log(rng, 256, 8192, 8)
            if m * n <= 4096 * 4096:
                break
        return dict(op="acc", m=m, n=n, k=k, transb=rng.random() < 0.5, dtype=dtype)
    if kind == "mha":                       # batches of whole sequences
        d = rng.choice([64, 128])
        h = 2048 // d if rng.random() < 0.6 else rng.choice([8, 16, 32])
        while True:
            s, b = _log(rng, 256, 8192), _log(rng, 1, 32)
            if rng.random() < 0.5:
                s = max(256, s // 128 * 128)
            if b * s <= 32768 and 4.0 * b * h * s * s * d <= _MAX_FLOPS:
                break
        return dict(op="mha", b=b, h=h, sq=s, sk=s, d=d, causal=rng.random() < 0.6, dtype=dtype)
    if kind == "mha_few":                   # few queries against more keys
        return dict(op="mha", b=_log(rng, 1, 8), h=rng.choice([8, 16, 32]), sq=_log(rng, 1, 800), sk=_log(rng, 64, 4096),
                    d=rng.choice([64, 128]), causal=False, dtype=dtype)
    while True:
        b, h, s = _log(rng, 1, 64), rng.choice([8, 16, 32]), _log(rng, 128, 32768)
        if b * s <= 64 * 4096:
            break
    return dict(op="paged", b=b, h=h, d=rng.choice([64, 128, 128]), block=rng.choice([16, 16, 32, 64]), s=s, dtype=dtype)


def _paged_lengths(case):
    """The lengths of a batch, before they are shuffled over its sequences: evenly from s/4 to s."""
    b, s = case["b"], case["s"]
    lo = max(1, s // 4)
    return [s - (s - lo) * i // max(1, b - 1) for i in range(b)]


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    dtype = _DTYPE[case["dtype"]]

    def normal(shape, std=1.0, dt=dtype):
        t = torch.randn(shape, generator=gen, device=dev, dtype=dt)
        return t if std == 1.0 else t.mul_(std)

    op = case["op"]
    if op in ("gemm", "bias_act", "acc"):
        m, n, k, tb = case["m"], case["n"], case["k"], case["transb"]
        # activations N(0, 1); weights stored N x K with a model's usual 0.02
        st = dict(op=op, A=normal((m, k)), B=normal((n, k), 0.02) if tb else normal((k, n)), transb=tb)
        if op == "bias_act":
            st.update(bias=normal((n,)), act=case["act"])
        st["C"] = normal((m, n), 1.0, torch.float32) if op == "acc" else torch.empty((m, n), dtype=dtype, device=dev)
        return st
    if op == "mha":
        q = normal((case["b"], case["h"], case["sq"], case["d"]))
        k, v = (normal((case["b"], case["h"], case["sk"], case["d"])) for _ in range(2))
        return dict(op=op, Q=q, K=k, V=v, O=torch.empty_like(q), scale=1.0 / math.sqrt(case["d"]), causal=case["causal"])
    b, h, d, bs = case["b"], case["h"], case["d"], case["block"]
    order = torch.randperm(b, generator=gen, device=dev)
    lens = torch.tensor(_paged_lengths(case), dtype=torch.int32, device=dev)[order].contiguous()
    per_seq = -(-case["s"] // bs)
    nb = b * per_seq                        # the cache a serving program sizes for its longest sequences
    table = torch.randperm(nb, generator=gen, device=dev).to(torch.int32).reshape(b, per_seq).contiguous()
    q, kc, vc = normal((b, h, d)), normal((nb, h, bs, d)), normal((nb, h, bs, d))
    return dict(op=op, Q=q, Kc=kc, Vc=vc, table=table, lens=lens, O=torch.empty_like(q), scale=1.0 / math.sqrt(d))


def run(st):
    op = st["op"]
    if op == "gemm":
        return binding.mlt_gemm(st["A"], st["B"], C=st["C"], transB=st["transb"])
    if op == "bias_act":
        return binding.mlt_gemm_bias_act(st["A"], st["B"], st["bias"], st["act"], C=st["C"], transB=st["transb"])
    if op == "acc":
        return binding.mlt_gemm_acc(st["A"], st["B"], st["C"], transB=st["transb"])
    if op == "mha":
        return binding.mlt_mha_fwd(st["Q"], st["K"], st["V"], st["scale"], causal=st["causal"], O=st["O"])
    return binding.mlt_paged_attn_decode(st["Q"], st["Kc"], st["Vc"], st["table"], st["lens"], st["scale"], O=st["O"])


def work(case):
    op = case["op"]
    if op in ("gemm", "bias_act", "acc"):
        m, n, k = case["m"], case["n"], case["k"]
        c = 8 * m * n if op == "acc" else 2 * m * n          # fp32 C is read and written
        return dict(bytes=2 * (m * k + k * n) + c + (2 * n if op == "bias_act" else 0), flops=2.0 * m * n * k)
    if op == "mha":
        b, h, sq, sk, d = (case[x] for x in ("b", "h", "sq", "sk", "d"))
        # causal: key j is visible to query i iff j <= i
        pairs = sum(min(i + 1, sk) for i in range(sq)) if case["causal"] else sq * sk
        return dict(bytes=4 * b * h * d * (sq + sk), flops=4.0 * b * h * d * pairs)
    keys = sum(_paged_lengths(case))
    b, h, d = case["b"], case["h"], case["d"]
    return dict(bytes=4 * keys * h * d + 4 * b * h * d + 4 * b * (1 + -(-case["s"] // case["block"])), flops=4.0 * keys * h * d)


def tolerance(case):
    # About four times the distance (2-norm) measured between each entry point's result and the same
    # computation in float64: one rounding of the output to 8 (bf16) or 11 (fp16) significant bits,
    # in attention also that of the weights; fp32 sums only where C is fp32.
    if case["op"] == "acc":
        return {"rel": 5e-6}                # 2.9e-7 at K = 2048, growing with K and repeated accumulation
    if case["op"] in ("mha", "paged"):
        return {"rel": 1e-2 if case["dtype"] == "bf16" else 1.25e-3}
    return {"rel": 7e-3 if case["dtype"] == "bf16" else 9e-4}
