"""GPU parity of the attention kernels that split the keys over groups of wavefronts (and over
workgroups) against the fp64 oracle, with the tolerances of tests/test_mha_gpu.py."""
import math

import pytest
import torch

from paper_2503_14985_amd import inputs
import parity_util as pu
from test_debug_barriers_gpu import dbg, _stream  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
BF16, FP16 = inputs.BF16, inputs.FP16


@pytest.fixture(autouse=True)
def _announce(request):
    from paper_2503_14985_amd import binding
    print("\n[case] %s" % request.node.name, flush=True)
    yield
    binding.mlt_diag_force_variant(mha="auto")
    binding.mlt_diag_force_key_split(0)


def _go(B, H, Sq, Sk, D, dtype, causal, seed, **kw):
    from paper_2503_14985_amd import binding
    scale = kw.pop("scale", 1.0 / math.sqrt(D))
    Q, K, V = inputs.mha_inputs(B, H, Sq, Sk, D, dtype, seed, q_gain=kw.pop("q_gain", 1.0))
    O = pu.run_mha(Q, K, V, scale, causal, dtype)
    st = pu.check_mha(Q, K, V, O, scale, causal, dtype, seed=seed, **kw)
    name = binding.mlt_last_kernel()
    print("   %s kernel=%s %s" % ((B, H, Sq, Sk, D, causal), name, st), flush=True)
    return name


# rows around a wavefront and a workgroup, keys around a tile, a round of all groups and the ring's depth
EDGES = [(1, 1, 1, 1), (1, 3, 31, 32), (2, 1, 33, 33), (1, 2, 64, 129), (1, 1, 65, 63), (1, 2, 128, 257), (2, 1, 129, 640),
         (1, 1, 200, 1000)]


@pytest.mark.parametrize("variant,tag", [("k2", "128x32_k2_pp"), ("k4", "64x32_k4_pp")])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_edges(variant, tag, causal, D):
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_variant(mha=variant)
    for i, (B, H, Sq, Sk) in enumerate(EDGES):
        assert _go(B, H, Sq, Sk, D, BF16 if i % 2 else FP16, causal, 40 + i).endswith(tag)
    _go(1, 2, 100, 300, D, BF16, causal, 50, scale=-0.11)
    _go(1, 2, 100, 300, D, BF16, causal, 51, q_gain=3.0, rounding_aware=True)


@pytest.mark.parametrize("variant", ["k2", "k4"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("ranges", [2, 3, 64])
def test_ranges_of_keys(variant, causal, ranges):
    # ranges of one tile, empty ones at the end, ranges that the mask empties for the first rows
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_variant(mha=variant)
    binding.mlt_diag_force_key_split(ranges)
    for D, dtype, (Sq, Sk) in ((64, FP16, (33, 300)), (128, BF16, (70, 65)), (128, FP16, (150, 517))):
        assert "_keysplit%d_" % ranges in _go(1, 2, Sq, Sk, D, dtype, causal, Sq, rounding_aware=True)


def test_automatic_choice():
    for shape, tag in (((1, 8, 200, 1000, 64, BF16, False), "64x32_k4_pp"), ((4, 16, 300, 2000, 128, BF16, False), "128x32_k2_pp"),
                       ((8, 32, 256, 256, 128, BF16, False), "256x64_pp"), ((1, 8, 5, 4096, 128, FP16, False), "64x32_k4_pp")):
        name = _go(*shape, seed=7)
        assert name.endswith(tag)
        assert ("_keysplit" in name) == (shape[2] == 5), name       # few queries, few heads, many keys


@pytest.mark.parametrize("variant,split", [("k2", 0), ("k4", 0), ("k4", 3)])
def test_agrees_with_the_debug_build(dbg, variant, split):  # noqa: F811
    from paper_2503_14985_amd import binding
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(6)
    try:
        for (B, H, Sq, Sk, D, causal) in ((2, 4, 300, 1501, 128, 0), (2, 4, 700, 700, 64, 1), (1, 2, 130, 2000, 64, 0)):
            q, k, v = (torch.randn((B, H, s, D), generator=g, device=dev).to(torch.bfloat16) for s in (Sq, Sk, Sk))
            binding.mlt_diag_force_variant(mha=variant)
            binding.mlt_diag_force_key_split(split)
            dbg.mlt_diag_force_variant(None, variant.encode())
            dbg.mlt_diag_force_key_split(split)
            want = binding.mlt_mha_fwd(q, k, v, 0.1, causal=bool(causal))
            for _ in range(3):
                got = torch.full_like(want, float("nan"))
                rc = dbg.mlt_mha_fwd(B, H, Sq, Sk, D, q.data_ptr(), k.data_ptr(), v.data_ptr(), got.data_ptr(), 0.1, causal,
                                     0, _stream())
                assert rc == 0
                torch.cuda.synchronize()
                assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    finally:
        dbg.mlt_diag_force_variant(b"auto", b"auto")
        dbg.mlt_diag_force_key_split(0)


def test_captured_call_needs_no_scratch():
    """A call whose keys are spread over workgroups, captured on the stream that has the library's scratch from
    an eager call: it runs without that, and every replay equals the oracle within its bound."""
    from paper_2503_14985_amd import binding
    Q, K, V = inputs.mha_inputs(1, 8, 9, 4096, 128, BF16, 3)
    dev = torch.device("cuda:0")
    q, k, v = (inputs.bits_to_torch(x, BF16, dev) for x in (Q, K, V))
    scale = 1.0 / math.sqrt(128)
    static = torch.empty_like(q)
    side = torch.cuda.Stream(device=dev)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        binding.mlt_mha_fwd(q, k, v, scale)
        assert "_keysplit" in binding.mlt_last_kernel()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        binding.mlt_mha_fwd(q, k, v, scale, O=static)
        assert "_keysplit" not in binding.mlt_last_kernel()
    for _ in range(3):
        static.fill_(0)
        graph.replay()
        binding.mlt_mha_fwd(q, k, v, scale)
        torch.cuda.synchronize()
        pu.check_mha(Q, K, V, static, scale, False, BF16, seed=3)
