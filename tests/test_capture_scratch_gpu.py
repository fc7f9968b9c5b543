"""Calls that are spread over workgroups through the library's scratch, captured on a stream that already has
such a buffer: the graph must not keep it (it may be replayed on another stream, beside eager calls of the
first one and beside a second graph), so the captured call runs without the split."""
import math

import pytest
import torch

from paper_2503_14985_amd import inputs
import oracle
import parity_util as pu

pytestmark = pytest.mark.gpu
BF16 = inputs.BF16
SCALE = 1.0 / math.sqrt(128)


@pytest.fixture(autouse=True)
def _announce(request):
    print("\n[case] %s" % request.node.name, flush=True)
    yield


class _Gemm:
    tag = "_splitk"

    def __init__(self, dev, seed):
        self.A_h, self.B_h = inputs.gemm_inputs(64, 2048, 64 * 160, BF16, seed, transB=True, std=0.02)
        self.A, self.B = (inputs.bits_to_torch(x, BF16, dev) for x in (self.A_h, self.B_h))
        self.shape = (64, 2048)

    def run(self, out):
        from paper_2503_14985_amd import binding
        binding.mlt_gemm(self.A, self.B, C=out, transB=True)

    def check(self, out):
        pu.check_gemm(self.A_h, self.B_h, out, BF16, True, seed=1)


class _Paged:
    tag = "_keysplit"

    def __init__(self, dev, seed):
        self.h = inputs.paged_inputs(3, 8, 128, 16, [4096, 1000, 2500], BF16, seed)[:5]
        self.t = [inputs.bits_to_torch(x, BF16, dev) for x in self.h[:3]] + [torch.from_numpy(x).to(dev) for x in self.h[3:]]
        self.shape = tuple(self.t[0].shape)

    def run(self, out):
        from paper_2503_14985_amd import binding
        binding.mlt_paged_attn_decode(*self.t, SCALE, O=out)

    def check(self, out):
        ref = oracle.paged_attn_decode(*self.h, SCALE, oracle.BF16)
        assert abs(out.double().cpu().numpy() - ref).max() <= 1e-2


@pytest.mark.parametrize("kind", [_Gemm, _Paged], ids=["gemm", "paged"])
def test_a_graph_does_not_share_the_streams_scratch(kind):
    from paper_2503_14985_amd import binding
    dev = torch.device("cuda:0")
    a, b, c = (kind(dev, s) for s in (1, 2, 3))
    outs = [torch.zeros(a.shape, dtype=torch.bfloat16, device=dev) for _ in range(3)]
    first, second = torch.cuda.Stream(device=dev), torch.cuda.Stream(device=dev)
    torch.cuda.synchronize()
    with torch.cuda.stream(first):
        c.run(outs[2])                                # the stream has its buffer from here on
        assert a.tag in binding.mlt_last_kernel()
    torch.cuda.synchronize()
    graphs = []
    for problem, out in ((a, outs[0]), (b, outs[1])):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=first):
            problem.run(out)
            name = binding.mlt_last_kernel()
        assert a.tag not in name, name
        graphs.append(g)
    for _ in range(3):
        for out in outs:
            out.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(first):
            c.run(outs[2])
            graphs[0].replay()
        with torch.cuda.stream(second):
            graphs[1].replay()
        with torch.cuda.stream(first):
            c.run(outs[2])
        torch.cuda.synchronize()
        for problem, out in ((a, outs[0]), (b, outs[1]), (c, outs[2])):
            problem.check(out)
