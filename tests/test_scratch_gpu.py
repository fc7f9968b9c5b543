"""The scratch of calls that are spread over workgroups, and the counters in front of it: threads on hipStreamPerThread at the same time,
and calls of different kinds and part counts one behind the other on one stream. Every result is a fixed function of its inputs, so
all are compared bit for bit with the same call made alone."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu
PER_THREAD = 2                        # hipStreamPerThread


@pytest.fixture(autouse=True)
def _announce(request):
    from paper_2503_14985_amd import binding
    print("\n[case] %s" % request.node.name, flush=True)
    yield
    binding.mlt_diag_force_variant(gemm="auto", mha="auto")
    binding.mlt_diag_force_k_parts(0)
    binding.mlt_diag_force_key_split(0)


def _gemm(gen, M, N, K):
    dev = torch.device("cuda:0")
    A = torch.randn((M, K), generator=gen, device=dev, dtype=torch.bfloat16)
    B = torch.randn((N, K), generator=gen, device=dev, dtype=torch.bfloat16)
    return A, B


def _paged(gen, B, H, D, keys):
    dev = torch.device("cuda:0")
    nb = B * keys // 16
    q, kc, vc = (torch.randn(s, generator=gen, device=dev, dtype=torch.bfloat16) for s in ((B, H, D), (nb, H, 16, D), (nb, H, 16, D)))
    table = torch.randperm(nb, generator=gen, device=dev).to(torch.int32).reshape(B, -1).contiguous()
    lens = torch.randint(keys // 2, keys + 1, (B,), generator=gen, device=dev, dtype=torch.int32)
    return q, kc, vc, table, lens


def _same(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_threads_on_hip_stream_per_thread():
    from paper_2503_14985_amd import binding
    raw = binding.raw()
    gen = torch.Generator(device="cuda:0")
    work, failures = [], []
    for t in range(4):
        gen.manual_seed(t)
        g, p = _gemm(gen, 16, 1024, 8192), _paged(gen, 1, 8, 64, 704)
        want_g = binding.mlt_gemm(*g, transB=True)
        assert "_splitk" in binding.mlt_last_kernel()
        want_p = binding.mlt_paged_attn_decode(*p, 0.125)
        assert "_keysplit" in binding.mlt_last_kernel()
        work.append((g, p, want_g, want_p, [torch.empty_like(want_g) for _ in range(20)], [torch.empty_like(want_p) for _ in range(20)]))
    torch.cuda.synchronize()
    start = threading.Barrier(len(work))

    def run(g, p, want_g, want_p, out_g, out_p):
        try:
            q, kc, vc, table, lens = p
            start.wait()
            for C, O in zip(out_g, out_p):
                binding.mlt_gemm(*g, C=C, transB=True, stream=PER_THREAD)
                rc = raw.mlt_paged_attn_decode(1, 8, 64, 16, table.shape[1], kc.shape[0], q.data_ptr(), kc.data_ptr(), vc.data_ptr(),
                                               table.data_ptr(), lens.data_ptr(), O.data_ptr(), 0.125, 0, PER_THREAD)
                assert rc == 0
        except Exception as e:        # noqa: BLE001  (shown by the main thread)
            failures.append(e)

    threads = [threading.Thread(target=run, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failures, failures
    for _, _, want_g, want_p, out_g, out_p in work:
        assert all(_same(c, want_g) for c in out_g) and all(_same(o, want_p) for o in out_p)


def test_calls_of_all_kinds_one_behind_the_other_on_one_stream():
    """Decode GEMMs in 2, 4 and 8 parts (their counters go up to one less) and paged decode in 2, 5 and 8 ranges use the same counter words
    in turn; a tile GEMM writes its parts over both; and the buffer grows from 4 MiB to 16 in between, with the
    calls before still under way."""
    from paper_2503_14985_amd import binding
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    small, wide, tall = _gemm(gen, 5, 1100, 2504), _gemm(gen, 32, 8200, 1032), _gemm(gen, 200, 1024, 64 * 80)
    seqs = _paged(gen, 3, 8, 128, 512)

    def gemm(problem, parts, C):
        binding.mlt_diag_force_k_parts(parts)
        binding.mlt_gemm(*problem, C=C, transB=True)
        assert binding.mlt_last_kernel().endswith("_splitk%d" % parts)

    def paged(_, ranges, O):
        binding.mlt_diag_force_key_split(ranges)
        binding.mlt_paged_attn_decode(*seqs, 0.1, O=O)
        assert binding.mlt_last_kernel().endswith("_keysplit%d" % ranges)

    steps = [(gemm, small, 2), (paged, None, 2), (gemm, small, 8), (paged, None, 5), (gemm, small, 4), (paged, None, 8), (gemm, small, 2),
             (gemm, wide, 8), (paged, None, 5), (gemm, small, 8), (gemm, tall, 2), (paged, None, 2), (gemm, wide, 4), (gemm, small, 4), (paged, None, 8)]
    assert 8 * 32 * 8200 * 4 > 4 << 20
    out = lambda f, p: torch.empty((p[0].shape[0], p[1].shape[0]), device="cuda:0", dtype=torch.bfloat16) if f is gemm else torch.empty_like(seqs[0])
    want = []
    for f, p, n in steps:
        want.append(out(f, p))
        f(p, n, want[-1])
        torch.cuda.synchronize()
        if f is gemm and p is not tall:      # and the second kernel adds the same parts in the same order
            C = torch.empty_like(want[-1])
            binding.mlt_gemm_noalloc(*p, C, transB=True)
            torch.cuda.synchronize()
            assert _same(C, want[-1])
    stream = torch.cuda.Stream()
    got = [[out(f, p) for f, p, _ in steps] for _ in range(3)]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for outs in got:
            for (f, p, n), o in zip(steps, outs):
                f(p, n, o)
    stream.synchronize()
    for outs in got:
        for step, (o, w) in enumerate(zip(outs, want)):
            assert _same(o, w), step
