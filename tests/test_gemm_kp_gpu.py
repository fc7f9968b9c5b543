"""GPU parity of the GEMM kernels whose two groups of wavefronts take alternate K steps (256 x 128 and
128 x 128 tiles) against the fp64 oracle, with the tolerances of tests/test_gemm_gpu.py, and bit for bit
against the build with extra waits and barriers."""

import numpy as np
import pytest
import torch

from paper_2503_14985_amd import inputs
import parity_util as pu
from test_debug_barriers_gpu import dbg, _stream  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
BF16, FP16 = inputs.BF16, inputs.FP16
VARIANTS = [("256x128kp", "256x128x64_w2x2_kp2"), ("128kp", "128x128x64_w2x2_kp2")]


@pytest.fixture(autouse=True)
def _announce(request):
    from paper_2503_14985_amd import binding
    print("\n[case] %s" % request.node.name, flush=True)
    yield
    binding.mlt_diag_force_variant(gemm="auto")
    binding.mlt_diag_force_k_parts(0)


def _go(M, N, K, dtype, transB, seed=0, **kw):
    from paper_2503_14985_amd import binding
    A, B = inputs.gemm_inputs(M, N, K, dtype, seed, transB=transB)
    C = pu.run_gemm(A, B, dtype, transB=transB, **kw)
    st = pu.check_gemm(A, B, C, dtype, transB, seed=seed)
    name = binding.mlt_last_kernel()
    print("   %d x %d x %d transB=%d kernel=%s %s" % (M, N, K, transB, name, st), flush=True)
    return name


# one row and one column more or less than a tile; K of one partial step, 1 to 7 whole ones (fewer than the
# ring holds, an odd and an even count) and a partial step behind them
@pytest.mark.parametrize("variant,tag", VARIANTS)
@pytest.mark.parametrize("transB", [False, True])
def test_edges(variant, tag, transB):
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_variant(gemm=variant)
    for i, K in enumerate((8, 56, 64, 72, 128, 192, 264, 320, 384, 448)):
        M, N = ((1, 8), (127, 120), (129, 136), (255, 128), (257, 264))[i % 5]
        assert _go(M, N, K, BF16 if i % 2 else FP16, transB, seed=i).endswith(tag)
    assert _go(300, 264, 200, BF16, transB, lda=208, ldb=(200 if transB else 264) + 8, ldc_pad=3).endswith(tag)


@pytest.mark.parametrize("variant,tag", VARIANTS)
@pytest.mark.parametrize("parts", [2, 8])
def test_k_split_across_workgroups(variant, tag, parts):
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_variant(gemm=variant)
    binding.mlt_diag_force_k_parts(parts)
    for transB in (False, True):
        for K in (64 * 64, 64 * 67 + 8):
            assert _go(200, 136, K, FP16, transB, seed=K % 64).endswith(tag + "_splitk%d" % parts)


@pytest.mark.parametrize("variant,tag", VARIANTS)
@pytest.mark.parametrize("parts", [1, 2])
def test_fp32_accumulate_and_fused_epilogue(variant, tag, parts):
    import oracle
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_variant(gemm=variant)
    binding.mlt_diag_force_k_parts(parts)
    dev = torch.device("cuda:0")
    M, N, K = 270, 141, 64 * 17
    A, B = inputs.gemm_inputs(M, N, K, BF16, 8, transB=True)
    C0 = np.random.default_rng(8).standard_normal((M, N)).astype(np.float32) * 10.0
    Ct = torch.from_numpy(C0.copy()).to(dev)
    binding.mlt_gemm_acc(inputs.bits_to_torch(A, BF16, dev), inputs.bits_to_torch(B, BF16, dev), Ct, transB=True)
    torch.cuda.synchronize()
    assert tag in binding.mlt_last_kernel()
    Cref, T = oracle.gemm(A, B, BF16, transB=True)
    err = np.abs(Ct.double().cpu().numpy() - (C0.astype(np.float64) + Cref))
    # fp32 accumulation over K terms, then the final addition (as in tests/test_gemm_gpu.py)
    bound = (K * 2.0 ** -24) * T + 2.0 ** -22 * (np.abs(C0) + T) + 1e-6
    assert np.all(err <= bound), "worst err/bound %.3f" % float(np.max(err / bound))
    for act in (0, 1, 2):
        pu.run_check_gemm_bias_act(A, B, inputs.bias_input(N, BF16, 9, std=4.0), act, BF16, transB=True)
        assert tag in binding.mlt_last_kernel()


def test_automatic_choice():
    for (M, N, K, tag) in ((1024, 8192, 2048, "256x128x64_w2x2_kp2"), (400, 4096, 11008, "256x128x64_w2x2_kp2_splitk4"),
                           (150, 8192, 28672, "256x128x64_w2x2_kp2_splitk4"), (1024, 4096, 4096, "128x128x64_w2x2_kp2")):
        assert tag in _go(M, N, K, BF16, True, seed=3)


@pytest.mark.parametrize("variant,tag", VARIANTS)
def test_agrees_with_the_debug_build(dbg, variant, tag):  # noqa: F811
    from paper_2503_14985_amd import binding
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(5)
    try:
        for (M, N, K, tb) in ((1000, 1000, 4096, False), (1000, 1000, 4096, True), (520, 392, 1000, True)):
            A = torch.randn((M, K), generator=g, device=dev).to(torch.bfloat16)
            B = torch.randn((N, K) if tb else (K, N), generator=g, device=dev).to(torch.bfloat16)
            binding.mlt_diag_force_variant(gemm=variant)
            dbg.mlt_diag_force_variant(variant.encode(), None)
            want = binding.mlt_gemm(A, B, transB=tb)
            assert binding.mlt_last_kernel().endswith(tag)
            for _ in range(3):
                got = torch.full_like(want, float("nan"))
                rc = dbg.mlt_gemm(M, N, K, A.data_ptr(), A.stride(0), B.data_ptr(), B.stride(0), int(tb), got.data_ptr(),
                                  got.stride(0), 0, _stream())
                assert rc == 0
                torch.cuda.synchronize()
                assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    finally:
        dbg.mlt_diag_force_variant(b"auto", b"auto")
