"""GPU parity of the two-group GEMM kernels on a K that is not a multiple of their K step, against
the fp64 oracle with the tolerances of tests/test_gemm_gpu.py."""
import pytest

from paper_2503_14985_amd import inputs
import parity_util as pu

pytestmark = pytest.mark.gpu
BF16, FP16 = inputs.BF16, inputs.FP16


@pytest.mark.parametrize("transB", [False, True])
@pytest.mark.parametrize("variant", ["256pp16", "128pp16"])
@pytest.mark.parametrize("K", [8, 56, 72, 120, 136, 64 * 3 + 32, 64 * 5 + 8, 64 * 6 + 56])
def test_partial_last_k_step(K, variant, transB):
    """One to seven K steps, the last one with 1 to 7 of its 8 chunks; ragged M and N, rows longer
    than K with NaN behind them, one row and one column of tiles (the streaming loads) among them."""
    from paper_2503_14985_amd import binding
    for dtype, (M, N) in ((BF16, (300, 264)), (FP16, (100, 520)), (BF16, (520, 72))):
        A, B = inputs.gemm_inputs(M, N, K, dtype, K + M, transB=transB)
        binding.mlt_diag_force_variant(gemm=variant)
        try:
            C = pu.run_gemm(A, B, dtype, transB=transB, lda=K + 8, ldb=(K if transB else N) + 16, ldc_pad=2)
        finally:
            binding.mlt_diag_force_variant(gemm="auto")
        assert binding.mlt_last_kernel().endswith("%sx%sx64_w2x4_pp16" % (variant[:3], variant[:3]))
        print("   %s" % pu.check_gemm(A, B, C, dtype, transB, seed=K), flush=True)
