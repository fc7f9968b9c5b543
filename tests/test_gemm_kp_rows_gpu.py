"""GPU parity of the kernels with two K groups on tiles of 224, 192 and 160 rows (tests/test_gemm_kp_gpu.py has the others)."""
import numpy as np
import pytest
import torch

from paper_2503_14985_amd import inputs
import parity_util as pu
from test_gemm_kp_gpu import _announce, _go  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
BF16, FP16 = inputs.BF16, inputs.FP16


# one row more or less than a tile and than half of one (a wavefront's rows); whole and partial K steps, fewer than the
# ring holds and more; then K in parts, one row of tiles and two
@pytest.mark.parametrize("rows", [224, 192, 160])
@pytest.mark.parametrize("transB", [False, True])
def test_edges(rows, transB):
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_variant(gemm="%dx128kp" % rows)
    tag = "256x128x64_w2x2_kp2"
    for i, (M, K) in enumerate(((1, 64), (rows // 2 + 1, 72), (rows - 1, 128), (rows, 192), (rows + 1, 320), (2 * rows + 17, 456))):
        N = (8, 120, 128, 136, 264)[i % 5]
        assert _go(M, N, K, BF16 if i % 2 else FP16, transB, seed=i).endswith(tag + "_rows%d" % rows)
    assert _go(rows + 1, 264, 200, BF16, transB, lda=208, ldb=(200 if transB else 264) + 8, ldc_pad=3).endswith(tag + "_rows%d" % rows)
    binding.mlt_diag_force_k_parts(2)
    for M in (rows - 3, rows + 3):
        assert _go(M, 136, 64 * 17 + 8, FP16, transB, seed=M).endswith(tag + "_splitk2_rows%d" % rows)


@pytest.mark.parametrize("rows", [224, 192, 160])
def test_fp32_accumulate_and_fused_epilogue(rows):
    import oracle
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_variant(gemm="%dx128kp" % rows)
    dev = torch.device("cuda:0")
    M, N, K = rows + rows // 2 + 3, 141, 64 * 9
    A, B = inputs.gemm_inputs(M, N, K, BF16, 8, transB=True)
    C0 = np.random.default_rng(8).standard_normal((M, N)).astype(np.float32) * 10.0
    Ct = torch.from_numpy(C0.copy()).to(dev)
    binding.mlt_gemm_acc(inputs.bits_to_torch(A, BF16, dev), inputs.bits_to_torch(B, BF16, dev), Ct, transB=True)
    torch.cuda.synchronize()
    Cref, T = oracle.gemm(A, B, BF16, transB=True)
    err = np.abs(Ct.double().cpu().numpy() - (C0.astype(np.float64) + Cref))
    # fp32 accumulation over K terms, then the final addition (as in tests/test_gemm_gpu.py)
    bound = (K * 2.0 ** -24) * T + 2.0 ** -22 * (np.abs(C0) + T) + 1e-6
    assert np.all(err <= bound), "worst err/bound %.3f" % float(np.max(err / bound))
    pu.run_check_gemm_bias_act(A, B, inputs.bias_input(N, BF16, 9, std=4.0), 2, BF16, transB=True)
    assert binding.mlt_last_kernel().endswith("_rows%d" % rows)
