"""fp32 accumulation of few K steps on the 64 x 64 tile with several K groups, which has its pieces of C in flight from the start:
tiles that end inside a piece, one that is whole, K steps that end inside one; C has rows of its own length and alignment."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_14985_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,transB,pad", [(1, 8, 256, False, 0), (64, 64, 448, True, 0), (65, 141, 264, True, 3), (130, 72, 320, False, 1),
                                              (200, 331, 440, True, 2)])
@pytest.mark.parametrize("dtype", [inputs.BF16, inputs.FP16])
def test_accumulate(M, N, K, transB, pad, dtype):
    from paper_2503_14985_amd import binding
    print("\n[case] %d x %d x %d" % (M, N, K), flush=True)
    dev = torch.device("cuda:0")
    A, B = inputs.gemm_inputs(M, N, K, dtype, 5, transB=transB)
    C0 = np.random.default_rng(5).standard_normal((M, N + pad)).astype(np.float32) * 10.0
    Ct = torch.from_numpy(C0.copy()).to(dev)
    binding.mlt_gemm_acc(inputs.bits_to_torch(A, dtype, dev), inputs.bits_to_torch(B, dtype, dev), Ct[:, :N], transB=transB)
    torch.cuda.synchronize()
    assert binding.mlt_last_kernel().endswith("64x64x64_w2x2_k4")
    got = Ct.double().cpu().numpy()
    assert np.array_equal(got[:, N:], C0[:, N:])
    Cref, T = oracle.gemm(A, B, dtype, transB=transB)
    err = np.abs(got[:, :N] - (C0[:, :N].astype(np.float64) + Cref))
    # fp32 accumulation over K terms, then the final addition (as in tests/test_gemm_gpu.py)
    bound = (K * 2.0 ** -24) * T + 2.0 ** -22 * (np.abs(C0[:, :N]) + T) + 1e-6
    assert np.all(err <= bound), "worst err/bound %.3f" % float(np.max(err / bound))
