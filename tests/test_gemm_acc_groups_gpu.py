"""fp32 accumulation in the kernels with several K groups, which have their pieces of C in flight from the start: 128 x 128 and 64 x 128 tiles
(four pieces and two of a thread's 1024), and 64 x 64 with four groups and with three (B stored K x N)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_14985_amd import inputs

pytestmark = pytest.mark.gpu


# M and N end inside a tile, N inside a piece of four columns; rows of C of any length. K: one step (idle groups), a partial one behind
# it, and more steps than groups with a partial last one
@pytest.mark.parametrize("variant", ["128k2", "64x128k2", "64k4"])
@pytest.mark.parametrize("transB", [False, True])
@pytest.mark.parametrize("M,N,K,pad", [(1, 8, 64, 0), (67, 131, 72, 3), (129, 264, 520, 0), (190, 127, 648, 1), (257, 386, 1088, 2)])
def test_accumulate(M, N, K, pad, transB, variant):
    from paper_2503_14985_amd import binding
    print("\n[case] %s %d x %d x %d" % (variant, M, N, K), flush=True)
    dev = torch.device("cuda:0")
    N = N if transB else N // 8 * 8                       # (rows of B that start on 16 bytes; others go to the kernels for any alignment)
    dtype = inputs.FP16 if K % 128 else inputs.BF16
    A, B = inputs.gemm_inputs(M, N, K, dtype, 6, transB=transB)
    C0 = np.random.default_rng(6).standard_normal((M + 1, N + pad)).astype(np.float32) * 10.0
    Ct = torch.from_numpy(C0.copy()).to(dev)
    Bt = inputs.bits_to_torch(B, dtype, dev)
    binding.mlt_diag_force_variant(gemm=variant)
    binding.mlt_diag_force_k_parts(1)
    try:
        binding.mlt_gemm_acc(inputs.bits_to_torch(A, dtype, dev), Bt, Ct[:M, :N], transB=transB)
        torch.cuda.synchronize()
        name = binding.mlt_last_kernel()
    finally:
        binding.mlt_diag_force_variant(gemm="auto")
        binding.mlt_diag_force_k_parts(0)
    assert name == "gemm_%s_%s" % ("nt" if transB else "nn", {"128k2": "128x128x64_w2x4_k2", "64x128k2": "64x128x64_w2x4_k2", "64k4": "64x64x64_w2x2_k4"}[variant])
    got = Ct.double().cpu().numpy()
    assert np.array_equal(got[:, N:], C0[:, N:]) and np.array_equal(got[M], C0[M])
    Cref, T = oracle.gemm(A, B, dtype, transB=transB)
    err = np.abs(got[:M, :N] - (C0[:M, :N].astype(np.float64) + Cref))
    # fp32 accumulation over K terms, then the final addition (as in tests/test_gemm_gpu.py)
    bound = (K * 2.0 ** -24) * T + 2.0 ** -22 * (np.abs(C0[:M, :N]) + T) + 1e-6
    assert np.all(err <= bound), "worst err/bound %.3f" % float(np.max(err / bound))
