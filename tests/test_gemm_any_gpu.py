"""GPU parity of the GEMM kernels for operands of any alignment (odd sizes and leading dimensions)
against the fp64 oracle, with the tolerances of tests/test_gemm_gpu.py."""
import pytest

from paper_2503_14985_amd import inputs
import parity_util as pu

pytestmark = pytest.mark.gpu
BF16, FP16 = inputs.BF16, inputs.FP16


@pytest.fixture(autouse=True)
def _announce(request):
    from paper_2503_14985_amd import binding
    print("\n[case] %s" % request.node.name, flush=True)
    yield
    binding.mlt_diag_force_variant(gemm="auto")
    binding.mlt_diag_force_k_parts(0)


def _go(M, N, K, dtype, transB, variant="auto", seed=0, **pads):
    from paper_2503_14985_amd import binding
    A, B = inputs.gemm_inputs(M, N, K, dtype, seed, transB=transB)
    binding.mlt_diag_force_variant(gemm=variant)
    C = pu.run_gemm(A, B, dtype, transB=transB, lda=pads.get("lda"), ldb=pads.get("ldb"), ldc_pad=pads.get("ldc_pad", 0))
    st = pu.check_gemm(A, B, C, dtype, transB, seed=seed)
    name = binding.mlt_last_kernel()
    print("   %d x %d x %d transB=%d kernel=%s %s" % (M, N, K, transB, name, st), flush=True)
    return name


# K around one 16-byte access, a K step and the K split inside the workgroup; N around an access and
# the tile widths; rows that end on every element of a chunk
EDGES = [(1, 8, 8), (3, 9, 9), (65, 15, 15), (64, 63, 63), (129, 129, 65), (130, 257, 71), (257, 131, 127), (100, 261, 129),
         (70, 70, 64 * 9 + 1), (131, 67, 64 * 8 + 7), (300, 133, 1021)]


@pytest.mark.parametrize("transB", [False, True])
@pytest.mark.parametrize("variant,tile", [("128w8", "128x128x64_w2x4"), ("64x128", "64x128x64_w2x4"), ("64", "64x64x64_w2x2"),
                                          ("128k2", "128x128x64_w2x4_k2"), ("64x128k2", "64x128x64_w2x4_k2"),
                                          ("64k4", "64x64x64_w2x2_k4"), ("256w8", "256x256x64_w2x4")])
def test_edges(variant, tile, transB):
    for i, (M, N, K) in enumerate(EDGES):
        if N % 8 == 0 and K % 8 == 0:
            continue                                     # (these allow aligned accesses: see the padded test)
        name = _go(M, N, K, BF16 if i % 2 else FP16, transB, variant, seed=70 + i)
        assert name == "gemm_general_%s_%s" % ("nt" if transB else "nn", tile), name


@pytest.mark.parametrize("transB", [False, True])
@pytest.mark.parametrize("pad", [1, 2, 3, 4, 7])
def test_padded_rows(pad, transB):
    # rows that start on every alignment, with NaN in the padding: nothing past a row may be read
    # into a result, or written
    for M, N, K in ((1, 8, 8), (70, 72, 136), (200, 264, 75), (131, 37, 600)):
        name = _go(M, N, K, BF16, transB, seed=pad, lda=K + pad, ldb=(K if transB else N) + pad, ldc_pad=pad)
        assert name.startswith("gemm_general_")


@pytest.mark.parametrize("parts", [2, 4, 8])
@pytest.mark.parametrize("transB", [False, True])
def test_k_split_across_workgroups(transB, parts):
    # the last part may be shorter than one 16-byte access
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_k_parts(parts)
    for K in (64 * 64 + 1, 64 * 64 + 63, 64 * 67 + 5):
        name = _go(70, 131, K, BF16, transB, seed=K % 64)
        assert name.endswith("_splitk%d" % parts), name


def test_rows_shorter_than_one_access():
    for M, N, K, transB in ((9, 70, 7, True), (9, 7, 70, False), (33, 5, 3, True)):
        assert _go(M, N, K, BF16, transB) == "gemm_general_64x64x32"


def test_epilogues_on_unaligned_operands():
    for act in (0, 1, 2):
        A, B = inputs.gemm_inputs(130, 133, 203, BF16, 5, transB=True)
        pu.run_check_gemm_bias_act(A, B, inputs.bias_input(133, BF16, 5, std=4.0), act, BF16, transB=True)


def test_fp32_accumulate_on_unaligned_operands():
    import numpy as np
    import torch
    import oracle
    from paper_2503_14985_amd import binding
    dev = torch.device("cuda:0")
    for M, N, K, transB, parts in ((130, 133, 203, True, 1), (130, 133, 203, False, 1), (300, 77, 64 * 20 + 3, True, 2)):
        binding.mlt_diag_force_k_parts(parts)
        A, B = inputs.gemm_inputs(M, N, K, BF16, 6, transB=transB)
        C0 = np.random.default_rng(6).standard_normal((M, N)).astype(np.float32) * 10.0
        Ct = torch.from_numpy(C0.copy()).to(dev)
        binding.mlt_gemm_acc(inputs.bits_to_torch(A, BF16, dev), inputs.bits_to_torch(B, BF16, dev), Ct, transB=transB)
        torch.cuda.synchronize()
        assert binding.mlt_last_kernel().startswith("gemm_general_n") and ("splitk" in binding.mlt_last_kernel()) == (parts > 1)
        Cref, T = oracle.gemm(A, B, BF16, transB=transB)
        err = np.abs(Ct.double().cpu().numpy() - (C0.astype(np.float64) + Cref))
        # fp32 accumulation over K terms, then the final addition (as in tests/test_gemm_gpu.py)
        bound = (K * 2.0 ** -24) * T + 2.0 ** -22 * (np.abs(C0) + T) + 1e-6
        assert np.all(err <= bound), "worst err/bound %.3f" % float(np.max(err / bound))


@pytest.mark.parametrize("transB", [False, True])
def test_tiling_hints_change_nothing_on_unaligned_operands(transB):
    import torch
    from paper_2503_14985_amd import binding
    dev = torch.device("cuda:0")
    for M, N, K in ((130, 333, 203), (9, 18, 77), (40, 70, 5)):
        A, B = (inputs.bits_to_torch(x, BF16, dev) for x in inputs.gemm_inputs(M, N, K, BF16, 4, transB=transB))
        want = binding.mlt_gemm(A, B, transB=transB)
        name = binding.mlt_last_kernel()
        for tiling in (1, 2, 3):
            got = binding.mlt_gemm_tiled(A, B, tiling, transB=transB)
            assert binding.mlt_last_kernel() == name
            assert torch.equal(got.view(torch.int16), want.view(torch.int16))
