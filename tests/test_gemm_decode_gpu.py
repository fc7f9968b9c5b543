"""GPU parity of the decode GEMM kernel around the sizes of its pieces of K, rings and column blocks, with K in parts, and with
bias and activation, against the fp64 oracle."""
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


# fewer pieces of 128 k than wavefronts, one for each, one more, two and more rounds of them (a wavefront starts at its share's first piece, or one
# of the first 2, 4 or 8, and goes round), pieces that end inside K; up to one column block per workgroup, and more
@pytest.mark.parametrize("M", [1, 16, 17, 33, 64])
@pytest.mark.parametrize("N", [1032, 4112, 16400, 32776])
def test_k_split_over_wavefronts(M, N):
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_variant(gemm="skinny")
    for i, K in enumerate((8, 72, 256, 1024, 1056, 2048, 2088, 3104, 4128, 5008, 9352)):
        if N > 4112 and i % 3:
            continue
        A, B = inputs.gemm_inputs(M, N, K, FP16 if i % 2 else BF16, i, transB=True)
        C = pu.run_gemm(A, B, FP16 if i % 2 else BF16, transB=True)
        pu.check_gemm(A, B, C, FP16 if i % 2 else BF16, True, seed=i)
        assert binding.mlt_last_kernel() == "gemm_nt_skinny_stream"


@pytest.mark.parametrize("M,N,K", [(1, 2048, 1024), (16, 4104, 520), (13, 1032, 4096), (24, 14336, 2048)])
@pytest.mark.parametrize("act", [0, 1, 2])
def test_streaming_with_bias_and_activation(M, N, K, act):
    from paper_2503_14985_amd import binding
    for dtype in (BF16, FP16):
        A, B = inputs.gemm_inputs(M, N, K, dtype, 4, transB=True)
        pu.run_check_gemm_bias_act(A, B, inputs.bias_input(N, dtype, 4, std=4.0), act, dtype, transB=True)
        assert binding.mlt_last_kernel() == "gemm_nt_skinny_stream"


# columns per workgroup that make blocks of 4, 8 and 16 (one block, a ragged second one, more than a group of 8 or 4 takes),
# up to 4 rows and beyond, one to four row tiles; K below one piece of 128, not a multiple of it, with idle wavefronts, several
# pieces of a wavefront; K in 1 to 8 parts, some of them empty. The sum over parts and wavefronts has one order: the bits repeat.
@pytest.mark.parametrize("M", [1, 4, 5, 16, 32, 47, 64])
@pytest.mark.parametrize("N", [1024, 1100, 2048, 2056, 4104, 34000])
def test_streaming_with_k_in_parts(M, N):
    import torch
    from paper_2503_14985_amd import binding
    try:
        for i, K in enumerate((8, 136, 1032, 2504) if N <= 4104 else (136, 1032)):
            dtype = (BF16, FP16)[i % 2]
            A, B = inputs.gemm_inputs(M, N, K, dtype, 5 + i, transB=True)
            for parts in (1, 2, 4, 8):
                binding.mlt_diag_force_variant(gemm="skinny")
                binding.mlt_diag_force_k_parts(parts)
                C = pu.run_gemm(A, B, dtype, transB=True)
                pu.check_gemm(A, B, C, dtype, True, seed=i)
                name = binding.mlt_last_kernel()
                assert name == "gemm_nt_skinny_stream" + ("" if parts == 1 else "_splitk%d" % parts)
                for _ in range(2):
                    assert torch.equal(pu.run_gemm(A, B, dtype, transB=True).view(torch.int16), C.view(torch.int16))
                if parts > 1 and parts * M * N * 4 <= 32 << 20:   # the fixed scratch: a second kernel adds the parts, in the same order
                    dev = torch.device("cuda:0")
                    tA, tB = inputs.bits_to_torch(A, dtype, dev), inputs.bits_to_torch(B, dtype, dev)
                    D = torch.empty((M, N), dtype=tA.dtype, device=dev)
                    binding.mlt_gemm_noalloc(tA, tB, D, transB=True)
                    torch.cuda.synchronize()
                    assert torch.equal(D.view(torch.int16).cpu(), C.view(torch.int16).cpu())
    finally:
        binding.mlt_diag_force_k_parts(0)
