"""GEMM results that leave in non-temporal stores (8 MB and more, rows of whole 128-byte lines) against the same call with rows that share lines,
which leave in plain ones: the same bits, up to a last column inside a 16-byte piece, and nothing written beyond it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

M, N, K = 2011, 2101, 520                                 # C of 8.1 MB; ends inside every tile, the last piece of a row holds 5 columns
VARIANTS = ["256pp16", "128pp16", "256x128kp", "224x128kp", "192x128kp", "160x128kp", "128kp", "256w8", "256", "256w8x1", "256w1x8", "128w8",
            "64x128", "64", "128k2", "64x128k2", "64k4", "auto"]


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("variant", VARIANTS)
def test_same_bits_and_edges(variant, aligned):
    from paper_2503_14985_amd import binding
    print("\n[case] %s aligned %d" % (variant, aligned), flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(4)
    A = torch.randn((M, K + 8), generator=gen, device=dev).to(torch.bfloat16)[:, (0 if aligned else 1):][:, :K]
    B = torch.randn((N, K), generator=gen, device=dev).to(torch.bfloat16)
    bias = torch.randn((N,), generator=gen, device=dev).to(torch.bfloat16)
    binding.mlt_diag_force_variant(gemm=variant)
    try:
        for act in (None, 0, 2):
            out = []
            for ldc in (2112, 2108):                      # 33 * 64; not a multiple of 64
                buf = torch.full((M + 1, ldc), 7.0, device=dev, dtype=torch.bfloat16)
                C = buf[:M, :N]
                assert buf.data_ptr() % 128 == 0
                if act is None:
                    binding.mlt_gemm(A, B, C=C, transB=True)
                else:
                    binding.mlt_gemm_bias_act(A, B, bias, act, C=C, transB=True)
                torch.cuda.synchronize()
                assert bool((buf[:M, N:] == 7.0).all()) and bool((buf[M] == 7.0).all())
                out.append(C.contiguous())
            assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
            ref = A.float() @ B.float().t().contiguous() + (0.0 if act is None else bias.float())
            ref = torch.nn.functional.gelu(ref) if act == 2 else ref
            # bf16 rounding of the result (2^-9 relative), fp32 sums of K terms of about sqrt(K), erf in fp32
            assert bool(((out[0].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + K * 2.0 ** -22 * K ** 0.5).all())
    finally:
        binding.mlt_diag_force_variant(gemm="auto")
