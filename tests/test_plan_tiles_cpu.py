"""The tile that the library chooses for a GEMM, asked on the host, where its height or the fp32 C decides."""
import pytest

from test_plan_cpu import gemm_line, plan  # noqa: F401  (fixture)


def tile(plan, M, N, K, transB, **kw):
    rows, cols, _, parts, _ = plan([gemm_line(M, N, K, transB, **kw).replace("gemm", "tile", 1)])[0].split()
    return int(rows), int(cols), int(parts)


# one tile of 160 rows covers these; in four or two parts all heights are bound by the operands' arrival and their estimates equal
@pytest.mark.parametrize("M,N,K,transB,parts", [(150, 8192, 28672, 1, 4), (130, 7296, 10624, 1, 4), (149, 12672, 12032, 0, 2), (146, 12288, 10176, 1, 2)])
def test_equal_estimates_take_the_smaller_height(plan, M, N, K, transB, parts):  # noqa: F811
    assert tile(plan, M, N, K, transB) == (160, 128, parts)


def test_heights(plan):  # noqa: F811
    """Problems whose padding the heights below 256 save, and some that stay on 256."""
    for M, N, K, transB, want in ((777, 4096, 14336, 1, (224, 128, 2)), (316, 6784, 10368, 0, (160, 128, 2)), (300, 8192, 8192, 1, (160, 128, 2)),
                                  (171, 7744, 9408, 1, (192, 128, 4)), (1700, 10816, 3584, 1, (192, 128, 1)), (1024, 8192, 2048, 1, (256, 128, 1)),
                                  (2048, 4096, 4096, 1, (256, 128, 1)), (8192, 8192, 8192, 0, (256, 256, 1))):
        assert tile(plan, M, N, K, transB) == want, (M, N, K)


def test_fp32_accumulate(plan):  # noqa: F811
    """C's traffic counts in every kernel that is alone on its CU and has nothing to hide it behind, not in one of them only."""
    for M, N, K, transB, want in ((680, 3200, 3200, 0, "nn_128x128x64_w2x2_kp2"), (720, 3968, 4608, 0, "nn_128x128x64_w2x2_kp2"),
                                  (2912, 1344, 3904, 0, "nn_128x128x64_w2x2_kp2"), (792, 4688, 352, 1, "nt_64x128x64_w2x4"),
                                  (2232, 2752, 968, 0, "nn_128x128x64_w2x4_pp16"), (4096, 4096, 2048, 0, "nn_256x256x64_w2x4_pp16")):
        assert plan([gemm_line(M, N, K, transB, acc=1)])[0].split()[0] == "gemm_" + want, (M, N, K)


def test_gelu(plan):  # noqa: F811
    """Problems of few K steps that the tall tiles take without GELU and not with it, and one of many that they take with it too."""
    for M, N, K, transB, plain, gelu in ((1607, 3840, 768, 1, "nt_256x128x64_w2x2_kp2", "nt_128x128x64_w2x4_pp16"),
                                         (805, 6272, 704, 1, "nt_256x128x64_w2x2_kp2", "nt_128x128x64_w2x4_pp16"),
                                         (5274, 960, 768, 1, "nt_256x128x64_w2x2_kp2", "nt_128x128x64_w2x4_pp16"),
                                         (2024, 8640, 704, 0, "nn_256x256x64_w2x4_pp16", "nn_128x128x64_w2x4_pp16"),
                                         (2048, 4096, 4096, 1, "nt_256x128x64_w2x2_kp2", "nt_256x128x64_w2x2_kp2")):
        assert [x.split()[0] for x in plan([gemm_line(M, N, K, transB, fused=f) for f in (1, 3)])] == ["gemm_" + plain, "gemm_" + gelu], (M, N, K)
