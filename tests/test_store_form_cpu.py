"""Which results leave in non-temporal stores, asked on the host: those whose next reader loses nothing by it."""
import re

import pytest

from test_codegen_cpu import _compile_to_asm
from test_plan_cpu import plan  # noqa: F401  (fixture)


# (M, N, ldc, address of C, fp32 accumulate) and the answer
@pytest.mark.parametrize("M,N,ldc,C,acc,want", [
    (512, 512, 512, 0x300000, 0, 0), (1024, 2048, 2048, 0x300000, 0, 0), (777, 4096, 4096, 0x300000, 0, 0),   # small: the reader finds it in a cache
    (2048, 2048, 2048, 0x300000, 0, 1), (2047, 2048, 2048, 0x300000, 0, 0), (3000, 4096, 4096, 0x300000, 0, 1),
    (4095, 4096, 4096, 0x300000, 0, 1), (4096, 4096, 4096, 0x300000, 0, 0),                                  # as large as the L2s
    (4096, 8192, 8192, 0x300000, 0, 0), (8192, 8192, 8192, 0x300000, 0, 0),
    (2048, 4096, 4096 + 64, 0x300000, 0, 1), (2048, 4096, 4096 + 8, 0x300000, 0, 0), (2048, 4096, 4096, 0x300000 + 64, 0, 0),   # rows that share lines
    (2048, 4000, 4032, 0x300000, 0, 1), (2048, 2048, 2048, 0x300000, 1, 0)])
def test_gemm(plan, M, N, ldc, C, acc, want):  # noqa: F811
    assert plan(["store %d %d %d %d %d" % (M, N, ldc, C, acc)]) == [str(want)]


@pytest.mark.parametrize("src,form", [("mha_ks.hip", False), ("mha_pp.hip", True)])
def test_attention(src, form, tmp_path):
    """The kernels for few query rows, whose results are small, store plainly; the 256-row kernels do not."""
    asm = _compile_to_asm(src, tmp_path)
    assert bool(re.search(r"global_store_dwordx4 [^\n]* nt\b", asm)) == form
