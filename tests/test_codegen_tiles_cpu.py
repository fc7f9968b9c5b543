"""The tile GEMM kernels keep their accumulators in registers (read from the assembly of this repository's own build)."""
import re

import pytest

from test_codegen_cpu import _compile_to_asm


@pytest.mark.parametrize("src", ["gemm.hip", "gemm_any.hip", "gemm_kp.hip"])
def test_no_accumulators_in_memory(src, tmp_path):
    """Scratch memory of every kernel: none, but for a few values that are used once per K step in the 256 x 256 forms with all wavefronts
    in one row or column (tiling hints 1 and 2), whose lanes hold 128 accumulators and as much of the operands. An accumulator
    with a run-time index moves all of them to memory: 1088 bytes per lane, 182 -> 1837 us for 4096 x 4096 x 4104."""
    asm = _compile_to_asm(src, tmp_path)
    found = re.findall(r"^(_ZN3mlt\S*kernel\S*):.*?\.end_amdhsa_kernel.*?; ScratchSize: (\d+)", asm, re.S | re.M)
    assert len(found) >= 8
    for name, scratch in found:
        few = "gemm_tile_kernel" in name and ("Li256ELi256ELi64ELi8ELi1E" in name or "Li256ELi256ELi64ELi1ELi8E" in name)
        assert int(scratch) <= (32 if few else 0), "%s: %s bytes of scratch" % (name, scratch)
