"""Paged decode with the pieces dealt out by sequence length: batches around the limits of the rank search
(2 and 256 sequences, one more than it takes), equal lengths, one key, more workgroups than CUs and a
last, incomplete round of CUs; against the fp64 oracle."""
import numpy as np
import pytest

from paper_2503_14985_amd import inputs
from test_paged_gpu import _check

BF16, FP16 = inputs.BF16, inputs.FP16
CASES = [(B, H, ranges, D, dtype) for D, dtype in ((128, BF16), (64, FP16))
         for B, H in ((2, 150), (3, 100), (33, 8), (256, 2), (257, 2)) for ranges in (1, 2, 16)]


def longest(B, H, ranges, D):
    """The longest sequence, that is the table's width, from which on such a batch is dealt by length: a cache of 192 MiB
    (224 in one range), and enough keys for the rank search to pay (tests/test_plan_cpu.py asks the library)."""
    cache = (224 if ranges == 1 else 192) << 20
    return max(-(-cache // (B * H * D * 4)), B * H * ranges ** 2 * B * 10 // (32 * D) + 1) + 40


@pytest.fixture(autouse=True)
def _announce(request):
    print("\n[case] %s" % request.node.name, flush=True)
    yield


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,ranges,D,dtype", CASES)
def test_every_sequence_is_taken_once(B, H, ranges, D, dtype):
    from paper_2503_14985_amd import binding
    rng = np.random.default_rng(B)
    lens = [int(x) for x in rng.choice([1, 16, 17, 40, 40, 96, 100], B)]
    lens[B // 2] = longest(B, H, ranges, D)
    binding.mlt_diag_force_key_split(ranges)
    try:
        _check(B, H, D, 16, lens, dtype, B)
        assert binding.mlt_last_kernel().endswith("_w4" if ranges == 1 else "_keysplit%d" % ranges)
    finally:
        binding.mlt_diag_force_key_split(0)
