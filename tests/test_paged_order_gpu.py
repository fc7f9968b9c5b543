"""Paged decode with the pieces dealt out by sequence length: batches around the limits of the rank search
(2 and 256 sequences, one more than it takes), equal lengths, one key, more workgroups than CUs and a
last, incomplete round of CUs; against the fp64 oracle."""
import numpy as np
import pytest

from paper_2503_14985_amd import inputs
from test_paged_gpu import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    from paper_2503_14985_amd import binding
    print("\n[case] %s" % request.node.name, flush=True)
    yield
    binding.mlt_diag_force_key_split(0)


@pytest.mark.parametrize("ranges", [1, 2, 64])
@pytest.mark.parametrize("B,H", [(2, 150), (3, 100), (33, 8), (256, 2), (257, 2)])
def test_every_sequence_is_taken_once(B, H, ranges):
    from paper_2503_14985_amd import binding
    binding.mlt_diag_force_key_split(ranges)
    rng = np.random.default_rng(B)
    lens = [int(x) for x in rng.choice([1, 16, 17, 40, 40, 96, 100], B)]
    # one sequence so long that the table's width is that of a cache of 192 MiB, where the ordering begins
    lens[B // 2] = (192 << 20) // (B * H * 128 * 4) + 40
    _check(B, H, 128, 16, lens, inputs.BF16, B)
