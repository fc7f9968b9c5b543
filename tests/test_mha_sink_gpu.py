"""Attention where one key in the first tile has nearly all the weight (an attention sink) and the many others, far below it, have
small weights that only their number makes count: what a 16-bit weight far below the row's largest still resolves."""
import math

import numpy as np
import pytest

import oracle
from paper_2503_14985_amd import inputs
import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("gap,Sk", [(18, 8192), (23, 8192), (23, 32768)])
@pytest.mark.parametrize("dtype", [inputs.BF16, inputs.FP16])
def test_sink_and_flat_tail(dtype, gap, Sk, D):
    """gap: how far the others' mean score lies below the first key's, in log2. Their values have a mean of 1."""
    from paper_2503_14985_amd import binding
    print("\n[case] D %d gap %d Sk %d dtype %d" % (D, gap, Sk, dtype), flush=True)
    Sq, scale = 256, D ** -0.5
    rng = np.random.default_rng(gap)
    Q = rng.standard_normal((1, 1, Sq, D)).astype(np.float32)
    K = 0.17 * rng.standard_normal((1, 1, Sk, D)).astype(np.float32)      # scores 0.25 apart in log2
    V = 1.0 + 0.25 * rng.standard_normal((1, 1, Sk, D)).astype(np.float32)
    Q[..., 0], K[..., 0] = 16.0, 0.0
    K[:, :, 0], V[:, :, 0] = 0.0, 0.0
    K[:, :, 0, 0] = gap * math.log(2.0) / scale / 16.0
    Q, K, V = (inputs.to_bits(x, dtype) for x in (Q, K, V))
    binding.mlt_diag_force_variant(mha="pp32")
    binding.mlt_diag_force_key_split(1)               # (a range of keys without the sink would have a maximum of its own)
    try:
        O = pu.run_mha(Q, K, V, scale, False, dtype).double().cpu().numpy()
    finally:
        binding.mlt_diag_force_variant(mha="auto")
        binding.mlt_diag_force_key_split(0)
    ref = oracle.mha_fwd(Q, K, V, scale, False, dtype)
    # With the row's largest weight at 1 or more, an fp16 weight is off by at most 2^-25 (half a subnormal step), one of bf16 by nothing
    # that counts; to that the relative rounding of the weights and of the result (2^-11, bf16 2^-8 each), and fp32 sums.
    step, u = (0.0, 2.0 ** -8) if dtype == inputs.BF16 else (2.0 ** -25, 2.0 ** -11)
    bound = Sk * step * 2.0 + 2 * u * np.abs(ref) + Sk * 2.0 ** -24 * np.abs(ref) + 1e-6
    err = np.abs(O - ref)
    print("   err %.3g, result %.3g" % (err.max(), np.abs(ref).max()), flush=True)
    assert np.all(err <= bound), "worst err %.3g, err/bound %.2f" % (err.max(), (err / bound).max())
