"""Attention with an infinite key element: where it makes a score -inf the key has no weight, where +inf the row is NaN. In the first
key tile and in later ones."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_14985_amd import inputs
import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", [inputs.BF16, inputs.FP16])
@pytest.mark.parametrize("key", [3, 100, 299])
def test_infinite_key_element(key, dtype, D):
    from paper_2503_14985_amd import binding
    print("\n[case] key %d D %d dtype %d" % (key, D, dtype), flush=True)
    Sq, Sk, scale = 300, 301, D ** -0.5
    Q, K, V = inputs.mha_inputs(1, 1, Sq, Sk, D, dtype, 17)
    Ki = K.copy()
    Ki[0, 0, key, 5] = 0x7F80 if dtype == inputs.BF16 else 0x7C00
    binding.mlt_diag_force_variant(mha="pp32")
    try:
        O = pu.run_mha(Q, Ki, V, scale, False, dtype).double().cpu().numpy()[0, 0]
    finally:
        binding.mlt_diag_force_variant(mha="auto")
    q5 = pu.widen(Q, dtype)[0, 0, :, 5]
    hidden = q5 < 0
    assert 50 < hidden.sum() < 250 and np.all(np.isnan(O[q5 > 0]))
    keep = [j for j in range(Sk) if j != key]
    ref = oracle.mha_fwd(Q, np.ascontiguousarray(K[:, :, keep]), np.ascontiguousarray(V[:, :, keep]), scale, False, dtype)[0, 0]
    assert np.abs(O[hidden] - ref[hidden]).max() <= pu.MHA_TOL[dtype]
