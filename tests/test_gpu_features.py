"""The score features where a pair of positions is shared by four lanes, by two, or has one of its own: against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
import workloads as W
from oracle import chai_oracle as O

from gpu_util import dev


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("n_tok", [1, 2, 4, 5, 6, 7, 8])
def test_features_however_many_lanes_share_a_pair(n_tok, dtype):
    """Both sides add in fp64 in element order and round once: almost every value is the same number, with scores that are large
    and nearly cancel as well (elements up to 2^20, so that the order of the sum is seen in its low bits)."""
    g = np.random.default_rng(n_tok + 100 * dtype)
    B, H = 2, 33
    wide = np.exp2(g.integers(-10, 11, size=(B, H, n_tok, 128))).astype(np.float32)
    q5 = W.store(g.standard_normal((B, H, n_tok, 128)).astype(np.float32) * wide, dtype)
    k5 = W.store(g.standard_normal((B, H, n_tok, 128)).astype(np.float32) * wide, dtype)
    feat = C.chai_score_features(dev(q5), dev(k5), n_tok, 1e-6)
    torch.cuda.synchronize()
    got, ref = feat.cpu().numpy(), O.score_features(q5, k5, 1e-6, n_tok=n_tok)
    assert np.abs(got - ref).max() <= 1e-6 and np.mean(got == ref) > 0.999
