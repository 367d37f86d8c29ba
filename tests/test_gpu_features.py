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
    """Both sides add in fp64 in element order and round once: almost every value is the same number, with scores of very different
    sizes (the factors of an element are spread over 2^-10 .. 2^10)."""
    g = np.random.default_rng(n_tok + 100 * dtype)
    B, H = 2, 33
    wide = np.exp2(g.integers(-10, 11, size=(B, H, n_tok, 128))).astype(np.float32)
    q5 = W.store(g.standard_normal((B, H, n_tok, 128)).astype(np.float32) * wide, dtype)
    k5 = W.store(g.standard_normal((B, H, n_tok, 128)).astype(np.float32) * wide, dtype)
    feat = C.chai_score_features(dev(q5), dev(k5), n_tok, 1e-6)
    torch.cuda.synchronize()
    got, ref = feat.cpu().numpy(), O.score_features(q5, k5, 1e-6, n_tok=n_tok)
    assert np.abs(got - ref).max() <= 1e-6 and np.mean(got == ref) > 0.999


def _cancelling(n_tok, dtype, B=2, H=33):
    """Elements 16 .. 111: products of +-2^50 that cancel from both ends of the row inwards, so that what is left of the others, of the
    order of 1, is the rounding of a sum of such numbers in its order."""
    g = np.random.default_rng(n_tok + 10 * dtype)
    q, k = (g.standard_normal((B, H, n_tok, 128)).astype(np.float32) * np.float32(0.3) for _ in range(2))
    big_q, big_k = (np.exp2(25 + g.random((B, H, n_tok, 48))).astype(np.float32) * g.choice([-1, 1], (B, H, n_tok, 48)).astype(np.float32) for _ in range(2))
    q[..., 16:64], q[..., 64:112] = big_q, big_q[..., ::-1]
    k[..., 16:64], k[..., 64:112] = big_k, -big_k[..., ::-1]
    return W.store(q, dtype), W.store(k, dtype)


def _features(q5, k5, add):
    """Softmax features of the scores that `add` makes of the products [..., 128] (fp64)."""
    q, k = W.as_f64(q5), W.as_f64(k5)
    B, H, n, _ = q.shape
    feat = np.zeros((B, H, n, n))
    for i in range(n):
        s = np.stack([add(q[:, :, i] * k[:, :, j]) for j in range(i + 1)], -1)
        e = np.exp(s - s.max(-1, keepdims=True))
        feat[:, :, i, :i + 1] = e / e.sum(-1, keepdims=True)
    return feat.reshape(B, H, n * n).astype(np.float32)


def _in_order(x):
    acc = np.zeros(x.shape[:-1])
    for e in range(x.shape[-1]):
        acc = acc + x[..., e]
    return acc


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("n_tok", [3, 5, 6, 8])
def test_products_are_added_in_element_order(n_tok, dtype):
    """Where the order of the sum decides the score, the features are the oracle's; sums of slices, a tree or the reverse order are
    far from them on the same data.  The bound is the last bit of an exponential and of a division, twice rounded to fp32."""
    q5, k5 = _cancelling(n_tok, dtype)
    ref = O.score_features(q5, k5, 1.0, n_tok=n_tok)
    mine = _features(q5, k5, _in_order)
    assert np.abs(mine - ref).max() <= 2.0 ** -22
    for other in (lambda x: _in_order(x[..., ::-1]), lambda x: x.sum(-1),
                  lambda x: _in_order(np.stack([_in_order(x[..., 32 * i:32 * i + 32]) for i in range(4)], -1))):
        moved = np.abs(_features(q5, k5, other) - ref).max(-1) > 1e-4
        assert moved.mean() > 0.9, moved.mean()
    feat = C.chai_score_features(dev(q5), dev(k5), n_tok, 1.0)
    torch.cuda.synchronize()
    got = feat.cpu().numpy()
    assert np.abs(got - ref).max() <= 2.0 ** -22 and np.mean(got == ref) > 0.99
