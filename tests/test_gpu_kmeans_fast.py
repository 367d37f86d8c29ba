"""k-means of features of whole positions, whose distances matrix instructions take first: bit for bit the oracle's result at the
edges of its tiles of 16 heads and 16 centres, of its lists and of what the quick distances can tell apart."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
from oracle import chai_oracle as O

from gpu_util import dev


def _same(feat, init, passes=(1, 2, 50)):
    for max_iter in passes:
        got = C.chai_assign_clusters(dev(feat), dev(init), max_iter)
        torch.cuda.synchronize()
        for a, b in zip(got, O.kmeans(feat, init, max_iter=max_iter)):
            assert np.array_equal(a.cpu().numpy(), b)


def _starts(g, B, H, k):
    return np.stack([g.choice(H, size=k, replace=False) for _ in range(B)]).astype(np.int32)


# heads and centres around a tile of 16, a mask word of 32, four words; 64 and 65 centres (the last of these
# and the first of the general kernel); lists that a count of heads fills up to and past whole words
@pytest.mark.parametrize("F", [9, 16, 25, 36, 49, 64])
@pytest.mark.parametrize("H,k", [(1, 1), (15, 3), (16, 15), (17, 16), (31, 17), (33, 32), (65, 33), (128, 48), (129, 64), (130, 65),
                                 (255, 5), (256, 1), (256, 16)])
def test_edges_of_tiles(F, H, k):
    print(f"[kmeans] F={F} H={H} k={k}", flush=True)
    g = np.random.default_rng(F * 1000 + H + k)
    feat = g.random((3, H, F)).astype(np.float32)
    feat[1] = g.integers(0, 2, (H, F))                      # distances tie, centres run empty
    feat[2, :, 1:] = 0                                      # many heads alike in all but one coordinate
    _same(feat, _starts(g, 3, H, k))


# 64 512 bytes of LDS, the most that the quick kernel takes, in the first and the fourth; just above it, and up to 65 484, in the
# others of 25 and 36 coordinates; the general kernel without leave for more (64 512), with it, and at 65 536
@pytest.mark.parametrize("H,k,F", [(196, 64, 25), (212, 58, 25), (231, 52, 25), (225, 33, 36), (139, 64, 36), (254, 226, 16),
                                   (96, 88, 55), (218, 203, 20)])
def test_sizes_at_the_limit_of_lds(H, k, F):
    print(f"[kmeans] F={F} H={H} k={k}", flush=True)
    g = np.random.default_rng(H + k)
    _same(g.random((2, H, F)).astype(np.float32), _starts(g, 2, H, k), passes=(1, 50))


@pytest.mark.parametrize("H,k", [(32, 8), (72, 16), (100, 40)])
@pytest.mark.parametrize("scale", [1e-42, 1e-30, 1e-22, 1e-12, 1.0, 1e12, 1e18, 3e19, 1e38])
def test_features_of_every_magnitude(H, k, scale):
    """From where all products underflow in 32 bits to where they overflow; half of the problem far larger than the rest."""
    g = np.random.default_rng(H + k)
    feat = (g.standard_normal((2, H, 25)) * scale).clip(-3e38, 3e38).astype(np.float32)
    feat[1, : H // 2] *= np.float32(1e-9)
    _same(feat, _starts(g, 2, H, k))


@pytest.mark.parametrize("F", [9, 25, 64])
@pytest.mark.parametrize("offset", [0.0, 1.0, 1e4, 1e7])
@pytest.mark.parametrize("ulps", [0, 1, 3])
def test_centres_closer_than_32_bits_tell(F, offset, ulps):
    """All heads within a few units in the last place of one point: every centre is left to the 64-bit distances."""
    g = np.random.default_rng(F + ulps)
    base = np.float32(offset) + g.random((2, 1, F)).astype(np.float32)
    feat = np.repeat(base, 72, 1)
    for _ in range(ulps):
        feat = np.where(g.random(feat.shape) < 0.5, np.nextafter(feat, np.float32(np.inf)), feat).astype(np.float32)
    _same(feat, _starts(g, 2, 72, 16))


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("H,k,bad", [(72, 16, 0), (72, 16, 15), (40, 33, 32)])
def test_a_starting_centre_that_is_not_finite(H, k, bad, value):
    g = np.random.default_rng(H + bad)
    feat = g.random((2, H, 16)).astype(np.float32)
    init = _starts(g, 2, H, k)
    feat[0, init[0, bad], 3] = value
    _same(feat, init)
