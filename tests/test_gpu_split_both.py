"""Band transform of 8-bit pixels with both directions in a workgroup, against the
oracle: images of more than 384 workgroups' worth of items take it (fewer go one
direction a workgroup), here through many bands, at widths on the edges of its tiles.
Saturated images hold the largest sums that share a register.  Integer, so equal.
"""

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu

ITEMS = 385  # the fewest that take both directions


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _bands(n, w):
    """The fewest bands of n rows that have ITEMS items."""
    block = min(n, 128)  # rows of a row block (taller bands: in 128-row ones)
    tile, groups = (240, 1) if block == 32 else (228, block // 64)
    return -(-ITEMS // (-(-(w + n) // tile) * groups * (n // block)))


def _widths(n):
    tile = 240 if n == 32 else 228
    widths = {1, n // 2 + 1}
    for cols in (tile // 2, tile, tile + 1, 2 * tile, 2 * tile + 3):
        widths.update(w for w in (cols - n, cols - n + 1) if w > 0)
    return sorted(widths) if n <= 128 else [1, 228 * 5 - n, 228 * 5 - n + 1]


@pytest.mark.parametrize("saturated", [False, True])
@pytest.mark.parametrize("n,w", [(n, w) for n in (32, 64, 128, 512, 1024) for w in _widths(n)])
def test_tables(dev, n, w, saturated):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(n + w)
    k = _bands(n, w)
    img = (np.full((k * n, w), 255, dtype=np.uint8) if saturated else
           rng.integers(0, 256, size=(k * n, w)).astype(np.uint8))
    announce(f"tables {k * n}x{w} k={k} saturated={saturated}")
    got = fhtp.fht_bands(torch.from_numpy(img).to(dev), k).cpu().numpy()
    assert np.array_equal(got, oracle.fht_bands(img, k))


# 16-bit tables of all bands but the last: the detection's own path, at odd widths (a
# row starts on either half of a word) and saturated
@pytest.mark.parametrize("n,w", [(32, 241), (64, 165), (128, 101)])
def test_detection(dev, n, w):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(n)
    k = _bands(n, w)
    img = np.full((k * n, w), 255, dtype=np.uint8)
    img[rng.integers(0, k * n, size=k * n // 2), rng.integers(0, w, size=k * n // 2)] = 0
    announce(f"detection {img.shape} k={k}")
    score, xs = fhtp.detect_polyline(torch.from_numpy(img).to(dev), k, bend=2)
    want, want_x = oracle.detect_polyline(img, k, bend=2)
    assert int(score.cpu()[0]) == want
    assert np.array_equal(xs.cpu().numpy(), want_x)
