"""Windows of a few rows, inside a block of the block kernel's rows and across the
ends of blocks, with many equal cells (the smallest displacement has to win).
Everything is integer, so results equal the oracle's.
"""

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


# mean windows of about 1, 4, 8 and 16 rows
@pytest.mark.parametrize("rows", [1, 4, 8, 16])
@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 1024])
def test_short_windows(dev, n, rows):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(n + rows)
    k = 4 if n <= 256 else 3
    gamma = rows / (2.67 * n)
    for w in (5, 70, 300):
        for dtype, top in ((np.uint8, 2), (np.uint16, 300)):
            img = rng.integers(0, top, size=(k * n, w)).astype(dtype)
            announce(f"{img.shape} {img.dtype} k={k} gamma={gamma}")
            score, xs = fhtp.detect_polyline(torch.from_numpy(img).to(dev), k, gamma=gamma)
            want, want_x = oracle.detect_polyline(img, k, gamma=gamma)
            assert int(score.cpu()[0]) == want
            assert np.array_equal(xs.cpu().numpy(), want_x)
