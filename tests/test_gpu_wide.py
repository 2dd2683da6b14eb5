"""Wide images at the fixed-window steps' rules, against the oracle: two steps per
launch from four bands on whatever the width, 16 displacements per thread below,
stripes of an XCD's eighth of the column tiles (8192, 16384 columns)."""

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("w", [8192, 8193, 16384, 16449])
@pytest.mark.parametrize("n,k,bound", [(128, 2, 3), (128, 3, 8), (128, 4, 8), (128, 5, 16),
                                       (16, 9, 0)])
def test_wide(dev, w, n, k, bound):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(w + n + k)
    dtype = np.uint16 if k % 2 else np.uint8
    img = rng.integers(0, 256, size=(n * k, w)).astype(dtype)
    announce(f"wide {img.shape} {img.dtype} k={k} bound {bound}")
    score, xs = fhtp.detect_polyline(torch.from_numpy(img).to(dev), k, bend=bound)
    want, want_x = oracle.detect_polyline(img, k, bend=bound)
    assert int(score.cpu()[0]) == want
    assert np.array_equal(xs.cpu().numpy(), want_x)
