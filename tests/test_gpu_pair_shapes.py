"""Two steps per launch on both sides of the small grids' rule (256 workgroups of 64
columns and 32 displacements), every bound's tile remainders, with and without a
pin, against the oracle."""

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


# (n, w): workgroups of 32 displacements a column tile times column tiles
SHAPES = [(8, 1), (8, 63), (32, 200), (64, 4096), (64, 4097), (128, 2048), (128, 2049),
          (256, 1024), (256, 1025), (512, 130)]


@pytest.mark.parametrize("n,w", SHAPES)
@pytest.mark.parametrize("bound", [0, 1, 3, 4, 7, 8, 13, 16])
def test_small_and_usual_shape(dev, n, w, bound):
    from paper_1912_01884_amd import fhtp
    if bound >= 2 * n - 2:
        pytest.skip("no bend limit at this band height")
    rng = np.random.default_rng(n + w + bound)
    k = 4 + (bound + n) % 2
    dtype = np.uint8 if bound % 2 else np.uint16
    img = rng.integers(0, 3 if bound == 4 else 256, size=(k * n, w)).astype(dtype)
    dimg = torch.from_numpy(img).to(dev)
    announce(f"pairs {img.shape} {img.dtype} k={k} bound {bound}")
    score, xs = fhtp.detect_polyline(dimg, k, bend=bound)
    want, want_x = oracle.detect_polyline(img, k, bend=bound)
    assert int(score.cpu()[0]) == want
    assert np.array_equal(xs.cpu().numpy(), want_x)
    pin = (2, w // 2)
    score, xs = fhtp.detect_polyline_ex(dimg, k, bend=bound, pin=pin)
    want, want_x = oracle.detect_ex(img, k, bend=bound, pin=pin)
    assert int(score.cpu()[0]) == want
    assert np.array_equal(xs.cpu().numpy(), want_x)
