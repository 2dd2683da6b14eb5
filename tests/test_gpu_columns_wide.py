"""The column recurrence with 64 columns a workgroup: wide images and packs of many
columns, on both sides of the line.  Integer results, equal to the oracle's.
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


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("n", [2, 16, 128, 512])
@pytest.mark.parametrize("w", [8192, 8193, 8257])
def test_wide(dev, n, w, dtype):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(n + w)
    img = rng.integers(0, 6, size=(3 * n, w)).astype(dtype)
    announce(f"{img.shape} {img.dtype} no limit")
    score, xs = fhtp.detect_polyline(torch.from_numpy(img).to(dev), 3, bend=10**6)
    want, want_x = oracle.detect_polyline(img, 3, bend=10**6)
    assert int(score.cpu()[0]) == want
    assert np.array_equal(xs.cpu().numpy(), want_x)


@pytest.mark.parametrize("count", [8, 9, 20])
def test_packs(dev, count):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(count)
    shapes = [((4, 32, 64)[q % 3], 1000 + q % 5, 2 + q % 4) for q in range(count)]
    imgs = [rng.integers(0, 256, size=(n * k, w)).astype(np.uint8) for n, w, k in shapes]
    ks = [k for _, _, k in shapes]
    announce(f"pack of {count} without a limit")
    got = fhtp.detect_batch([torch.from_numpy(i).to(dev) for i in imgs], ks, bends=[10**6] * count)
    torch.cuda.synchronize()
    for img, k, (score, xs) in zip(imgs, ks, got):
        want, want_x = oracle.detect_polyline(img, k, bend=10**6)
        assert int(score.cpu()[0]) == want
        assert np.array_equal(xs.cpu().numpy(), want_x)
