"""The block kernel on every tile it has: bands of 3 to 2047 displacements under
scanned windows, with and without a through-point pin, at widths on both sides of
the columns' rules (one workgroup a CU: 1024, 2048 columns) and of a tile.
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


def _check(dev, img, k, pin=None, **bend):
    from paper_1912_01884_amd import fhtp
    announce(f"{img.shape} {img.dtype} k={k} {bend} pin={pin}")
    dimg = torch.from_numpy(img).to(dev)
    if pin is None:
        score, xs = fhtp.detect_polyline(dimg, k, **bend)
        want, want_x = oracle.detect_polyline(img, k, **bend)
    else:
        score, xs = fhtp.detect_polyline_ex(dimg, k, pin=pin, **bend)
        want, want_x = oracle.detect_ex(img, k, pin=pin, **bend)
    assert int(score.cpu()[0]) == want
    assert np.array_equal(xs.cpu().numpy(), want_x)


@pytest.mark.parametrize("n", [2, 8, 16, 32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("w", [1, 3, 4, 17, 300])
def test_every_tile(dev, n, w):
    rng = np.random.default_rng(1000 * n + w)
    k = 4 if n <= 256 else 3
    dtype = np.uint8 if (n + w) % 2 else np.uint16
    img = rng.integers(0, 4 if w == 17 else 256, size=(k * n, w)).astype(dtype)
    for gamma in (0.01, 0.2, 0.8):
        _check(dev, img, k, gamma=gamma)
    if n >= 16:
        _check(dev, img, k, bend=17)
    for j in (0, 1, k - 1, k):
        _check(dev, img, k, pin=(j, w // 2), gamma=0.2)
    _check(dev, img, k, pin=(1, w - 1), bend=10**6)


@pytest.mark.parametrize("w", [1024, 1025, 2048, 2049])
@pytest.mark.parametrize("n", [32, 64, 128, 256])
def test_columns_rule(dev, n, w):
    rng = np.random.default_rng(n + w)
    img = rng.integers(0, 256, size=(3 * n, w)).astype(np.uint8)
    _check(dev, img, 3, gamma=0.15)
    _check(dev, img, 3, pin=(2, w // 3), gamma=0.15)


def test_batch_of_every_tile(dev):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(5)
    imgs = [rng.integers(0, 256, size=(k * n, w)).astype(np.uint8)
            for n, w, k in [(16, 200, 5), (64, 333, 4), (128, 90, 3), (256, 70, 4), (512, 140, 2),
                            (1024, 33, 2), (32, 500, 9)]]
    ks = [5, 4, 3, 4, 2, 2, 9]
    announce("batch of scanned windows")
    got = fhtp.detect_batch([torch.from_numpy(i).to(dev) for i in imgs], ks, gammas=[0.1] * len(ks))
    torch.cuda.synchronize()
    for img, k, (score, xs) in zip(imgs, ks, got):
        want, want_x = oracle.detect_polyline(img, k, gamma=0.1)
        assert int(score.cpu()[0]) == want
        assert np.array_equal(xs.cpu().numpy(), want_x)
