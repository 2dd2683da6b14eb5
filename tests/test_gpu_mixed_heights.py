"""Batches of scanned windows whose images share launches of the block kernel: tiles of
every height and width, and a pack of more tiles than the chip holds many times over.
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


def _check(dev, imgs, ks, **bend):
    from paper_1912_01884_amd import fhtp
    announce(f"batch {[i.shape for i in imgs]} {bend}")
    got = fhtp.detect_batch([torch.from_numpy(i).to(dev) for i in imgs], ks,
                            bends=[bend.get("bend", 0)] * len(imgs),
                            gammas=[bend["gamma"]] * len(imgs) if "gamma" in bend else None)
    torch.cuda.synchronize()
    for q, (img, k, (score, xs)) in enumerate(zip(imgs, ks, got)):
        want, want_x = oracle.detect_polyline(img, k, **bend)
        assert int(score.cpu()[0]) == want, q
        assert np.array_equal(xs.cpu().numpy(), want_x), q


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("bend", [dict(gamma=0.02), dict(gamma=0.4), dict(bend=20), dict(bend=70)])
def test_heights_together(dev, dtype, bend):
    rng = np.random.default_rng(11)
    shapes = [(2, 100, 7), (4, 65, 3), (8, 17, 2), (32, 260, 4), (64, 129, 3), (128, 33, 5),
              (256, 70, 3), (512, 41, 2), (1024, 19, 2), (256, 301, 2)]
    imgs = [rng.integers(0, 5, size=(n * k, w)).astype(dtype) for n, w, k in shapes]
    _check(dev, imgs, [k for _, _, k in shapes], **bend)


@pytest.mark.parametrize("n,w,count", [(16, 9000, 8), (256, 9000, 8)])
def test_many_tiles(dev, n, w, count):
    rng = np.random.default_rng(n)
    k = 2
    shapes = [(n, w + 7 * q) for q in range(count)] + [(2 * n, 130)]
    imgs = [rng.integers(0, 256, size=(k * m, v)).astype(np.uint8) for m, v in shapes]
    _check(dev, imgs, [k] * len(imgs), gamma=0.2 if n == 16 else 0.03)
