"""Packs whose step launches have 2^32 threads or more and go out in several dispatches.

Images of few rows and 2^20 columns, two contents dealt to all jobs of a batch, so
that an image of every dispatch is compared with the oracle.
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


@pytest.mark.parametrize("count,h,bend", [(66, 2, dict(bend=1 << 20)), (70, 4, dict(gamma=0.3)),
                                          (130, 4, dict(bend=1 << 20)), (256, 4, dict(bend=1 << 20))])
def test_packs_of_the_widest_images(dev, count, h, bend):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(count)
    w, k = 1 << 20, 2
    imgs = [rng.integers(0, 250, size=(h, w)).astype(np.uint8) for _ in range(2)]
    for q, x in enumerate((777, w - 888)):  # one best polyline each, far apart
        imgs[q][:, x] = 255
    want = [oracle.detect_polyline(i, k, **bend) for i in imgs]
    dimg = [torch.from_numpy(i).to(dev) for i in imgs]
    jobs = [dimg[q % 2] for q in range(count)]
    announce(f"batch of {count} images {h}x{w} {bend}")
    got = fhtp.detect_batch(jobs, [k] * count, bends=[bend.get("bend", 0)] * count,
                            gammas=[bend["gamma"]] * count if "gamma" in bend else None)
    scores = torch.cat([s for s, _ in got]).cpu().numpy()
    xs = torch.stack([x for _, x in got]).cpu().numpy()
    for q in range(count):
        assert scores[q] == want[q % 2][0], q
        assert np.array_equal(xs[q], want[q % 2][1]), q
