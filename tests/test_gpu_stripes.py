"""Batches of images with stripes of different widths in the order of the multi-step
kernels' workgroups, set by rules and by the images' widths.  Integer results, equal
to the oracle's.
"""

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [2, 3])
def test_stripes_of_a_batch(steps):
    from paper_1912_01884_amd import autotune, fhtp
    dev = require_gpu()
    rng = np.random.default_rng(steps)
    shapes = [(8, 300, 6), (8, 9000, 8), (16, 12000, 7), (32, 2100, 5), (128, 1500, 6)]
    imgs = [rng.integers(0, 256, size=(n * k, w)).astype(np.uint8) for n, w, k in shapes]
    ks = [k for _, _, k in shapes]
    fhtp.tune_set([autotune.rule(window=0, steps=steps, stripe=1, w_max=1000),
                   autotune.rule(window=0, steps=steps, stripe=5, w_max=2200),
                   autotune.rule(window=0, steps=steps)])
    try:
        announce(f"batch with stripes of different widths, {steps} steps a launch")
        got = fhtp.detect_batch([torch.from_numpy(i).to(dev) for i in imgs], ks, bends=[3] * len(ks))
        torch.cuda.synchronize()
    finally:
        fhtp.tune_set([])
    for img, k, (score, xs) in zip(imgs, ks, got):
        want, want_x = oracle.detect_polyline(img, k, bend=3)
        assert int(score.cpu()[0]) == want
        assert np.array_equal(xs.cpu().numpy(), want_x)
