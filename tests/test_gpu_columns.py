"""The column recurrence on both sides of its columns' rule (one workgroup a CU: 2048,
4096 columns), and images alone on a workgroup whose 4-row sums need more than 64 KB
of LDS, against the oracle."""

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _check(dev, img, k, **bend):
    from paper_1912_01884_amd import fhtp
    announce(f"{img.shape} {img.dtype} k={k} {bend}")
    score, xs = fhtp.detect_polyline(torch.from_numpy(img).to(dev), k, **bend)
    want, want_x = oracle.detect_polyline(img, k, **bend)
    assert int(score.cpu()[0]) == want
    assert np.array_equal(xs.cpu().numpy(), want_x)


@pytest.mark.parametrize("w", [7, 9, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("n", [2, 16, 64, 128, 512])
def test_column_recurrence(dev, w, n):
    rng = np.random.default_rng(w + n)
    dtype = np.uint8 if (w + n) % 2 else np.uint16
    img = rng.integers(0, 3 if w < 10 else 256, size=(3 * n, w)).astype(dtype)
    _check(dev, img, 3, bend=10**6)


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("n,w,k", [(8, 80, 12), (8, 250, 3), (16, 100, 3), (32, 60, 1), (4, 60, 45)])
@pytest.mark.parametrize("bend", [dict(bend=1), dict(bend=6), dict(bend=10**6), dict(gamma=0.4)])
def test_alone_on_a_workgroup(dev, dtype, n, w, k, bend):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(n + w)
    img = rng.integers(0, np.iinfo(dtype).max + 1, size=(k * n, w)).astype(dtype)
    fhtp.timing_start()
    _check(dev, img, k, **bend)
    assert set(fhtp.timing_stop()) == {"detect_small"}
