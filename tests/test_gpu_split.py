"""Band transform at the edges of the split kernel's tiles, against the oracle.

A workgroup of the split kernel makes 228 columns (240 for 32-row bands) of the
w + n wide table, in two halves of 114 (120); bands are chosen on both sides of
each rule (32 rows up to 128 of 8-bit pixels, 64 up to 256 of 16-bit ones, the
rest by other kernels).  Everything is integer, so results are equal.
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


def _image(rng, h, w, dtype, saturated):
    top = np.iinfo(dtype).max
    if saturated:
        return np.full((h, w), top, dtype=dtype)
    return rng.integers(0, top + 1, size=(h, w)).astype(dtype)


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("n", [16, 32, 64, 128, 256, 512, 1024])
def test_tables_at_tile_edges(dev, n, dtype):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(n)
    tile = 240 if n == 32 else 228
    widths = {1, 2, n - 1, n}
    for cols in (tile // 2, tile, tile + 1, 2 * tile - 1, 2 * tile, 5 * tile + 1):
        widths.update(w for w in (cols - n, cols - n + 1) if w > 0)
    for q, w in enumerate(sorted(widths)):
        k = 1 + q % 2
        img = _image(rng, k * n, w, dtype, q % 5 == 4)
        announce(f"tables {k * n}x{w} k={k} {img.dtype}")
        got = fhtp.fht_bands(torch.from_numpy(img).to(dev), k).cpu().numpy()
        assert np.array_equal(got, oracle.fht_bands(img, k))


@pytest.mark.parametrize("dtype,n", [(np.uint8, 32), (np.uint8, 128), (np.uint8, 256),
                                     (np.uint16, 64), (np.uint16, 256)])
@pytest.mark.parametrize("w", [229, 700, 1001])
def test_detection_from_an_unaligned_image(dev, dtype, n, w):
    """An image that starts one pixel into its allocation, odd widths: every
    row's alignment occurs (8-bit images keep 16-bit tables)."""
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(w)
    img = _image(rng, 3 * n, w, dtype, False)
    flat = torch.zeros(img.size + 1, dtype=torch.from_numpy(img).dtype, device=dev)
    view = flat[1:].view(img.shape)
    view.copy_(torch.from_numpy(img))
    announce(f"detection {img.shape} {img.dtype} one pixel off")
    score, xs = fhtp.detect_polyline(view, 3, bend=3)
    want, want_x = oracle.detect_polyline(img, 3, bend=3)
    assert int(score.cpu()[0]) == want
    assert np.array_equal(xs.cpu().numpy(), want_x)
