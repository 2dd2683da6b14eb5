"""The prepared image at the edges of its 64 x 64 tiles and at every alignment of
the output (four outputs are one store only where they are aligned)."""

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
@pytest.mark.parametrize("horizontal", [False, True])
@pytest.mark.parametrize("offset", [0, 1, 2, 3, 4])
def test_output_alignment(dev, dtype, horizontal, offset):
    from paper_1912_01884_amd import fhtp
    rng = np.random.default_rng(offset)
    for q, (h, w) in enumerate([(64, 64), (63, 68), (65, 129), (130, 61), (3, 200), (200, 4)]):
        radius = (offset + q) % 8
        img = rng.integers(0, np.iinfo(dtype).max + 1, size=(h, w)).astype(dtype)
        shape = (w, h) if horizontal else (h, w)
        flat = torch.zeros(h * w + 8, dtype=torch.from_numpy(img).dtype, device=dev)
        out = flat[offset:offset + h * w].view(shape)
        announce(f"prepare {h}x{w} {img.dtype} radius {radius} horizontal {horizontal} +{offset}")
        fhtp.prepare_image(torch.from_numpy(img).to(dev), radius, horizontal, out=out)
        want = oracle.smooth_rows(np.ascontiguousarray(img.T) if horizontal else img, radius)
        assert np.array_equal(out.cpu().numpy(), want)
        # nothing outside the image was written
        rest = torch.cat([flat[:offset].to(torch.int32), flat[offset + h * w:].to(torch.int32)])
        assert not rest.any()
