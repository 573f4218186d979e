"""Window errors and labels of images cut into several row chunks, against
numpy in float64 (the float32 result is the rounded float64 mean: 2^-24
relative, plus float64 summation error)."""
import math

import numpy as np
import pytest
import torch

from paper_2603_15186_amd import hgs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    r = hgs.Renderer(0)
    yield r
    r.close()


# (window w, h, reference W, H, x0, y0): 16-byte rows or not, one chunk, a last chunk of one row, rows longer than
# a chunk, more rows than chunks of the usual size, single pixels
SHAPES = [(1280, 720, 1280, 720, 0, 0), (1001, 61, 1003, 70, 1, 9), (256, 22, 512, 40, 4, 3), (256, 64, 260, 64, 2, 0),
          (20004, 2, 20004, 2, 0, 0), (3, 6000, 8, 6001, 4, 1), (1, 1, 5, 5, 3, 4), (64, 85, 64, 85, 0, 0)]


def _images(rng, w, h, W, H, x0, y0):
    ref = rng.uniform(size=(3, H, W)).astype(np.float32)
    crop = ref[:, y0:y0 + h, x0:x0 + w]
    return ref, crop, (crop + rng.normal(size=crop.shape) * 0.05).astype(np.float32)


def test_region_mse_over_chunks(R):
    rng = np.random.default_rng(5)
    regions, want = [], []
    for s in SHAPES:
        ref, crop, img = _images(rng, *s)
        regions.append((torch.from_numpy(img).cuda(), torch.from_numpy(ref).cuda(), s[4], s[5]))
        want.append(((img.astype(np.float64) - crop) ** 2).mean())
    out = torch.full((len(SHAPES),), -1.0, dtype=torch.float32, device="cuda")
    R.region_mse(regions, out)
    np.testing.assert_allclose(out.cpu().numpy(), want, rtol=1.2e-7)
    for i in (0, 5, 6):                      # alone: other chunk numbers, the same value
        one = torch.empty(1, dtype=torch.float32, device="cuda")
        R.region_mse(regions[i:i + 1], one)
        np.testing.assert_allclose(one.item(), want[i], rtol=1.2e-7)


def test_lod_labels_over_chunks(R):
    rng = np.random.default_rng(6)
    pairs, drop = [], []
    for s in SHAPES:
        ref, crop, a = _images(rng, *s)
        b = (a + rng.normal(size=a.shape) * 0.03).astype(np.float32)
        pairs.append((torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), torch.from_numpy(ref).cuda(), s[4], s[5]))
        ea, eb = (max(((x.astype(np.float64) - crop) ** 2).mean(), 1e-10) for x in (a, b))
        drop.append(10.0 * math.log10(eb / ea))
    labels, got = R.lod_labels(pairs, 0.05)
    # two errors of 2^-24 in 10 log10 of their ratio: 5.2e-7 dB, and the float32 result
    np.testing.assert_allclose(got.cpu().numpy(), drop, rtol=1.2e-7, atol=6e-7)
    np.testing.assert_array_equal(labels.cpu().numpy(), (np.array(drop) > 0.05).astype(np.float32))
