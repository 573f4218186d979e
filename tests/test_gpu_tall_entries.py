"""Entries of many tile rows are counted and listed by their own lane or by
their whole wave, depending on their neighbours: the tiles found are the same."""
import math

import numpy as np
import pytest

from paper_2603_15186_amd.synth import Scene, yaw_camera

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _scene(tall, small, seed):
    """Elongated, tilted Gaussians that span many tile rows, then small ones."""
    rng = np.random.default_rng(seed)
    n = tall + small
    means = rng.uniform((-2.0, 2.0, -1.5), (2.0, 6.0, 1.5), (n, 3))
    scales = np.exp(rng.uniform(math.log(0.005), math.log(0.02), (n, 3)))
    scales[:tall] = np.exp(rng.uniform(math.log(0.005), math.log(1.0), (tall, 3)))
    f = np.float32
    return Scene(means.astype(f), scales.astype(f), rng.normal(size=(n, 4)).astype(f),
                 rng.uniform(0.02, 0.2, n).astype(f), rng.normal(0.0, 0.5, (n, 1, 3)).astype(f), 0)


@pytest.mark.parametrize("binning", [1, 2])
@pytest.mark.parametrize("w, h", [(640, 512), (333, 1001)])
def test_alone_and_together(w, h, binning):
    from paper_2603_15186_amd import hgs
    tall, small = 512, 512 * 63
    s = _scene(tall, small, 1)
    together = np.arange(tall + small)                      # eight waves of tall ones
    alone = np.concatenate([np.concatenate([[k], tall + 63 * k + np.arange(63)]) for k in range(tall)])
    r = hgs.Renderer(0)
    r.set_option(hgs.HGS_OPT_BINNING, binning)
    counts, images, pairs = [], [], []
    for order in (together, alone):
        r.load_scene(Scene(s.means[order], s.scales[order], s.quats[order], s.opacity[order], s.sh[order], 0))
        r.set_cameras([yaw_camera(w, h, 400.0, (0.0, 0.0, 0.0), math.pi / 2)])
        outs = r.render()
        assert r.route()["lists"] == (binning == 2)
        torch.cuda.synchronize()
        n = np.empty(len(order))
        n[order] = r.get_projected(0)[:, 10]
        counts.append(n)
        images.append([t.clone() for t in outs[0]])
        pairs.append(r.stats()["pairs"])
    assert (counts[0][:tall] > 64).sum() > 100
    np.testing.assert_array_equal(counts[0], counts[1])
    assert pairs[0] == pairs[1] == counts[0].sum()
    for a, b in zip(*images):
        assert torch.equal(a, b)
    r.close()
