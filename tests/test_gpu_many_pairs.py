"""Per-tile lists of a view with more than 2^32 (tile, Gaussian) pairs: their
number does not wrap, so the overflow of the pair buffers is reported."""
import math

import numpy as np
import pytest

from paper_2603_15186_amd.synth import Scene, yaw_camera

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# 4,096 tiles (one step of the scan over the tiles) that every Gaussian covers:
# 2^32 + 4,096 * 16 pairs wrap to 65,536, fewer than the buffers hold
def test_pairs_past_32_bits():
    from paper_2603_15186_amd import hgs
    n = (1 << 20) + 16
    rng = np.random.default_rng(0)
    means = rng.uniform(-0.1, 0.1, (n, 3)) + (0.0, 5.0, 0.0)
    quats = np.tile(np.array([1, 0, 0, 0], np.float32), (n, 1))
    s = Scene(means.astype(np.float32), np.full((n, 3), 50.0, np.float32), quats, np.full(n, 0.01, np.float32),
              np.zeros((n, 1, 3), np.float32), 0)
    r = hgs.Renderer(0)
    r.load_scene(s)
    r.set_option(hgs.HGS_OPT_BINNING, 2)
    r.set_option(hgs.HGS_OPT_INITIAL_CAPACITY, n)           # entries and pairs
    r.set_option(hgs.HGS_OPT_SYNC_CHECK, 0)
    r.set_cameras([yaw_camera(1024, 1024, 500.0, (0.0, 0.0, 0.0), math.pi / 2)])
    r.render()
    torch.cuda.synchronize()
    st = r.stats()
    assert r.route()["lists"] and st["tiles"] == 4096
    assert st["visible"] == st["cut_size"] == n
    assert st["pairs"] == n                                  # the buffers' end, not the wrapped count
    r.close()
