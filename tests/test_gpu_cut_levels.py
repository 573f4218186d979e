"""The cut at view counts that move the border between the levels one
workgroup runs (at most 1,024 entries) and those with a launch of their own,
node-grouped and in plain order, against the oracle's cut."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_15186_amd.synth import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def setup():
    from paper_2603_15186_amd import hgs
    scene, cams = W.plan2m(scale=0.01, n_poses=150)
    r = hgs.Renderer(0)
    r.load_scene(scene)
    small = [type(c)(80, 45, c.fx / 16, c.fy / 16, c.cx / 16, c.cy / 16, c.position, c.R, c.znear, c.bg) for c in cams]
    yield r, scene, small, hgs
    r.close()


# 20,000 leaves: levels of 1, 1, 5, 40, 313, 2,500 and 20,000 nodes
@pytest.mark.parametrize("n", [1, 3, 4, 25, 26, 64, 65, 150])
@pytest.mark.parametrize("plain", [0, 1])
def test_cut_at_level_borders(setup, n, plain):
    r, scene, cams, hgs = setup
    r.set_option(hgs.HGS_OPT_KEEP_STATE, plain)      # renders that keep states use the plain order
    r.set_lod(hgs.HGS_LOD_THRESHOLD, 0.5)
    r.set_cameras(cams[:n])
    r.render()
    total = 0
    for v in sorted({0, 1, n // 2, n - 1, min(n - 1, 31), min(n - 1, 32), min(n - 1, 64)} & set(range(n))):
        got = r.get_cut(v)
        np.testing.assert_array_equal(got, O.cut(scene, cams[v], O.MODE_THRESHOLD, 0.5))
        total += got.size
    assert total > 0
    r.set_option(hgs.HGS_OPT_KEEP_STATE, 0)
