"""Replayed renders whose poses reach depths that the recorded one did not: a
graph's depth keys cover every pose it is replayed with."""
import math

import pytest

from paper_2603_15186_amd.synth import make_random_box, yaw_camera

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _poses(views):
    """Inside the 4 x 4 x 3 m box, 3 m before it, then 60 and 900 m away (and back)."""
    for d in (-1.5, 3.0, 60.0, 900.0, 3.0, -1.5):
        yield [yaw_camera(160, 120, 120.0 * max(1.0, d), (2.0 + 0.1 * v, -d, 1.5), math.pi / 2) for v in range(views)]


@pytest.mark.parametrize("checks", [0, 1])
@pytest.mark.parametrize("views, binning", [(1, 1), (1, 2), (3, 1), (70, 1)])
def test_replays_at_other_depths(views, binning, checks):
    from paper_2603_15186_amd import hgs
    plain, graph = hgs.Renderer(0), hgs.Renderer(0)
    for r in (plain, graph):
        r.load_scene(make_random_box(3000, seed=5))
        r.set_option(hgs.HGS_OPT_BINNING, binning)
    graph.set_option(hgs.HGS_OPT_USE_GRAPH, 1)
    graph.set_option(hgs.HGS_OPT_SYNC_CHECK, checks)
    outs = None
    for cams in _poses(views):
        plain.set_cameras(cams)
        want = plain.render()
        graph.set_cameras(cams)
        outs = graph.render(outs)
        torch.cuda.synchronize()
        assert graph.check() == hgs.HGS_OK
        assert graph.stats()["regrows"] == 0
        for a, b in zip(want, outs):
            for x, y in zip(a, b):
                assert torch.equal(x, y)
    assert graph.stats()["graph_launches"] == 6
    plain.close()
    graph.close()
