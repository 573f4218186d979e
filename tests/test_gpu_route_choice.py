"""Which renders the choice of binning goes by: the renders of the last few
calls, counted whether or not they were checked, and nothing else that uses the
device's counters."""
import math

import pytest

from paper_2603_15186_amd.synth import make_random_box, workloads as W, yaw_camera

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def hgs():
    from paper_2603_15186_amd import hgs
    return hgs


def _views():
    """A view of few pairs (looking away from most of the scene) and one of many."""
    near = yaw_camera(640, 480, 640.0, (2.0, -1.0, 1.5), math.pi / 2)
    away = yaw_camera(640, 480, 640.0, (2.0, 3.7, 1.5), math.pi / 2)
    return away, near


@pytest.fixture()
def r(hgs):
    r = hgs.Renderer(0)
    r.load_scene(make_random_box(70000, seed=1))       # too many for the lists while nothing is counted
    r.set_option(hgs.HGS_OPT_TILE_SHAPE, (8 << 16) | 8)
    yield r
    r.close()


def _step(r, cam, outs=None):
    r.set_cameras([cam])
    outs = r.render(outs)
    torch.cuda.synchronize()
    return r.route()["lists"], r.stats()["pairs"], [t.clone() for o in outs for t in o]


@pytest.mark.parametrize("graph", [0, 1])
def test_alternating_views_keep_to_the_sorts(hgs, r, graph):
    """Light and heavy views in turn: the heavy ones are never listed because
    the light one before them was counted."""
    r.set_option(hgs.HGS_OPT_USE_GRAPH, graph)
    light, heavy = _views()
    _, few, _ = _step(r, light)
    assert few <= 1 << 18
    assert _step(r, light)[0]
    _, many, want = _step(r, heavy)
    assert many > 1 << 19
    for _ in range(4):
        _step(r, light)
        lists, _, img = _step(r, heavy)
        assert not lists
        assert all(torch.equal(a, b) for a, b in zip(want, img))
    for _ in range(20):                                 # the heavy ones are over
        lists = _step(r, light)[0]
    assert lists


@pytest.mark.parametrize("graph", [0, 1])
def test_streams_without_checks_learn_their_pairs(hgs, r, graph):
    light, heavy = _views()
    want = _step(r, heavy)[2]
    r.set_option(hgs.HGS_OPT_TILE_SHAPE, (16 << 16) | 16)   # forget the counts
    r.set_option(hgs.HGS_OPT_TILE_SHAPE, (8 << 16) | 8)
    r.set_option(hgs.HGS_OPT_USE_GRAPH, graph)
    r.set_option(hgs.HGS_OPT_SYNC_CHECK, 0)
    outs = r.alloc_outputs()
    assert not _step(r, light, outs)[0]
    assert _step(r, light, outs)[0]
    for k in range(3):
        lists, _, img = _step(r, heavy, outs)
        assert all(torch.equal(a, b) for a, b in zip(want, img))
        assert lists == (k == 0)
    assert r.check() == hgs.HGS_OK


def test_candidates_are_not_counted_as_a_render(hgs):
    """Collecting candidates uses the same device counters; the next render
    still goes by the last render."""
    scene, cams = W.plan2m(scale=0.1, n_poses=1)
    r = hgs.Renderer(0)
    r.load_scene(scene)
    r.set_option(hgs.HGS_OPT_TILE_SHAPE, (8 << 16) | 8)
    r.set_option(hgs.HGS_OPT_EXACT_TILES, 0)
    r.set_lod(hgs.HGS_LOD_THRESHOLD, 1.0)
    r.set_cameras([yaw_camera(640, 480, 450.0, cams[0].position, math.atan2(cams[0].R[2][1], cams[0].R[2][0]))])
    r.render()
    assert r.stats()["pairs"] > 1 << 18
    r.render()
    assert not r.route()["lists"]
    r.lod_candidates(64.0)
    assert r.check() == hgs.HGS_OK
    r.render()
    assert not r.route()["lists"]
    r.close()


def test_backward_after_each_replay(hgs):
    """Gradients of renders replayed from either choice's graph, whichever was
    recorded last: the pairs are read where that render left them."""
    light, heavy = _views()
    plain, graph = hgs.Renderer(0), hgs.Renderer(0)
    for r in (plain, graph):
        r.load_scene(make_random_box(100000, seed=1))
        r.set_cameras([light])
        r.set_option(hgs.HGS_OPT_BINNING, 1 if r is plain else 0)
    graph.set_option(hgs.HGS_OPT_USE_GRAPH, 1)
    gen = torch.Generator(device="cuda").manual_seed(3)
    routes = []
    for cam in [light, light, heavy, heavy, heavy, heavy, light] + [light] * 9 + [heavy]:
        got = []
        for r in (plain, graph):
            r.set_cameras([cam])
            outs = r.render()
            grads = [tuple(torch.randn(t.shape, generator=gen.manual_seed(7), device="cuda") for t in outs[0])]
            got.append(r.backward(grads))
        torch.cuda.synchronize()
        routes.append(graph.route()["lists"])
        for k in got[0]:
            a, b = got[0][k].double(), got[1][k].double()
            # equal but for the order of the atomic sums
            assert ((a - b).abs() <= 1e-4 * a.abs() + 1e-5 * a.abs().max()).all(), (len(routes), k)
    assert routes[0] is False and routes[1] is True and routes[6] is False and routes[-1] is True
    plain.close()
    graph.close()
