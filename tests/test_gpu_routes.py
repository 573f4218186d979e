"""The renderer's two ways of binning (radix sorts, per-tile lists) and its
compositor shapes, each forced and checked to be the one that ran; and the
rule that picks one by itself, by what it picked.

Scenes small enough for the lists take them without being asked, so checks of
the sorts (digit widths, full-width depth keys, all-tiles rectangles, tile
shapes) ask for the sorts here."""
import dataclasses
import math

import numpy as np
import pytest

from paper_2603_15186_amd.synth import make_random_box, workloads as W, yaw_camera
from tests import parity
from oracle import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SORTS, LISTS = 1, 2


@pytest.fixture(scope="module")
def hgs():
    from paper_2603_15186_amd import hgs
    return hgs


@pytest.fixture(scope="module")
def box():
    return W.box20k()


def _images(outs):
    torch.cuda.synchronize()
    return [t.clone() for o in outs for t in o]


def _same(a, b, label=""):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert torch.equal(x, y), label


def _render(hgs, r, binning, **opts):
    r.set_option(hgs.HGS_OPT_BINNING, binning)
    for k, v in opts.items():
        r.set_option(getattr(hgs, "HGS_OPT_" + k), v)
    img = _images(r.render())
    assert r.route()["lists"] == (binning == LISTS), (binning, opts)
    return img


def _check_full(img, scene, cam):
    res, _, _ = O.render(scene, cam, O.MODE_THRESHOLD, 1.0)
    g = parity.gpu_pixels(*[t.cpu().numpy() for t in img], res.px, res.py)
    ok, best, skipped = parity.branch_errors(g, res)
    assert ok.all() and not skipped.any(), parity.summary(ok, best, skipped)


@pytest.mark.parametrize("binning", [SORTS, LISTS])
def test_box_by_each_route(hgs, box, binning):
    """Oracle parity, and the same image for every digit width and both tile sets."""
    scene, cams = box
    r = hgs.Renderer(0)
    r.load_scene(scene)
    r.set_cameras(cams)
    ref = _render(hgs, r, binning)
    _check_full(ref, scene, cams[0])
    for d in (6, 7, 9, 10, 11):
        _same(ref, _render(hgs, r, binning, SORT_DIGIT_BITS=d), d)
    pairs = r.stats()["pairs"]
    _same(ref, _render(hgs, r, binning, EXACT_TILES=0), "all tiles")
    assert r.stats()["pairs"] > pairs
    r.close()


@pytest.mark.parametrize("binning", [SORTS, LISTS])
def test_full_width_depth_keys_by_each_route(hgs, box, binning):
    """A camera matrix scaled by 3 leaves the depth keys' range: the render is
    redone with full keys, by the same route, and matches the oracle."""
    scene, cams = box
    cam = dataclasses.replace(cams[0], R=(np.asarray(cams[0].R, np.float32) * 3).astype(np.float32))
    r = hgs.Renderer(0)
    r.load_scene(scene)
    r.set_cameras([cam])
    img = _render(hgs, r, binning)
    assert r.stats()["regrows"] >= 1
    _check_full(img, scene, cam)
    r.close()


@pytest.mark.parametrize("shape", [(8, 8, 1), (16, 8, 2), (16, 16, 2), (32, 8, 1), (32, 16, 4)])
def test_tile_shapes_by_each_route(hgs, shape):
    r = hgs.Renderer(0)
    r.load_scene(make_random_box(5000, seed=2))
    r.set_cameras([yaw_camera(251, 133, 200.0, (2.0, -1.0, 1.5), math.pi / 2)])
    want = _render(hgs, r, SORTS)
    r.set_tile_shape(*shape)
    for binning in (SORTS, LISTS):
        _same(want, _render(hgs, r, binning), (shape, binning))
        assert r.route()["pixels_per_thread"] == shape[2]
    r.close()


def test_views_in_the_sort_keys(hgs):
    """Batches of views by each route, with wide depth keys too (the views then
    join the key in the sort's first pass or follow in a pass of their own)."""
    scene = make_random_box(3000, seed=4)
    cams = [yaw_camera(97, 61, 80.0, (2.0 + 0.02 * v, -1.0, 1.5), math.pi / 2) for v in range(70)]
    wide = [dataclasses.replace(c, R=(np.asarray(c.R, np.float32) * 3).astype(np.float32)) for c in cams]
    for views in (cams, wide):
        r = hgs.Renderer(0)
        r.load_scene(scene)
        r.set_cameras(views)
        ref = _render(hgs, r, LISTS)
        for d in (6, 8, 11):
            _same(ref, _render(hgs, r, SORTS, SORT_DIGIT_BITS=d), d)
        r.close()


def test_rule_of_the_lists(hgs):
    """A hierarchical scene sorts while nothing is counted, then lists; a small
    flat scene lists at once; more than 8,192 tiles a pass sort."""
    scene, cams = W.plan2m(scale=0.005, n_poses=1)
    cam = yaw_camera(160, 90, 112.0, cams[0].position, 0.3)
    r = hgs.Renderer(0)
    with pytest.raises(hgs.HgsError):
        r.route()
    r.load_scene(scene)
    r.set_cameras([cam])
    first = _images(r.render())
    assert not r.route()["lists"]
    second = _images(r.render())
    assert r.route()["lists"]
    _same(first, second)
    r.load_scene(make_random_box(5000, seed=2))
    r.set_cameras([cam])
    r.render()
    assert r.route()["lists"]
    r.set_option(hgs.HGS_OPT_BINNING, LISTS)
    r.set_cameras([yaw_camera(1024, 1024, 900.0, (2.0, -1.0, 1.5), math.pi / 2)] * 3)
    r.render()
    assert not r.route()["lists"]
    with pytest.raises(hgs.HgsError):
        r.set_option(hgs.HGS_OPT_BINNING, 3)
    r.close()


# 1,280 tiles a view: 24,320 tiles are too few for two pixels a thread, 25,600 not, unless their lists are long
@pytest.mark.parametrize("views, n, px", [(19, 3000, 1), (20, 3000, 2), (20, 200000, 1)])
def test_rule_of_the_shape(hgs, views, n, px):
    r = hgs.Renderer(0)
    r.load_scene(make_random_box(n, seed=3))
    r.set_cameras([yaw_camera(640, 512, 500.0, (2.0 + 0.01 * v, -1.0, 1.5), math.pi / 2) for v in range(views)])
    r.render()
    assert r.route()["pixels_per_thread"] == 1
    r.render()
    assert r.route()["pixels_per_thread"] == px
    st = r.stats()
    assert (st["pairs"] <= 384 * st["tiles"]) == (n == 3000)
    r.set_option(hgs.HGS_OPT_BATCH_DEPTH, 256)      # chosen by hand
    r.render()
    assert r.route()["pixels_per_thread"] == 1
    r.close()
