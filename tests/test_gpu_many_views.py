"""Batches whose (view, depth) keys exceed 32 bits, and node-grouped cuts of
more views than one LDS window holds: every view's image equals its render
alone, bit for bit."""
import dataclasses
import math

import numpy as np
import pytest

from paper_2603_15186_amd.synth import make_random_box, workloads as W, yaw_camera

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def setup():
    from paper_2603_15186_amd import hgs
    scene, cams = W.plan2m(scale=0.01, n_poses=150)
    r = hgs.Renderer(0)
    yield r, scene, cams, hgs
    r.set_option(hgs.HGS_OPT_SORT_DIGIT_BITS, 8)
    r.close()


def _images(outs):
    torch.cuda.synchronize()
    return [[t.clone() for t in o] for o in outs]


def _check(r, views, picks):
    r.set_cameras(views)
    got = _images(r.render())
    for v in picks:
        r.set_cameras([views[v]])
        for a, b in zip(_images(r.render())[0], got[v]):
            assert torch.equal(a, b), v


# 65 views: a second window of one view; 96 and 97: a full and a started
# third group; 150: windows that move more than once
@pytest.mark.parametrize("n, digit", [(65, 8), (96, 8), (97, 6), (150, 8), (150, 11)])
def test_batch_equals_single_views(setup, n, digit):
    r, scene, cams, hgs = setup
    r.load_scene(scene)
    r.set_lod(hgs.HGS_LOD_THRESHOLD, 1.0)
    r.set_option(hgs.HGS_OPT_SORT_DIGIT_BITS, digit)
    views = []
    for v in range(n):
        w, h = 40 + 8 * (v % 7), 30 + 3 * (v % 5)
        c = cams[v % len(cams)]
        views.append(yaw_camera(w, h, 0.7 * w, c.position, math.atan2(c.R[2][1], c.R[2][0]) + 0.05 * v))
    _check(r, views, sorted({0, 1, 31, 32, 63, 64, 66 % n, n // 2, n - 1}))
    assert r.stats()["passes"] == 1


# depths outside the estimated range: 32-bit depth keys, to which the first
# pass can add 8 bits of view number but not 9
@pytest.mark.parametrize("n", [3, 256, 257])
def test_full_depth_keys(setup, n):
    r, _, _, hgs = setup
    scene = make_random_box(3000, seed=5)
    r.load_scene(scene)
    r.set_option(hgs.HGS_OPT_SORT_DIGIT_BITS, 8)
    views = []
    for v in range(n):
        c = yaw_camera(24, 20, 18.0, (2.0 + 0.002 * v, 0.3, 1.5), math.pi / 2 + 0.01 * v)
        views.append(dataclasses.replace(c, R=(np.asarray(c.R, np.float32) * 3).astype(np.float32)))
    _check(r, views, sorted({0, 1, 2, n // 2, n - 1}))
