"""Batches of tiles on both sides of the count and the list length at which the
compositor takes two pixels per thread by itself: the first render (nothing
counted yet), the second and a replayed graph give the same images as a shape
set by hand."""
import math

import pytest

from paper_2603_15186_amd.synth import make_random_box, yaw_camera

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# 640 x 512 views of 1,280 tiles: 23,040, 24,320 and 25,600 tiles; few pairs, and some 700 per tile
@pytest.mark.parametrize("views, n", [(18, 3000), (19, 3000), (20, 3000), (20, 60000)])
def test_same_images(views, n):
    from paper_2603_15186_amd import hgs
    r = hgs.Renderer(0)
    r.load_scene(make_random_box(n, seed=3))
    r.set_cameras([yaw_camera(640, 512, 500.0, (2.0 + 0.01 * v, -1.0, 1.5), math.pi / 2) for v in range(views)])
    grab = lambda outs: [t.clone() for o in outs for t in o]  # noqa: E731
    first = grab(r.render())
    second = grab(r.render())
    r.set_option(hgs.HGS_OPT_USE_GRAPH, 1)
    outs = r.alloc_outputs()
    for _ in range(3):
        for o in outs:
            for t in o:
                t.zero_()
        r.render(outs)
    third = grab(outs)
    r.set_option(hgs.HGS_OPT_BATCH_DEPTH, 256)      # chosen: one pixel per thread
    fourth = grab(r.render())
    torch.cuda.synchronize()
    for a, b, c, d in zip(first, second, third, fourth):
        assert torch.equal(a, b) and torch.equal(a, c) and torch.equal(a, d)
    r.close()
