"""Binning through per-tile lists (few pairs) against binning through the two
sorts (everything else): the same images bit for bit.  A render takes the
lists when the last one counted few pairs, or at once for a small flat scene;
a batch of more than 8,192 tiles always sorts."""
import numpy as np
import pytest

from paper_2603_15186_amd.synth import Scene, make_random_box, workloads as W, yaw_camera

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def hgs():
    from paper_2603_15186_amd import hgs
    return hgs


def _images(outs):
    torch.cuda.synchronize()
    return [t.clone() for o in outs for t in o]


def _same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def _cluster(n, seed):
    """n small Gaussians that project into one 16x16 tile, a third of them at
    equal depths, and 500 others around them."""
    rng = np.random.default_rng(seed)
    means = np.concatenate([np.stack([rng.uniform(1.98, 2.0, n), rng.uniform(1.0, 3.0, n), rng.uniform(1.48, 1.5, n)], 1),
                            rng.uniform(0.0, 4.0, (500, 3))])
    means[: n // 3, 1] = 2.0
    m = len(means)
    return Scene(means.astype(np.float32), np.full((m, 3), 0.004, np.float32),
                 rng.normal(size=(m, 4)).astype(np.float32), rng.uniform(0.02, 0.3, m).astype(np.float32),
                 rng.normal(0.0, 0.5, (m, 1, 3)).astype(np.float32), 0)


# one tile's list around the ranked 256 pairs, the bitonic 4,096 and the merges of 2 to 5 runs
@pytest.mark.parametrize("n", [1, 255, 256, 257, 1023, 1025, 2049, 4096, 4097, 6000, 13000, 18000])
def test_long_lists_of_one_tile(hgs, n):
    cam = yaw_camera(512, 512, 512.0, (2.0, -1.0, 1.5), np.pi / 2)
    r = hgs.Renderer(0)
    r.load_scene(_cluster(n, n))
    r.set_cameras([cam])
    lists = _images(r.render())
    pairs = r.stats()["pairs"]
    r.set_cameras([cam] * 9)                       # 9,216 tiles: sorted
    outs = r.render()
    assert r.stats()["pairs"] == 9 * pairs
    _same(lists, _images(outs[:1]))
    r.close()


@pytest.mark.parametrize("views, w, h", [(1, 160, 90), (1, 161, 87), (3, 97, 61), (9, 64, 48)])
@pytest.mark.parametrize("options", [{}, {"HGS_OPT_EXACT_TILES": 0}, {"HGS_OPT_LOD_BLEND": 1}, {"HGS_OPT_KEEP_STATE": 1},
                                     {"HGS_OPT_LANES": 2}, {"HGS_OPT_PERSISTENT": 1}, {"HGS_OPT_COUNT_NALG": 1}])
def test_second_render_equals_the_first(hgs, views, w, h, options):
    scene, cams = W.plan2m(scale=0.005, n_poses=views)
    cams = [yaw_camera(w, h, 0.7 * w, c.position, 0.3 * i, bg=(0.1, 0.2, 0.3)) for i, c in enumerate(cams)]
    r = hgs.Renderer(0)
    r.load_scene(scene)
    for k, v in options.items():
        r.set_option(getattr(hgs, k), v)
    r.set_lod(hgs.HGS_LOD_THRESHOLD, 2.0)
    r.set_cameras(cams)
    first, a = _images(r.render()), r.stats()
    second, b = _images(r.render()), r.stats()
    _same(first, second)
    for k in ("cut_size", "visible", "pairs", "n_alg", "n_eval", "tiles"):
        assert a[k] == b[k], k
    assert b["pairs"] <= 512 * b["tiles"]          # the second one took the lists
    r.close()


@pytest.mark.parametrize("shape", [(8, 8, 1), (16, 8, 2), (32, 8, 1), (32, 16, 4)])
def test_tile_shapes(hgs, shape):
    r = hgs.Renderer(0)
    r.load_scene(make_random_box(5000, seed=2))
    cam = yaw_camera(251, 133, 200.0, (2.0, -1.0, 1.5), np.pi / 2)
    r.set_cameras([cam])
    want = _images(r.render())
    r.set_tile_shape(*shape)
    _same(want, _images(r.render()))
    r.close()


def test_graph_follows_the_choice(hgs):
    """A graph recorded with the sorts is recorded again with the lists once
    the pairs are known, and replays follow new poses."""
    scene, cams = W.plan2m(scale=0.005, n_poses=6)
    cams = [yaw_camera(128, 96, 100.0, c.position, 0.5 * i) for i, c in enumerate(cams)]
    r, g = hgs.Renderer(0), hgs.Renderer(0)
    for x in (r, g):
        x.load_scene(scene)
    g.set_option(hgs.HGS_OPT_USE_GRAPH, 1)
    for c in cams + cams:
        r.set_cameras([c])
        g.set_cameras([c])
        _same(_images(r.render()), _images(g.render()))
        torch.zeros(1000, device="cuda").add_(1.0).sum().item()
    assert g.stats()["graph_launches"] == 2 * len(cams)
    r.close()
    g.close()


def test_small_buffers_regrow(hgs):
    """Pair buffers that overflow in the lists grow and give the same image."""
    cam = yaw_camera(256, 256, 256.0, (2.0, -1.0, 1.5), np.pi / 2)
    r = hgs.Renderer(0)
    r.load_scene(make_random_box(20000, seed=0))
    r.set_cameras([cam])
    want = _images(r.render())
    r.set_option(hgs.HGS_OPT_INITIAL_CAPACITY, 1024)
    got = _images(r.render())
    assert r.stats()["regrows"] > 0
    _same(want, got)
    r.close()
