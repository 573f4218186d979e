"""Slice occupancy where a cell's mark could go wrong between the marking by
rows and the cell-by-cell definition: ellipses whose centres and extents lie
on cell edges, more planes than are listed at a time, ellipses of hundreds of
cells, grids beside the scene.  And discs at the widths where the map is read
eight cells at a time."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_15186_amd.synth import Scene

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    from paper_2603_15186_amd import hgs
    r = hgs.Renderer(0)
    yield r
    r.close()


def _scene(kind, n=1500):
    rng = np.random.default_rng(7)
    means = rng.uniform(0.0, 2.0, (n, 3))
    scales = np.exp(rng.uniform(np.log(0.01), np.log(0.2), (n, 3)))
    quats = rng.normal(size=(n, 4))
    opac = rng.uniform(0.3, 1.0, n)
    if kind == "edges":                      # axis-aligned, centres on the grid, slices through them
        means = np.round(means * 8.0) / 8.0
        quats[:] = (1.0, 0.0, 0.0, 0.0)
        scales = np.exp2(rng.integers(-6, -2, (n, 3)))
        opac[: n // 2] = 0.5                   # the slice through the centre is one point
    elif kind == "large":
        scales *= 20.0
    f = np.float32
    return Scene(means.astype(f), scales.astype(f), quats.astype(f), opac.astype(f), np.zeros((n, 1, 3), f), 0)


@pytest.mark.parametrize("kind, cell, n, planes, corner", [
    ("plain", 0.05, 45, 1, 0.0), ("plain", 0.05, 45, 16, 0.0), ("plain", 0.05, 45, 17, -0.013), ("plain", 0.05, 45, 40, 1.9),
    ("edges", 0.125, 18, 17, 0.0), ("edges", 0.0625, 36, 5, 0.0), ("large", 0.01, 200, 3, 0.0),
    ("plain", 0.3, 9, 20, 0.0), ("plain", 0.05, 45, 3, 50.0)])
def test_rows_equal_the_definition(R, kind, cell, n, planes, corner):
    s = _scene(kind)
    R.load_scene(s)
    h = (np.arange(planes) / 8.0 if kind == "edges" else np.linspace(0.05, 1.95, planes)).astype(np.float32)
    rho = 0.5 if kind != "large" else 0.1
    occ, m = R.slice_occupancy(corner, corner, cell, n, n + 3, h, rho_min=rho)
    g = occ.cpu().numpy()
    want = O.slice_occupancy(s.means, s.scales, s.quats, s.opacity, corner, corner, cell, n, n + 3, h, rho_min=rho)
    ok = (want == 2) | (g == want)
    assert ok.all(), f"{(~ok).sum()} of {ok.size} cells differ"
    assert corner == 50.0 or (want == 1).any()
    np.testing.assert_array_equal(m.cpu().numpy(), g.max(axis=0))


# boxes of 1 to 25 cells a side, cut by the grid's edges
@pytest.mark.parametrize("radius", [0.0, 0.1, 0.32, 0.36, 0.41, 0.75, 1.2])
def test_discs(R, radius):
    rng = np.random.default_rng(3)
    m = (rng.random((37, 41)) < 0.02).astype(np.uint8) * rng.integers(1, 256, (37, 41)).astype(np.uint8)
    xy = rng.uniform(-0.5, 4.6, (4000, 2))
    got = R.disc_collision(torch.from_numpy(m).cuda(), 0.0, 0.0, 0.1, torch.from_numpy(xy).cuda(), radius).cpu().numpy()
    want = O.disc_collision(m, 0.0, 0.0, 0.1, xy, radius)
    ok = (want == 2) | (got.astype(np.int8) == want)
    assert ok.all()
    assert radius == 0.0 or 0 < (want == 1).sum() < want.size
