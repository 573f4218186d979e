"""Slices of very large and elongated Gaussians: the marking by rows gives what
the cell-by-cell definition gives.  Scaled by a power of two, a scene and its
grid keep every digit of the definition's arithmetic, and at 2^-70 a Gaussian's
inverse covariance passes the range that the rows serve (1e30), so that the
scaled call takes the definition."""
import math

import numpy as np
import pytest

from paper_2603_15186_amd.synth import Scene

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, CELL, RHO = 256, 2.0 ** -7, 0.25
CELLS = 128


def _scene(cells, aspect, tip, seed):
    """One flat Gaussian per plane (1 m apart), its long axis `cells` cells at
    sigma, turned at random; the window holds an arc of its solid ellipse, or
    the ellipse's top, where a row's width is known least well."""
    rng = np.random.default_rng(seed)
    f = np.float32
    long_ = cells * CELL * rng.uniform(0.5, 1.0, N)
    scales = np.stack([long_, long_ / aspect, np.full(N, 1e-3)], 1).astype(f)
    yaw = rng.uniform(0.0, 2.0 * math.pi, N)
    tilt = rng.uniform(-1.0, 1.0, (N, 2)) * (3e-5 / long_)[:, None]      # (the slice keeps its size)
    quats = np.stack([np.cos(yaw / 2), tilt[:, 0], tilt[:, 1], np.sin(yaw / 2)], 1).astype(f)
    opac = rng.uniform(0.26, 1.0, N).astype(f)
    r = np.sqrt(2.0 * np.log(opac.astype(float) / RHO))
    a, b, c, s = scales[:, 0], scales[:, 1], np.cos(yaw), np.sin(yaw)
    phi = np.arctan2(b * c, a * s) if tip else rng.uniform(0.0, 2.0 * math.pi, N)
    ex, ey = r * a * np.cos(phi), r * b * np.sin(phi)
    at = rng.uniform(0.3, 0.7, (N, 2)) * CELLS * CELL
    means = np.stack([at[:, 0] - (ex * c - ey * s), at[:, 1] - (ex * s + ey * c), np.arange(N)], 1).astype(f)
    return Scene(means, scales, quats, opac, np.zeros((N, 1, 3), f), 0)


def _occ(r, s, k):
    """Occupancy of the scene and its grid scaled by 2^k."""
    f = np.float32(2.0) ** k
    r.load_scene(Scene(s.means * f, s.scales * f, s.quats, s.opacity, s.sh, 0))
    h = np.arange(N, dtype=np.float32) * f
    return r.slice_occupancy(0.0, 0.0, CELL * 2.0 ** k, CELLS, CELLS, h, rho_min=RHO)[0]


@pytest.mark.parametrize("aspect", [1.5, 30.0, 600.0])
@pytest.mark.parametrize("cells", [1e2, 1e4, 1e6, 3e7])
@pytest.mark.parametrize("tip", [False, True])
def test_rows_equal_the_definition(tip, cells, aspect):
    from paper_2603_15186_amd import hgs
    r = hgs.Renderer(0)
    s = _scene(cells, aspect, tip, 0)
    rows, cells_ = _occ(r, s, 0), _occ(r, s, -70)
    d, marked = int((rows != cells_).sum()), float(rows.float().mean())
    print(f"{cells:g} cells, tip {tip}, aspect {aspect}: {d} cells differ, {marked:.3f} marked", flush=True)
    assert 0.0 < marked < 1.0
    assert d == 0
    r.close()


def _edge_grids(seed):
    """A Gaussian a million cells long, 600 times its width, and grids of 4 x 4
    cells near its slice's top whose columns meet the slice's right end in
    one row within 3e-5 cells."""
    rng = np.random.default_rng(seed)
    f, ld = np.float32, np.longdouble
    long_ = 2.0 ** 20 * CELL * rng.uniform(0.7, 1.0)
    yaw = rng.uniform(0.7, 0.87)
    scales = np.array([[long_, long_ / 600.0, 1e-3]], f)
    quats = np.array([[math.cos(yaw / 2), 0.0, 0.0, math.sin(yaw / 2)]], f)
    s = Scene(rng.uniform(-0.5, 0.5, (1, 3)).astype(f) * (1, 1, 0), scales, quats, np.array([0.9], f),
              np.zeros((1, 1, 3), f), 0)
    s.means = s.means.astype(f)
    w, z = ld(quats[0, 0]), ld(quats[0, 3])
    n = w * w + z * z
    c, sn = (w * w - z * z) / n, 2 * w * z / n
    ia, ib = 1 / ld(scales[0, 0]) ** 2, 1 / ld(scales[0, 1]) ** 2
    A, B, C = c * c * ia + sn * sn * ib, c * sn * (ia - ib), sn * sn * ia + c * c * ib
    det = ia * ib
    r2 = 2 * np.log(ld(f(0.9)) / ld(RHO))
    mx, my = ld(s.means[0, 0]), ld(s.means[0, 1])
    top = np.sqrt(r2 * A / det)
    y = float(my + top - ld(rng.uniform(4.0, 40.0)) * CELL)           # upper edge of the row
    dy = ld(y) - my                                                   # its right end lies lower: leftward slope
    lo = dy - CELL
    x = max(float((np.sqrt(A * r2 - det * t * t) - B * t) / A) for t in (lo, dy))
    grids = [(float(mx) + x - CELL * (2.0 + o), y - 2.0 * CELL) for o in np.linspace(-3e-5, 3e-5, 301)]
    return s, grids


def _edge_occ(r, s, grids, k):
    f = np.float32(2.0) ** k
    r.load_scene(Scene(s.means * f, s.scales * f, s.quats, s.opacity, s.sh, 0))
    g = 2.0 ** k
    h = np.zeros(1, np.float32)
    return torch.stack([r.slice_occupancy(x * g, y * g, CELL * g, 4, 4, h, rho_min=RHO)[0] for x, y in grids])


def test_ends_on_cell_edges():
    from paper_2603_15186_amd import hgs
    r = hgs.Renderer(0)
    differ = 0
    for seed in range(12):
        s, grids = _edge_grids(seed)
        rows, cells_ = _edge_occ(r, s, grids, 0), _edge_occ(r, s, grids, -70)
        assert 0 < int(cells_.sum()) < cells_.numel()
        d = int((rows != cells_).any(-1).any(-1).any(-1).sum())
        print(f"seed {seed}: {d} of {len(grids)} grids differ", flush=True)
        differ += d
    assert differ == 0
    r.close()
