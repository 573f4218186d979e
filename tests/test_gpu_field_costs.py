"""Distance fields on both sides of the cell count up to which the sweeps work
on whole-number costs (250,000), with paths of up to a hundred thousand moves:
pairs of moves bit for bit against the oracle."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _corridor(ny, nx, period, turns):
    """Walls every `period` rows, open at alternating ends; with `turns`, posts
    in the corridors that make their paths change rows by diagonal moves."""
    nav = np.ones((ny, nx), np.uint8)
    if turns:
        j, i = np.mgrid[:ny, :nx]
        post = ((i % 6 == 2) & (j % period < period - 2)) | ((i % 6 == 5) & (j % period > 0))
        nav[post & (i > 2) & (i < nx - 3)] = 0
    for k, j in enumerate(range(period - 1, ny - 1, period)):
        nav[j, :] = 0
        nav[j, :3] = k % 2
        nav[j, -3:] = 1 - k % 2
    return nav


@pytest.mark.parametrize("ny, nx, period, turns", [(500, 500, 2, False), (500, 500, 4, True), (500, 501, 4, True),
                                                   (400, 625, 5, True), (1, 300, 9, False), (33, 31, 4, True)])
def test_pairs_bit_exact(ny, nx, period, turns):
    from paper_2603_15186_amd import hgs
    nav = _corridor(ny, nx, period, turns)
    goals = [0, int(np.flatnonzero(nav)[-1])]
    r = hgs.Renderer(0)
    dist, rounds = r.distance_fields(torch.from_numpy(nav).cuda(), goals)
    got = dist.cpu().numpy().view(np.int32).reshape(len(goals), ny, nx, 2)
    want = np.asarray(O.distance_fields(nav, goals)).reshape(got.shape)
    np.testing.assert_array_equal(got, want)
    print(f"{ny}x{nx}: {rounds} rounds, up to {want.sum(axis=-1).max()} moves", flush=True)
    assert want.sum(axis=-1).max() > (ny * nx) // 8
    r.close()
