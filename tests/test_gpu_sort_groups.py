"""The radix sort at the sizes where its histogram groups change (1,024,
2,048, 4,096 and 8,192 elements), bit for bit against numpy's stable sort."""
import numpy as np
import pytest
import torch

from paper_2603_15186_amd import hgs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    r = hgs.Renderer(0)
    yield r
    r.set_option(hgs.HGS_OPT_SORT_DIGIT_BITS, 8)
    r.close()


EDGES = [1, 1023, 1025, 3 * 1024, 512 * 1024, 512 * 1024 + 1, 1024 * 1024, 1024 * 1024 + 1, 2048 * 1024,
         2048 * 1024 + 1, 4096 * 1024]


@pytest.mark.parametrize("n", EDGES)
def test_sort_at_group_edges(R, n):
    rng = np.random.default_rng(n)
    keys = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    keys[::3] &= 0xffff                      # many equal digits
    vals = np.arange(n, dtype=np.uint32)
    for digit, bits in ((6, 12), (8, 26), (11, 21)):
        R.set_option(hgs.HGS_OPT_SORT_DIGIT_BITS, digit)
        order = np.argsort(keys & np.uint32((1 << bits) - 1), kind="stable")
        for sort in (R.sort_pairs, R.sort_pairs_noalloc):
            k = torch.from_numpy(keys.view(np.int32).copy()).cuda()
            v = torch.from_numpy(vals.view(np.int32).copy()).cuda()
            sort(k, v, bits)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(v.cpu().numpy().view(np.uint32), vals[order])
            np.testing.assert_array_equal(k.cpu().numpy().view(np.uint32), keys[order])
