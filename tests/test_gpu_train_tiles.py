"""The training step at batch sizes around its tiles (16 samples per wave, 64
per workgroup, several tiles per wave beyond 16,384 samples), against the
float64 network."""
import numpy as np
import pytest
import torch

from oracle import mlp as M
from paper_2603_15186_amd import hgs
from paper_2603_15186_amd.synth import mlp_init

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    r = hgs.Renderer(0)
    yield r
    r.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, 1000, 16384, 16385, 40001])
def test_gradient_at_tile_edges(R, n):
    rng = np.random.default_rng(n)
    F = rng.normal(1.0, 2.0, size=(n, 8)).astype(np.float32)
    y = (rng.uniform(size=n) < 0.4).astype(np.float32)
    mean, std = rng.normal(1.0, 0.2, 8).astype(np.float32), rng.uniform(1.0, 3.0, 8).astype(np.float32)
    bits = M.bf16_bits(mlp_init(n))
    w = torch.from_numpy(bits.view(np.int16).copy()).cuda()
    g = torch.full((hgs.N_MLP_PARAMS,), 7.0, device="cuda")
    loss = torch.zeros(1, device="cuda")
    Fd, yd = torch.from_numpy(F).cuda(), torch.from_numpy(y).cuda()
    R.mlp_backward(Fd, yd, mean, std, w, g, loss_out=loss)
    wv, X = M.bf16_value(bits), M.standardise(F, mean, std)
    want = M.grad(wv, X, y)
    # products of three float32 factors summed over n samples: far below 1e-5
    # of the largest gradient (n 2^-24 only if every rounding agreed)
    assert np.abs(g.cpu().numpy() - want).max() <= 1e-5 * np.abs(want).max() + 1e-7
    assert loss.item() == pytest.approx(M.loss(wv, X, y), rel=1e-5)
    g2 = torch.empty_like(g)
    R.mlp_backward(Fd, yd, mean, std, w, g2)
    assert torch.equal(g, g2)
