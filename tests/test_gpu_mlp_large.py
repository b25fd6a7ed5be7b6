"""The network's products where a wavefront holds 64 x 64 of the result (needs an
MI355X): batches just past the size that chooses it, odd ones, up to 64 columns
(wavefronts above each other) and more."""
import numpy as np
import pytest

import mlp_reference as mr
from gpu_helpers import log

pytestmark = pytest.mark.gpu


# As at smaller batches: FP32 operands 1e-4, with sums over the batch of up to
# 131137 terms in eight parts, whose rounding errors of 6e-8 add up at random to
# below 1e-5; BF16 operands 2e-2.
@pytest.mark.parametrize("d_in,width,layers,batch,prec,tol", [
    (17, 64, 3, 131137, 1, 1e-4), (17, 64, 3, 131137, 0, 2e-2),
    (5, 33, 3, 131073, 1, 1e-4), (33, 65, 3, 65601, 1, 1e-4),
    (9, 130, 3, 43700, 1, 1e-4), (9, 130, 3, 43700, 0, 2e-2)])
def test_products_of_large_batches(d_in, width, layers, batch, prec, tol):
    import torch
    from paper_1403_5524_amd import native
    rng = np.random.default_rng(width + batch)
    X = rng.normal(size=(batch, d_in)).astype(np.float32)
    t = 3.0 + rng.normal(size=batch).astype(np.float32)
    mlp = native.Mlp(d_in, width, layers, prec, seed=7)
    Xt = torch.as_tensor(X, device="cuda:0")
    _, g = mlp.grad(Xt, torch.as_tensor(t, device="cuda:0"), want_grad=True)
    p = mlp.get_params().cpu().numpy().astype(np.float64)
    _, ref_g = mr.loss_and_grad(p, X, t, d_in, width, layers)
    y = mlp.forward(Xt).cpu().numpy()
    # the same samples in a batch that takes the smaller tiles: the same bits
    few = mlp.forward(Xt[-500:].contiguous()).cpu().numpy()
    mlp.free()
    ref_y, _ = mr.forward(p, X, d_in, width, layers)
    g = g.cpu().numpy().astype(np.float64)
    err_g = np.linalg.norm(g - ref_g) / np.linalg.norm(ref_g)
    err_y = np.abs(y - ref_y).max() / np.abs(ref_y).max()
    log("mlp %d-%d x%d batch %d prec %d: gradient %.2e output %.2e"
        % (d_in, width, layers, batch, prec, err_g, err_y))
    assert err_g < tol and err_y < tol
    assert np.array_equal(few, y[-500:])
