"""The network's products at the edges of their tiles (needs an MI355X):
widths and batches of one, either side of 16, 32 and 64, odd strides, batches
whose split over wavefronts leaves some without work, and the size above
which a block's result is four times as large."""
import numpy as np
import pytest

import mlp_reference as mr
from gpu_helpers import log

pytestmark = pytest.mark.gpu


# FP32 operands: sums of up to 2100 terms and 2 L - 1 <= 7 products in a row
# at unit roundoff 6e-8 stay below 1e-4.  BF16 operands: two roundings of
# 2^-9 per product that average over the sums, 2e-2 over the chain.
@pytest.mark.parametrize("d_in,width,layers,batch,prec,tol", [
    (1, 1, 2, 1, 1, 1e-4), (3, 5, 3, 7, 1, 1e-4), (16, 16, 2, 32, 1, 1e-4),
    (17, 31, 4, 257, 1, 1e-4), (33, 65, 3, 63, 1, 1e-4),
    (16, 256, 4, 1024, 1, 1e-4), (16, 256, 4, 1024, 0, 2e-2),
    (41, 521, 3, 2100, 1, 1e-4), (41, 521, 3, 2100, 0, 2e-2)])
def test_gradients_at_tile_edges(d_in, width, layers, batch, prec, tol):
    import torch
    from paper_1403_5524_amd import native
    rng = np.random.default_rng(d_in + width + batch)
    X = rng.normal(size=(batch, d_in)).astype(np.float32)
    t = 3.0 + rng.normal(size=batch).astype(np.float32)
    mlp = native.Mlp(d_in, width, layers, prec, seed=7)
    Xt = torch.as_tensor(X, device="cuda:0")
    loss, g = mlp.grad(Xt, torch.as_tensor(t, device="cuda:0"), want_grad=True)
    p = mlp.get_params().cpu().numpy().astype(np.float64)
    ref_loss, ref_g = mr.loss_and_grad(p, X, t, d_in, width, layers)
    y = mlp.forward(Xt).cpu().numpy()
    ref_y, _ = mr.forward(p, X, d_in, width, layers)
    mlp.free()
    g = g.cpu().numpy().astype(np.float64)
    err_g = np.linalg.norm(g - ref_g) / np.linalg.norm(ref_g)
    err_y = np.linalg.norm(y - ref_y) / np.linalg.norm(ref_y)
    log("mlp %d-%d x%d batch %d prec %d: gradient %.2e output %.2e"
        % (d_in, width, layers, batch, prec, err_g, err_y))
    assert err_g < tol and err_y < tol
    assert abs(float(loss.item()) - ref_loss) < tol * max(1.0, ref_loss)
