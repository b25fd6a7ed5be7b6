"""T from large K (needs an MI355X) where every energy takes the complex route:
fewer energies than the route has slots, and more, so that slots serve several
energies in turn."""
import numpy as np
import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu


# 1 - iK has condition number |K|: the error is at most a few n u |K|, and the
# energies among small K are those of the call without them, bit for bit.
@pytest.mark.parametrize("n,M,share", [
    (1, 1100, 1.0), (20, 1, 1.0), (20, 1100, 1.0), (20, 3000, 0.4), (33, 3, 1.0),
    (33, 1100, 0.5), (129, 300, 1.0)])
def test_large_k_over_the_slots(n, M, share):
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    s = wl.tiny(n=n, n_poles=64, M=6, seed=n).syms[0]
    h = native.load_symmetry(s)
    E = s.e_thr.max() + 1.0 + 1e-3 * np.arange(M)  # all channels open
    rng = np.random.default_rng(n)
    K = rng.standard_normal((M, n, n))
    K = K + K.transpose(0, 2, 1)
    big = rng.random(M) < share
    K[big] *= 1e6

    def omega(k):
        no = torch.full((k.size,), n, dtype=torch.int32, device="cuda:0")
        om = torch.zeros((k.size, n * (n + 1) // 2), dtype=torch.float64,
                         device="cuda:0")
        return native.rm_collision_strengths(
            h, torch.as_tensor(K[k], device="cuda:0"), no,
            torch.as_tensor(E[k], device="cuda:0"), n, om).cpu().numpy()
    om = omega(np.arange(M))
    for k in (np.flatnonzero(big)[-2:], np.flatnonzero(~big)[:5]):
        if k.size:
            assert np.array_equal(omega(k), om[k])
    h.free()
    tgt = np.arange(n) if s.target is None else np.asarray(s.target)
    G = np.zeros((n, n))
    G[np.arange(n), tgt] = 1.0
    worst = 0.0
    for e in np.flatnonzero(big):
        T = 2j * np.linalg.solve(np.eye(n) - 1j * K[e], K[e].astype(complex))
        O = (G.T @ (0.5 * s.g * np.abs(T) ** 2) @ G)[np.triu_indices(n)]
        worst = max(worst, np.abs(om[e] - O).max() / np.abs(O).max())
    bound = 8 * n * 2.0 ** -53 * np.linalg.norm(K[big], 2, axis=(1, 2)).max()
    log("large K n=%d, %d of %d energies: err %.2e bound %.2e"
        % (n, big.sum(), M, worst, bound))
    assert worst < bound
