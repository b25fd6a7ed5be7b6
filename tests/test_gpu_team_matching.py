"""Matching, K, T and Omega by teams of wavefronts (needs an MI355X) at the
edges of their tiles, register panels and team sizes: 16- and 32-row blocks,
64 rows (one wavefront), 256 rows (four) and above (eight)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import log, omega_normwise_err

pytestmark = pytest.mark.gpu


# Omega against the oracle, normwise per energy, to the 1e-6 that the sweeps'
# other oracle tests use.
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96,
                               97, 128, 129, 256, 257])
@pytest.mark.parametrize("fp32", [0, 1])
def test_sweep_at_block_edges(n, fp32):
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    M = 24 if n < 100 else 4
    w = wl.tiny(n=n, n_poles=8 * n + 40, M=M, seed=100 + n)
    h = native.load_symmetry(w.syms[0])
    om, st = native.rm_sweep_energies(
        [h], n, torch.as_tensor(w.mesh, device="cuda:0"),
        native.make_opts(solve_fp32=fp32))
    om, st = om.cpu().numpy(), st.cpu().numpy()
    h.free()
    ref = oracle.sweep(w.syms[0].as_dict(), w.mesh)
    err, _, _ = omega_normwise_err(om, ref["omega"])
    log("team sweep n=%d fp32=%d: omega err %.2e" % (n, fp32, err))
    assert err < 1e-6
    keep = ~native.RM_E_REFINE_NOCONV if fp32 else -1
    assert np.array_equal(st & keep, ref["status"])


# T from K with |K| near 1e6 goes through the complex system (2 n rows, so 8,
# 32 and 128 channels end a block, a panel or a team size).  1 - iK has
# condition number |K|: the error is at most a few n u |K|.
@pytest.mark.parametrize("n", [1, 8, 9, 16, 17, 20, 32, 33, 64, 65, 128, 129])
def test_large_k_at_block_edges(n):
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    w = wl.tiny(n=n, n_poles=64, M=6, seed=n)
    s = w.syms[0]
    h = native.load_symmetry(s)
    E = np.full(70, s.e_thr.max() + 1.0) + 0.01 * np.arange(70)  # all open
    rng = np.random.default_rng(n)
    K = rng.standard_normal((70, n, n)) * 1e6
    K = K + K.transpose(0, 2, 1)
    no = torch.full((70,), n, dtype=torch.int32, device="cuda:0")
    om = torch.zeros((70, n * (n + 1) // 2), dtype=torch.float64, device="cuda:0")
    native.rm_collision_strengths(h, torch.as_tensor(K, device="cuda:0"), no,
                                  torch.as_tensor(E, device="cuda:0"), n, om)
    om = om.cpu().numpy()
    h.free()
    tgt = np.arange(n) if s.target is None else np.asarray(s.target)
    worst = 0.0
    for e in range(70):
        T = 2j * np.linalg.solve(np.eye(n) - 1j * K[e], K[e].astype(complex))
        V = 0.5 * s.g * np.abs(T) ** 2
        G = np.zeros((n, n))
        G[np.arange(n), tgt] = 1.0
        O = (G.T @ V @ G)[np.triu_indices(n)]
        worst = max(worst, np.abs(om[e] - O).max() / np.abs(O).max())
    bound = 8 * n * 2.0 ** -53 * np.linalg.norm(K, 2, axis=(1, 2)).max()
    log("team large K n=%d: err %.2e bound %.2e" % (n, worst, bound))
    assert worst < bound
