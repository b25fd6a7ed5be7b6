"""Photoionization with the matching solved by FP32 factors refined in FP64
(solve_fp32 = 1; needs an MI355X) against the oracle, where every channel is
open and where some are closed, at one channel, a few, and one past a team's
rows."""
import numpy as np
import pytest

import oracle
from gpu_helpers import log
from paper_1403_5524_amd import workloads as wl

pytestmark = pytest.mark.gpu


# relative to the largest cross section, to the 1e-6 of the FP64 solve's oracle
# tests: refined solutions meet the FP64 tolerance, the others are solved in FP64
@pytest.mark.parametrize("lo,hi", [(2.05, 8.0), (0.3, 2.2)])
@pytest.mark.parametrize("n", [1, 2, 5, 8, 33, 64, 65])
def test_photoionization_with_fp32_solve(n, lo, hi):
    import torch
    from paper_1403_5524_amd import native
    M = 48 if n < 64 else 12
    w = wl.tiny(n=n, n_poles=12 * n + 40, M=M, seed=7 * n, mesh_lo=lo, mesh_hi=hi)
    s = w.syms[0]
    d = np.random.default_rng(n).normal(size=s.n_poles)
    n_open = (w.mesh[:, None] > s.e_thr[None]).sum(1)
    assert (n_open == n).all() if lo > 2.0 else n < 3 or (n_open < n).any()
    h = native.load_symmetry(s)
    native.rm_load_dipoles(h, d)
    sig, st = native.rm_photoionization(
        [h], torch.as_tensor(w.mesh, device="cuda:0"), -0.8,
        native.make_opts(solve_fp32=1))
    sig, st = sig.cpu().numpy(), st.cpu().numpy()
    h.free()
    ref = oracle.photoionization([s.as_dict()], [d], w.mesh, -0.8)
    err = np.abs(sig - ref).max() / np.abs(ref).max()
    log("photo fp32 solve n=%d mesh [%g, %g]: %.2e" % (n, lo, hi, err))
    assert err < 1e-6
    assert not (st[n_open > 0] & ~native.RM_E_REFINE_NOCONV).any()
