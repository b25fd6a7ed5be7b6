"""Dipole pole sums (needs an MI355X) where channels and energies end inside a
tile of 32 x 16, poles inside a turn of the eight wavefronts, and at one
channel and one energy: cross sections against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_helpers import log
from paper_1403_5524_amd import workloads as wl

pytestmark = pytest.mark.gpu


# relative to the largest cross section, to the 1e-6 of the other oracle tests
@pytest.mark.parametrize("n,nh,M", [(1, 1, 1), (2, 33, 15), (31, 64, 16),
                                    (32, 65, 17), (33, 200, 33), (64, 129, 5),
                                    (65, 511, 70)])
def test_photoionization_at_tile_edges(n, nh, M):
    import torch
    from paper_1403_5524_amd import native
    w = wl.tiny(n=n, n_poles=nh, M=M, seed=n + nh, mesh_lo=2.05)
    d = np.random.default_rng(nh).normal(size=nh)
    h = native.load_symmetry(w.syms[0])
    native.rm_load_dipoles(h, d)
    sig, _ = native.rm_photoionization(
        [h], torch.as_tensor(w.mesh, device="cuda:0"), -0.8)
    h.free()
    ref = oracle.photoionization([w.syms[0].as_dict()], [d], w.mesh, -0.8)
    err = np.abs(sig.cpu().numpy() - ref).max() / np.abs(ref).max()
    log("photo edges n=%d nh=%d M=%d: %.2e" % (n, nh, M, err))
    assert err < 1e-6
