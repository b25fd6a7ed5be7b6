"""Grouped FP64 pole sum (needs an MI355X) with enough poles that groups are
formed: at the edges of tiles and groups, on meshes that the grouping must leave
to the direct sum, and with poles on the edge of a group's near window."""
import numpy as np
import pytest

import oracle
from gpu_helpers import log
from test_gpu_polesum_group import _mesh

pytestmark = pytest.mark.gpu


def _check(s, E, chunk=0):
    """R(E) of the mapping s against the plain sum: every element a sum of nh
    products in FP64, so its error is at most (nh + 64) u sum |terms|, as in the
    tests of other grouped meshes; returns the largest error over the bound."""
    import torch
    from paper_1403_5524_amd import native
    h = native.load_symmetry(s)
    R = native.rm_rmatrix(h, torch.as_tensor(E, device="cuda:0"),
                          native.make_opts(chunk=chunk)).cpu().numpy()
    h.free()
    w, p = np.asarray(s["w"]), np.asarray(s["E_pole"])
    bound = 2 * (p.size + 64) * 2.0 ** -53
    worst = 0.0
    for e in range(E.size):
        d = 1.0 / (p - E[e])
        ref = (w * d) @ w.T / (2 * s["a"])
        mag = (np.abs(w) * np.abs(d)) @ np.abs(w).T / (2 * s["a"])
        worst = max(worst, (np.abs(R[e] - ref) / mag).max())
    assert np.array_equal(R, R.transpose(0, 2, 1))
    assert worst < bound
    return worst / bound


@pytest.mark.parametrize("n,nh,M,kind,chunk", [
    (1, 512, 64, "fine", 0), (16, 520, 127, "fine", 0), (17, 512, 128, "fine", 0),
    (20, 600, 200, "coarse", 0), (20, 600, 200, "shuffled", 0),
    (20, 600, 130, "same", 0), (20, 600, 300, "same", 90),
    (5, 512, 256, "outside", 0), (33, 575, 257, "coarse", 50)])
def test_rmatrix_of_groups_and_of_refused_meshes(n, nh, M, kind, chunk):
    from paper_1403_5524_amd import workloads as wl
    s = wl.tiny(n=n, n_poles=nh, M=8, seed=n + nh).syms[0]
    E = _mesh(kind, M, s, np.random.default_rng(M))
    E = E + 1e-9 * (np.abs(E[:, None] - s.E_pole[None]).min(1) == 0)
    log("%s n=%d M=%d: %.2f of the bound" % (kind, n, M, _check(s.as_dict(), E, chunk)))


# Poles at the ends of the near window, cen +- 6 h, and one rounding to either
# side, as the last and the first pole of a chunk of 32: which chunks are near
# turns on the last bit.
@pytest.mark.parametrize("ulps", [-2, -1, 0, 1, 2])
def test_poles_on_the_edge_of_the_near_window(ulps):
    rng = np.random.default_rng(3)
    E = 2.0 + 1e-3 * (np.arange(128) + rng.uniform(0, 0.5, 128))
    cen = 0.5 * (E.min() + E.max())
    half = max(E.max() - cen, cen - E.min())
    lo, hi = cen - 6.0 * half, cen + 6.0 * half
    for _ in range(abs(ulps)):
        lo, hi = (np.nextafter(x, np.sign(ulps) * np.inf) for x in (lo, hi))
    p = np.concatenate([np.sort(rng.uniform(-20, lo - 0.1, 32 * 9 - 1)), [lo],
                        np.sort(rng.uniform(lo + 0.01, hi - 0.01, 32)), [hi],
                        np.sort(rng.uniform(hi + 0.1, 40, 300))])
    assert (np.diff(p) > 0).all()
    n = 18
    s = dict(E_pole=p, w=rng.standard_normal((n, p.size)), a=10.0,
             e_thr=np.zeros(n), l=np.zeros(n, dtype=np.int32), z=1.0, g=1.0)
    log("window edge %+d ulps: %.2f of the bound" % (ulps, _check(s, E)))


# sigma relative to its largest value, to the 1e-6 of the other oracle tests
@pytest.mark.parametrize("n,nh,M,kind", [
    (5, 600, 130, "coarse"), (17, 512, 140, "shuffled"), (5, 512, 128, "same"),
    (17, 600, 129, "step"), (33, 520, 200, "fine")])
def test_damped_photoionization_of_refused_meshes(n, nh, M, kind):
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    s = wl.tiny(n=n, n_poles=nh, M=8, seed=n + nh).syms[0]
    rng = np.random.default_rng(nh)
    E = _mesh(kind, M, s, rng)
    E = E + 1e-9 * (np.abs(E[:, None] - s.e_thr[None]).min(1) == 0)
    d, g = rng.normal(size=nh), 10.0 ** rng.uniform(-4, -1, nh)
    h = native.load_symmetry(s)
    native.rm_load_dipoles(h, d)
    native.rm_load_widths(h, g)
    sig, _ = native.rm_photoionization(
        [h], torch.as_tensor(E, device="cuda:0"), -0.8,
        native.make_opts(flags=native.RM_FLAG_RADIATION_DAMPING))
    h.free()
    ref = oracle.photoionization_damped([s.as_dict()], [d], [g], E, -0.8)
    err = np.abs(sig.cpu().numpy() - ref).max() / np.abs(ref).max()
    log("damped %s n=%d M=%d: %.2e" % (kind, n, M, err))
    assert err < 1e-6


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_energies_that_are_not_finite(bad):
    """They spoil no other energy of their group, and have no open channel or
    no finite result."""
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    n, M = 17, 200
    s = wl.tiny(n=n, n_poles=600, M=8, seed=3).syms[0]
    E = 2.5 + 1e-4 * (np.arange(M) + 0.5)
    ref = E.copy()
    at = [0, 63, 130]
    E[at] = bad
    keep = np.setdiff1d(np.arange(M), at)
    h = native.load_symmetry(s)
    R = native.rm_rmatrix(h, torch.as_tensor(E, device="cuda:0")).cpu().numpy()
    om, st = native.rm_sweep_energies([h], n, torch.as_tensor(E, device="cuda:0"))
    good, gst = native.rm_sweep_energies([h], n, torch.as_tensor(ref, device="cuda:0"))
    h.free()
    p, w = s.E_pole, np.asarray(s.w)
    for e in keep:
        d = 1.0 / (p - E[e])
        exact = (w * d) @ w.T / (2 * s.a)
        mag = (np.abs(w) * np.abs(d)) @ np.abs(w).T / (2 * s.a)
        assert (np.abs(R[e] - exact) / mag).max() < 2 * (p.size + 64) * 2.0 ** -53
    om, good = om.cpu().numpy(), good.cpu().numpy()
    err = np.abs(om - good)[keep].max() / np.abs(good).max()
    log("%s: others off by %.1e, status there %s" % (bad, err, st.cpu().numpy()[at]))
    assert err < 1e-6
    assert np.array_equal(st.cpu().numpy()[keep], gst.cpu().numpy()[keep])
    assert (st.cpu().numpy()[at] != 0).all()
