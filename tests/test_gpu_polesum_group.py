"""FP64 pole sum in groups of 128 energies (needs an MI355X): R(E) of meshes
whose far poles are interpolated and of meshes that must be summed directly,
at the edges of tiles, groups and chunks, against the plain sum."""
import numpy as np
import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu


def _mesh(kind, M, s, rng):
    lo, hi = s.E_pole[0], s.E_pole[-1]
    mid = lo + 0.37 * (hi - lo)
    if kind == "fine":        # far poles interpolated
        return mid + 1e-5 * np.arange(M)
    if kind == "step":        # one group astride a gap of half the range
        E = mid + 1e-5 * np.arange(M)
        E[M // 2:] += 0.3 * (hi - lo)
        return E
    if kind == "coarse":      # every pole near
        return np.linspace(lo - 0.5, hi + 0.5, M)
    if kind == "shuffled":
        return rng.permutation(np.linspace(lo, hi, M))
    if kind == "same":        # a group without extent
        return np.full(M, mid)
    if kind == "descending":
        return mid - 1e-4 * np.arange(M)
    if kind == "outside":     # no pole near, on either side
        return hi + 3.0 + 1e-3 * np.arange(M)
    raise ValueError(kind)


# Each element is a sum of nh products in FP64: its error is at most
# (nh + 64) u sum |terms| (64 for the 16-point interpolation, whose weights'
# magnitudes sum to less than 3, and for the scaling).
@pytest.mark.parametrize("n,nh,M,kind,chunk", [
    (1, 70, 64, "fine", 0), (16, 500, 127, "fine", 0),
    (17, 500, 128, "fine", 0), (33, 900, 129, "fine", 0),
    (33, 900, 300, "fine", 37), (48, 900, 300, "step", 0),
    (20, 300, 200, "coarse", 0), (20, 300, 200, "shuffled", 0),
    (20, 300, 130, "same", 0), (31, 2000, 257, "descending", 100),
    (5, 64, 256, "outside", 0), (64, 1500, 1000, "fine", 0)])
def test_rmatrix_of_grouped_energies(n, nh, M, kind, chunk):
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    s = wl.tiny(n=n, n_poles=nh, M=8, seed=n + nh).syms[0]
    E = _mesh(kind, M, s, np.random.default_rng(M))
    E = E + 1e-9 * (np.abs(E[:, None] - s.E_pole[None]).min(1) == 0)
    h = native.load_symmetry(s)
    R = native.rm_rmatrix(h, torch.as_tensor(E, device="cuda:0"),
                          native.make_opts(chunk=chunk)).cpu().numpy()
    h.free()
    w = np.asarray(s.w, dtype=np.float64)
    d = 1.0 / (s.E_pole[None] - E[:, None])
    worst = 0.0
    for e in range(M):
        ref = (w * d[e]) @ w.T / (2 * s.a)
        mag = (np.abs(w) * np.abs(d[e])) @ np.abs(w).T / (2 * s.a)
        worst = max(worst, (np.abs(R[e] - ref) / mag).max())
    log("grouped pole sum n=%d nh=%d M=%d %s: error over sum of magnitudes %.1e"
        % (n, nh, M, kind, worst))
    assert worst < 2 * (nh + 64) * 2.0 ** -53
    assert np.array_equal(R, R.transpose(0, 2, 1))
