"""Workloads whose speed is tracked, each through the public entry points.

Every kind below is one thing a program built on this library does with it:

* ``sweep``     collision strengths of one symmetry on a mesh
                (rm_sweep_energies), in FP64 or with the split-BF16 pole sum;
* ``kmatrix``   K- and R-matrices of one symmetry (rm_kmatrix);
* ``plan``      several symmetries that share target levels, captured once
                and replayed (rm_plan_create / rm_plan_execute);
* ``photo``     photoionization cross sections, undamped or damped
                (rm_photoionization);
* ``outer``     a sweep with the R-matrix propagated to A, matched there to
                Coulomb functions or to the asymptotic expansion;
* ``inner``     the inner-region eigen-solve that supplies the poles
                (rm_inner_region, host arrays in and out);
* ``post``      smoothing, effective collision strengths and level groups of
                an Omega table;
* ``train``     one training step of the learned mesh's network.

Poles are uniform in [-5, 200] Ry, amplitudes N(0, 0.1^2), thresholds in
[0, 2] Ry and l in 0..5, as in paper_1403_5524_amd/workloads.py; a is 20 and
z is 1.  A mesh is M points from ``lo`` on, ``step`` Ry apart (or clustered
around some points, as an adaptive mesh is), stepped over the 0.02 Ry below
each threshold, where a run that is not after the Rydberg series of that
level has no points.
"""
import math

import numpy as np
import torch

from paper_1403_5524_amd import native

A_BOUND, Z_RES, GAP = 20.0, 1.0, 0.02
SIGMA = 4.0 * math.pi ** 2 * 7.2973525693e-3 * 28.00285205 / 3.0
N_GROUPS, N_TEMPS = 20, 8


def listed():
    return [
        # the smallest call: the 8-channel system on a few energies, where
        # launches and host work are all there is
        dict(name="sweep_smallest", kind="sweep", n=8, nh=200, levels=0, M=64,
             lo=0.3, step=0.15, mesh="uniform", prec="fp64"),
        # the headline system on a stretch of its 1e5-point mesh
        dict(name="sweep_200", kind="sweep", n=200, nh=8000, levels=20, M=4096,
             lo=1.2, step=2e-4, mesh="uniform", prec="fp64"),
        # the same with the mixed-precision pole sum
        dict(name="sweep_200_bf16x3", kind="sweep", n=200, nh=8000, levels=20,
             M=4096, lo=1.2, step=2e-4, mesh="uniform", prec="bf16x3"),
        # K- and R-matrices of a ragged system on a coarse survey mesh
        dict(name="kmatrix_ragged", kind="kmatrix", n=117, nh=4001, levels=20,
             M=1001, lo=0.05, step=0.015, mesh="uniform", prec="fp64"),
        # several symmetries of very different size, replayed from a plan
        dict(name="plan_batched", kind="plan", n_sym=8, n_lo=20, n_hi=400,
             levels=20, M=1500, lo=3.0, step=3e-4, mesh="clustered"),
        # photoionization, the B II shape (400 channels, 62 poles a channel),
        # above the first thresholds, where its resonances are
        dict(name="photo_400", kind="photo", n=400, nh=24800, M=256, lo=0.06,
             step=5e-5, mesh="uniform", damped=False),
        # the same physics with radiation damping on a smaller target
        dict(name="photo_damped_200", kind="photo", n=200, nh=12400, M=512,
             lo=1.1, step=2e-4, mesh="uniform", damped=True),
        # many channels and few energies, the Ca II ratio of poles
        dict(name="photo_wide", kind="photo", n=1000, nh=12700, M=64, lo=0.06,
             step=1e-3, mesh="uniform", damped=False),
        # outer region: 20 sectors beyond a, then Coulomb matching
        dict(name="outer_200", kind="outer", n=200, nh=8000, levels=10, M=256,
             lo=5.1, step=2e-3, mesh="uniform", A=40.0, n_sec=20, terms=0),
        # all poles and amplitudes of an 8-channel model, D = 1024
        dict(name="inner_1024", kind="inner", n=8, n_basis=128),
        # what follows a sweep: 100 levels on an 8192-point mesh
        dict(name="post_100", kind="post", n_target=100, M=8192, step=2e-4,
             fwhm=7.35e-3),
        # a training step at the learned mesh's own size
        dict(name="train_1024", kind="train", d_in=16, width=256, n_layers=4,
             batch=1024),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["sweep", "sweep", "sweep", "kmatrix", "plan", "photo",
                       "photo", "outer", "inner", "post", "train"])
    mesh = rng.choice(["uniform", "uniform", "clustered"])
    lo, step = rng.uniform(0.05, 12.0), _log(rng, 5e-5, 5e-3)
    if kind in ("sweep", "kmatrix"):
        n = int(_log(rng, 3, 400))
        M = int(min(_log(rng, 32, 6000), 4096 * min(1.0, (200 / n) ** 3)))
        c = dict(kind=kind, n=n, nh=int(n * rng.uniform(25, 62)) + 1,
                 levels=0 if n < 60 else rng.randint(10, 20), M=max(M, 16),
                 lo=lo, step=step, mesh=mesh, prec="fp64")
        if c["levels"] == 0:  # one level a channel: a stretch of the mesh
            c["step"] = min(c["step"], 4.0 / c["M"])
        if kind == "sweep" and rng.random() < 0.3:
            c["prec"] = "bf16x3"
        return c
    if kind == "plan":
        return dict(kind=kind, n_sym=rng.randint(2, 8), n_lo=rng.randint(5, 25),
                    n_hi=rng.randint(60, 400), levels=rng.randint(5, 20),
                    M=int(_log(rng, 64, 1500)), lo=lo, step=step, mesh=mesh)
    if kind == "photo":
        damped = rng.random() < 0.4
        n = int(_log(rng, 20, 200 if damped else 700))
        M = int(_log(rng, 32, 512 if damped else 256) * min(1.0, (300 / n) ** 2))
        lo = lo if damped else rng.uniform(0.03, 0.1)
        return dict(kind=kind, n=n, nh=int(n * rng.uniform(13, 62)) + 1,
                    M=max(M, 16), lo=lo, step=min(step, 4.0 / max(M, 16)),
                    mesh=mesh, damped=damped)
    if kind == "outer":
        A = rng.uniform(25.0, 60.0)
        return dict(kind=kind, n=int(_log(rng, 10, 200)), nh=rng.randint(2000, 8000),
                    levels=rng.randint(4, 10), M=int(_log(rng, 16, 256)),
                    lo=lo, step=step, mesh=mesh, A=A,
                    n_sec=max(1, min(20, int((A - 20.0) / 2))),
                    terms=rng.choice([0, 0, 30]))
    if kind == "inner":
        return dict(kind=kind, n=rng.randint(3, 9), n_basis=rng.randint(24, 140))
    if kind == "post":
        return dict(kind=kind, n_target=rng.randint(5, 100),
                    M=int(_log(rng, 500, 8192)), step=_log(rng, 2e-4, 5e-3),
                    fwhm=_log(rng, 2e-3, 2e-2))
    return dict(kind=kind, d_in=rng.randint(8, 32), width=rng.choice([128, 256]),
                n_layers=rng.randint(3, 5), batch=rng.randint(200, 2048))


# --------------------------------------------------------------- inputs

def _mesh(case, rng):
    M, lo, step = case["M"], case["lo"], case["step"]
    if case["mesh"] == "uniform":
        return lo + step * (np.arange(M) + 0.5)
    # clustered: half the points uniform, half around narrow structures
    k = M // 2
    span = step * M
    at = rng.uniform(lo, lo + span, size=max(1, M // 64))
    x = at[rng.integers(0, at.size, size=k)] + 0.3 * step * rng.standard_cauchy(k)
    x = np.clip(x, lo, lo + span)
    return np.sort(np.concatenate([x, rng.uniform(lo, lo + span, size=M - k)]))


def _off_thresholds(E, thr):
    """Steps E over the GAP below every threshold; ascending."""
    E = E.copy()
    for _ in range(1000):
        d = thr[None, :] - E[:, None]
        bad = ((d > -1e-6) & (d < GAP)).any(axis=1)
        if not bad.any():
            break
        E[bad] += GAP
    return np.sort(E)


def _system(n, nh, rng, E, levels=None, target=None):
    """Host arrays of one symmetry; thresholds off the mesh."""
    poles = np.sort(rng.uniform(-5.0, 200.0, size=nh))
    w = 0.1 * rng.standard_normal((n, nh))
    if levels is None:
        thr = rng.uniform(0.0, 2.0, size=n)
        thr[0] = 0.0  # the ground level
        for _ in range(1000):
            k = np.searchsorted(E, thr - GAP)
            near = E[np.minimum(k, E.size - 1)]
            bad = (k < E.size) & (near <= thr + 1e-6)
            if not bad.any():
                break
            thr[bad] = rng.uniform(0.0, 2.0, size=int(bad.sum()))
        # a window that covers [0, 2]: every level at the bottom is open
        thr[bad] = -0.05 * rng.random(int(bad.sum()))
    else:
        thr = levels[target]
    l = rng.integers(0, 6, size=n).astype(np.int32)
    return dict(E_pole=poles, w=w, a=A_BOUND, e_thr=thr, l=l, z=Z_RES, g=1.0,
                target=None if target is None else target.astype(np.int32))


def _inputs(case, seed):
    """Everything host-side: mesh, systems and what goes with them."""
    rng = np.random.default_rng([seed, 77])
    kind = case["kind"]
    if kind in ("sweep", "kmatrix", "outer"):
        E = _mesh(case, rng)
        nl = case["levels"]
        if nl:
            levels = np.sort(rng.uniform(0.0, 2.0, size=nl))
            levels -= levels[0]
            if kind == "outer":
                levels = 0.5 * np.arange(nl)
            E = _off_thresholds(E, levels)
            tgt = rng.integers(0, nl, size=case["n"])
            sym = _system(case["n"], case["nh"], rng, E, levels, tgt)
        else:
            sym = _system(case["n"], case["nh"], rng, E)
        out = dict(E=E, syms=[sym], n_target=nl or case["n"])
        if kind == "outer":
            beta = [s * rng.standard_normal((case["n"],) * 2) for s in (1.0, 4.0)]
            out["beta"] = np.stack([0.5 * (b + b.T) for b in beta])
        return out
    if kind == "plan":
        levels = np.sort(rng.uniform(0.0, 2.0, size=case["levels"]))
        levels -= levels[0]
        E = _off_thresholds(_mesh(case, rng), levels)
        syms = []
        for s in range(case["n_sym"]):
            f = s / max(1, case["n_sym"] - 1)
            n = int(round(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** f))
            tgt = rng.integers(0, case["levels"], size=n)
            syms.append(_system(n, 30 * n, rng, E, levels, tgt))
            syms[-1]["g"] = float(1 + s % 10)
        return dict(E=E, syms=syms, n_target=case["levels"])
    if kind == "photo":
        E = _mesh(case, rng)
        sym = _system(case["n"], case["nh"], rng, E)
        return dict(E=E, syms=[sym], dip=rng.standard_normal(case["nh"]),
                    widths=10.0 ** rng.uniform(-6, -3, size=case["nh"]), e0=-0.8)
    if kind == "inner":
        n = case["n"]
        e = np.sort(rng.uniform(0.0, 2.0, n))
        e[0] = 0.0
        off = rng.uniform(0.1, 1.0, (n, n))
        depth = 0.5 * (off + off.T)
        depth[np.arange(n), np.arange(n)] = rng.uniform(1.0, 4.0, n)
        rg = rng.uniform(1.5, 4.0, (n, n))
        return dict(model=dict(e_thr=e, l=rng.integers(0, 4, n), z=Z_RES,
                               a=A_BOUND, depth=depth, range=0.5 * (rg + rg.T)))
    if kind == "post":
        nt = case["n_target"]
        lev = np.sort(rng.uniform(0.0, 2.0, size=nt))
        lev[0] = 0.0
        return dict(E=0.01 + case["step"] * (np.arange(case["M"]) + 0.5), lev=lev,
                    group=rng.integers(0, min(N_GROUPS, nt), size=nt).astype(np.int32),
                    kT=np.geomspace(0.01, 2.0, N_TEMPS))
    return {}


def _omega_table(case, inp, seed):
    """Omega [M, P] of resonances on a smooth background (device)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    nt, M = case["n_target"], case["M"]
    P = nt * (nt + 1) // 2
    E = torch.as_tensor(inp["E"], device="cuda")
    o = torch.rand((1, P), generator=g, device="cuda", dtype=torch.float64)
    o = o / (1.0 + 0.3 * E[:, None])
    o += 0.2 * torch.rand((M, P), generator=g, device="cuda", dtype=torch.float64)
    return E, o.contiguous()


def _net(case, seed):
    """Layer sizes, flat parameters, batch and target of the network."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    d, W, nl = case["d_in"], case["width"], case["n_layers"]
    sizes = [(d if i == 0 else W, 1 if i == nl - 1 else W) for i in range(nl)]
    parts = []
    for fi, fo in sizes:
        b = math.sqrt(6.0 / fi)
        parts.append((torch.rand(fo * fi, generator=g, device="cuda") * 2 - 1) * b)
        parts.append(0.1 * torch.randn(fo, generator=g, device="cuda"))
    X = torch.randn((case["batch"], d), generator=g, device="cuda")
    t = torch.randn(case["batch"], generator=g, device="cuda")
    return sizes, torch.cat(parts), X, t


def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind)
    if kind == "train":
        sizes, p, X, t = _net(case, seed)
        s["mlp"] = native.Mlp(case["d_in"], case["width"], case["n_layers"], 0, 1)
        s["mlp"].set_params(p)
        return dict(s, X=X, t=t)
    inp = _inputs(case, seed)
    if kind == "inner":
        return dict(s, model=inp["model"], n_basis=case["n_basis"])
    if kind == "post":
        E, om = _omega_table(case, inp, seed)
        return dict(s, E=E, omega=om, nt=case["n_target"], lev=inp["lev"],
                    group=inp["group"], kT=inp["kT"], fwhm=case["fwhm"])
    s["E"] = torch.as_tensor(inp["E"], device="cuda")
    s["syms"] = [native.load_symmetry(d) for d in inp["syms"]]
    s["nt"] = inp.get("n_target")
    prec = {"fp64": native.RM_PREC_FP64, "bf16x3": native.RM_PREC_BF16X3}
    s["opts"] = native.make_opts(prec=prec[case.get("prec", "fp64")])
    if kind == "photo":
        native.rm_load_dipoles(s["syms"][0], inp["dip"])
        s["e0"] = inp["e0"]
        if case["damped"]:
            native.rm_load_widths(s["syms"][0], inp["widths"])
            s["opts"] = native.make_opts(flags=native.RM_FLAG_RADIATION_DAMPING)
    if kind == "outer":
        native.rm_set_propagation(s["syms"][0], case["A"], case["n_sec"], inp["beta"])
        if case["terms"]:
            native.rm_set_gailitis(s["syms"][0], case["terms"])
    if kind == "plan":
        s["plan"] = native.Plan(s["syms"], s["nt"], s["E"], s["opts"])
    return s


def run(s):
    kind = s["kind"]
    if kind in ("sweep", "outer"):
        return native.rm_sweep_energies(s["syms"], s["nt"], s["E"], s["opts"])
    if kind == "kmatrix":
        return native.rm_kmatrix(s["syms"][0], s["E"], s["opts"], want_R=True)
    if kind == "plan":
        return s["plan"].execute()
    if kind == "photo":
        return native.rm_photoionization(s["syms"], s["E"], s["e0"], s["opts"])
    if kind == "inner":
        E, w, _, _ = native.rm_inner_region(s["model"], s["n_basis"])
        return E, w
    if kind == "post":
        sm = native.rm_convolve_gaussian(s["E"], s["omega"], s["fwhm"])
        ups = native.rm_effective_collision_strengths(
            s["E"], s["omega"], s["lev"], s["nt"], s["kT"])
        grp = native.rm_group_collision_strengths(
            s["omega"], s["nt"], s["group"], min(N_GROUPS, s["nt"]))
        return sm, ups, grp
    loss, grad = s["mlp"].grad(s["X"], s["t"], want_grad=True)
    s["mlp"].adam_step(lr=1e-3)
    return loss, grad


def _dense_flops(n, photo=False):
    """LU with n right-hand sides, then the T step (or its photo part)."""
    return (2.0 / 3 + 2.0) * n ** 3 + (1.5 if photo else 3.0) * n ** 3


def work(case):
    kind = case["kind"]
    if kind in ("sweep", "kmatrix", "outer", "photo"):
        n, nh, M = case["n"], case["nh"], case["M"]
        nt = case.get("levels") or n
        fl = float(n) * (n + 1) * nh + _dense_flops(n, kind == "photo")
        by = 8.0 * (nh * (n + 1.0) + M)
        if kind == "kmatrix":
            by += 16.0 * M * n * n
        elif kind == "photo":
            by += 8.0 * M
            if case["damped"]:  # complex: two sums, a complex solve
                fl = 2.0 * n * (n + 1) * nh + 8.0 / 3 * n ** 3
        else:
            by += 4.0 * M * nt * (nt + 1)
        if kind == "outer":
            fl += case["n_sec"] * (3.0 + 8.0 / 3) * n ** 3
            by += 8.0 * case["n_sec"] * n * n
        return dict(bytes=by, flops=M * fl)
    if kind == "plan":
        by, fl, L = 8.0 * case["M"], 0.0, case["levels"]
        for s in range(case["n_sym"]):
            f = s / max(1, case["n_sym"] - 1)
            n = int(round(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** f))
            fl += n * (n + 1.0) * 30 * n + _dense_flops(n)
            by += 8.0 * 30 * n * (n + 1)
        return dict(bytes=by + 4.0 * case["M"] * L * (L + 1), flops=case["M"] * fl)
    if kind == "inner":
        n, N = case["n"], case["n_basis"]
        D = n * N  # tridiagonalisation plus the eigenvectors, once
        return dict(bytes=8.0 * D * (n + 1), flops=9.0 * D ** 3 + n * n * N ** 2 * (N + 48.0))
    if kind == "post":
        M, P = case["M"], case["n_target"] * (case["n_target"] + 1) // 2
        win = 2 * 8 * case["fwhm"] / 2.3548 / case["step"] + 1
        return dict(bytes=8.0 * M * P * 2, flops=2.0 * M * P * min(win, M) + 4.0 * M * P * N_TEMPS)
    par = sum((fi + 1) * fo for fi, fo in
              [(case["d_in"] if i == 0 else case["width"],
                1 if i == case["n_layers"] - 1 else case["width"])
               for i in range(case["n_layers"])])
    return dict(bytes=4.0 * (par * 6 + case["batch"] * (case["d_in"] + 1)),
                flops=6.0 * par * case["batch"])


# ------------------------------------------------- the same in plain torch

def _lentz(a, b, f0, tol=1e-16, itmax=200000, done_from=None):
    """b0 + a1/(b1 + a2/(b2 + ...)): value and the sign flips of its
    denominators (modified Lentz); a(j), b(j) give the terms."""
    tiny = 1e-150
    f = torch.where(f0 == 0, tiny, f0)
    C, D, sgn = f.clone(), torch.zeros_like(f), torch.ones_like(f)
    calm = torch.zeros_like(f)
    for j in range(1, itmax):
        D = b(j) + a(j) * D
        D = 1.0 / torch.where(D == 0, tiny, D)
        C = b(j) + a(j) / C
        C = torch.where(C == 0, tiny, C)
        dlt = C * D
        live = calm < 3
        f = torch.where(live, f * dlt, f)
        sgn = torch.where(live & (D < 0), -sgn, sgn)
        ok = (dlt - 1.0).abs() < 4 * tol
        if done_from is not None:
            ok &= j > done_from
        calm = torch.where(live, torch.where(ok, calm + 1, 0.0), calm)
        if j % 32 == 0 and bool((calm >= 3).all()):
            break
    return f, sgn


def _channels(E, thr, l, r):
    """d1, d2, s, r s' [M, n] at radius r: (c, r c', s, r s') of the open
    Coulomb channels, the normalised decaying Whittaker pair of the closed."""
    diff = E[:, None] - thr[None, :]
    op = diff > 0
    L = l[None, :].expand_as(diff).to(torch.float64)
    k = diff.clamp(min=1e-300).sqrt()
    out = [torch.zeros_like(diff) for _ in range(4)]
    if bool(op.any()):
        Lo, ko = L[op], k[op]
        eta, rho = -Z_RES / ko, ko * r
        S = lambda m: m / rho + eta / m  # noqa: E731
        f, sgn = _lentz(lambda j: -(1.0 + (eta / (Lo + j)) ** 2),
                        lambda j: S(Lo + j) + S(Lo + j + 1), S(Lo + 1))
        a = torch.complex(-(eta * eta + Lo * (Lo + 1)), eta)
        b = torch.complex(2 * (rho - eta), torch.full_like(rho, 2.0))
        D = 1.0 / b
        dH = 1j / rho * a * D
        pq = 1j * (1 - eta / rho) + dH
        done = torch.zeros_like(op[op])
        for j in range(1, 200000):
            a = a + (2.0 * j + 2j * eta)
            b = b + 2j
            D = 1.0 / (a * D + b)
            dH = (b * D - 1.0) * dH
            pq = torch.where(done, pq, pq + dH)
            done = done | (dH.abs() < 1e-17 * pq.abs())
            if j % 32 == 0 and bool(done.all()):
                break
        p, q = pq.real, pq.imag
        F = sgn * (q / ((f - p) ** 2 + q * q)).sqrt()
        G = (f - p) * F / q
        sk = ko.sqrt()
        for o, v in zip(out, (G / sk, r * (p * G - q * F) * sk, F / sk, r * f * F * sk)):
            o[op] = v
    cl = ~op
    if bool(cl.any()):
        Lc, phi = L[cl], (-diff[cl]).sqrt()
        kap, x, mu = Z_RES / phi, 2 * phi * r, Lc + 0.5

        def an(j):
            return torch.ones_like(kap) if j == 1 else -((kap - (j - 1) - 0.5) ** 2 - mu * mu)
        f, _ = _lentz(an, lambda j: x + 2.0 * j - 2 * kap, torch.zeros_like(kap),
                      done_from=kap + mu + 2)
        ld = kap - 0.5 * x + ((kap - 0.5) ** 2 - mu * mu) * f
        nrm = torch.hypot(torch.ones_like(ld), ld)
        out[0][cl], out[1][cl] = 1.0 / nrm, ld / nrm
    return op, out


def _solve(A, B):
    """Batched solve, a few systems at a time (its library workspace grows
    with the batch)."""
    B = B.expand(A.shape[:1] + B.shape[-2:])
    k = max(1, int(1e6 / A.shape[-1] ** 2))
    return torch.cat([torch.linalg.solve(a, b) for a, b in
                      zip(torch.split(A, k), torch.split(B, k))])


def _dev(sym):
    return {k: torch.as_tensor(v, device="cuda") if isinstance(v, np.ndarray) else v
            for k, v in sym.items()}


def _pole_sum(S, E, poles=None):
    """R(E) [m, n, n]."""
    poles = S["E_pole"] if poles is None else poles
    d = 1.0 / (poles[None, :] - E[:, None])
    w = S["w"].to(d.dtype)
    return torch.stack([(w * x) @ w.T for x in d]) / (2 * S["a"])


def _solution(R, op, d1, d2, s, asp):
    """Z = [K; X] with zero columns at closed channels, and K [m, n, n]."""
    A = torch.diag_embed(d1) - R * d2[:, None, :]
    Bm = R * asp[:, None, :] - torch.diag_embed(s)
    Z = _solve(A, Bm * op[:, None, :])
    K = Z * op[:, :, None]
    return Z, 0.5 * (K + K.transpose(1, 2))


def _omega_of(K, target, nt, g):
    """Omega [m, P] of K [m, n, n] (closed rows and columns zero)."""
    m, n, _ = K.shape
    eye = torch.eye(n, device="cuda", dtype=torch.complex128)
    T2 = _solve(eye - 1j * K, 2j * K).abs() ** 2
    G = torch.zeros((n, nt), device="cuda", dtype=torch.float64)
    G[torch.arange(n), target] = 1.0
    V = torch.matmul(G.T.contiguous(), torch.matmul(T2, G)) * (g / 2)
    iu = torch.triu_indices(nt, nt, device="cuda")
    return V[:, iu[0], iu[1]]


def _propagate(X, S, case, beta, E):
    """a R(a) -> R(A) through the sectors (W frozen at each midpoint)."""
    h = (case["A"] - A_BOUND) / case["n_sec"]
    thr, l = S["e_thr"].cpu().numpy(), S["l"].cpu().numpy().astype(float)
    for t in range(case["n_sec"]):
        r = A_BOUND + (t + 0.5) * h
        W = np.diag(thr + l * (l + 1) / r ** 2 - 2 * Z_RES / r)
        for lam in range(beta.shape[0]):
            W = W + beta[lam] / r ** (lam + 2)
        eps, U = (torch.as_tensor(v, device="cuda") for v in np.linalg.eigh(W))
        X = torch.matmul(torch.matmul(U.T.contiguous(), X), U)
        k2 = E[:, None] - eps[None, :]
        k = k2.abs().sqrt()
        c = torch.where(k2 > 0, torch.cos(k * h), torch.cosh(k * h))
        s = torch.where(k2 > 0, torch.sin(k * h), torch.sinh(k * h)) / k
        N = c[:, :, None] * X + torch.diag_embed(s)
        D = torch.diag_embed(c) - (k2 * s)[:, :, None] * X
        Y = _solve(D.transpose(1, 2).contiguous(), N.transpose(1, 2).contiguous())
        X = 0.5 * (Y + Y.transpose(1, 2))
        X = torch.matmul(torch.matmul(U, X), U.T.contiguous())
    return X / case["A"]


def _chunks(E, n):
    return torch.split(E, max(1, min(E.numel(), int(2e7 / (n * n)))))


def _exact_sweep(case, inp):
    E = torch.as_tensor(inp["E"], device="cuda")
    nt, total = inp["n_target"], None
    for sym in inp["syms"]:
        S = _dev(sym)
        n = sym["e_thr"].size
        tgt = torch.arange(n, device="cuda") if sym["target"] is None else S["target"].long()
        rows = []
        for Ec in _chunks(E, n):
            R, r = _pole_sum(S, Ec), A_BOUND
            if case["kind"] == "outer":
                R, r = _propagate(A_BOUND * R, S, case, inp["beta"], Ec), case["A"]
            op, (d1, d2, s, asp) = _channels(Ec, S["e_thr"], S["l"], r)
            _, K = _solution(R, op, d1, d2, s, asp)
            if case["kind"] == "kmatrix":
                first = torch.argsort((~op).to(torch.int8), dim=1, stable=True)
                K = torch.gather(K, 1, first[:, :, None].expand_as(K))
                K = torch.gather(K, 2, first[:, None, :].expand_as(K))
                rows.append((K, R))
            else:
                rows.append(_omega_of(K, tgt, nt, sym["g"]))
        if case["kind"] == "kmatrix":
            return (torch.cat([k for k, _ in rows]), None, torch.cat([x for _, x in rows]), None)
        om = torch.cat(rows)
        total = om if total is None else total + om
    return total, None


def _exact_photo(case, inp):
    S = _dev(inp["syms"][0])
    n = case["n"]
    dip = torch.as_tensor(inp["dip"], device="cuda")
    poles = S["E_pole"]
    if case["damped"]:
        poles = poles - 0.5j * torch.as_tensor(inp["widths"], device="cuda")
    out = []
    for E in _chunks(torch.as_tensor(inp["E"], device="cuda"), n):
        R = _pole_sum(S, E, poles)
        w = S["w"].to(R.dtype)
        g = ((dip[None, :] / (poles[None, :] - E[:, None])) @ w.T) / math.sqrt(2.0)
        op, (d1, d2, s, asp) = _channels(E, S["e_thr"], S["l"], A_BOUND)
        if case["damped"]:
            A = torch.diag_embed(torch.complex(d1, s)) - R * torch.complex(d2, asp)[:, None, :]
            x = _solve(A, -g[:, :, None])[:, :, 0]
            S2 = ((x.abs() ** 2) * op).sum(1) / math.pi
        else:
            Z, K = _solution(R, op, d1, d2, s, asp)
            v = (asp * g * op + torch.matmul((d2 * g)[:, None, :], Z)[:, 0, :]) / A_BOUND
            eye = torch.eye(n, device="cuda", dtype=torch.float64)
            y = _solve(eye - 1j * K, v[:, :, None].to(torch.complex128))
            S2 = (y.abs() ** 2).sum((1, 2)) / math.pi
        out.append(SIGMA * (E - inp["e0"]) * S2)
    return torch.cat(out), None


def _exact_inner(case, inp):
    m, N = inp["model"], case["n_basis"]
    a, n, Q = m["a"], m["e_thr"].size, N + 48
    x, wq = np.polynomial.legendre.leggauss(Q)
    r, wq = 0.5 * a * (1 + x), 0.5 * a * wq
    kap = (np.arange(N) + 0.5) * math.pi / a
    phi = math.sqrt(2.0 / a) * np.sin(np.outer(r, kap))
    H = np.zeros((n * N, n * N))
    for i in range(n):
        for j in range(n):
            V = -m["depth"][i, j] * np.exp(-(r / m["range"][i, j]) ** 2)
            if i == j:
                V = V + m["l"][i] * (m["l"][i] + 1.0) / r ** 2 - 2 * m["z"] / r + m["e_thr"][i]
            H[i * N:(i + 1) * N, j * N:(j + 1) * N] = phi.T @ (phi * (wq * V)[:, None])
    H[np.arange(n * N), np.arange(n * N)] += np.tile(kap ** 2, n)
    return np.linalg.eigvalsh(0.5 * (H + H.T)), None


def _exact_post(case, inp, seed):
    E, om = _omega_table(case, inp, seed)
    M, nt = case["M"], case["n_target"]
    s = case["fwhm"] / (2 * math.sqrt(2 * math.log(2.0)))
    dE = torch.zeros_like(E)
    dE[:-1] += 0.5 * E.diff()
    dE[1:] += 0.5 * E.diff()
    x = E[None, :] - E[:, None]
    g = torch.where(x.abs() <= 8 * s, torch.exp(-0.5 * (x / s) ** 2) * dE, 0.0)
    sm = (g @ om) / g.sum(1, keepdim=True)
    lev, kT = torch.as_tensor(inp["lev"], device="cuda"), inp["kT"]
    iu = torch.triu_indices(nt, nt, device="cuda")
    up = torch.maximum(lev[iu[0]], lev[iu[1]])
    eps = E[:, None] - up[None, :]
    ok = eps > 0
    first = ok & ~torch.cat([torch.zeros_like(ok[:1]), ok[:-1]])
    ups = []
    for T in kT:
        y = torch.where(ok, om * torch.exp(-eps.clamp(min=0) / T), 0.0)
        mid = 0.5 * (y[1:] + y[:-1]) * (E.diff() / T)[:, None]
        ups.append((mid * ok[:-1]).sum(0) +
                   (torch.where(first, om * -torch.expm1(-eps.clamp(min=0) / T), 0.0)).sum(0))
    ng = min(N_GROUPS, nt)
    grp = torch.as_tensor(inp["group"], device="cuda").long()
    ga, gb = torch.minimum(grp[iu[0]], grp[iu[1]]), torch.maximum(grp[iu[0]], grp[iu[1]])
    go = torch.zeros((M, ng * (ng + 1) // 2), device="cuda", dtype=torch.float64)
    go.index_add_(1, ga * ng - ga * (ga - 1) // 2 + gb - ga, om)
    return sm, torch.stack(ups, 1), go


def _exact_train(case, seed):
    sizes, p, X, t = _net(case, seed)
    p = p.double().requires_grad_(True)
    h, at = X.double(), 0
    for i, (fi, fo) in enumerate(sizes):
        W = p[at:at + fo * fi].view(fo, fi)
        b = p[at + fo * fi:at + fo * fi + fo]
        at += fo * fi + fo
        h = h @ W.T + b
        if i + 1 < len(sizes):
            h = h * torch.sigmoid(h)
    loss = ((h[:, 0] - t.double()) ** 2).mean()
    loss.backward()
    return loss.detach().reshape(1), p.grad


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "outer" and case["terms"]:
        return None  # the coupled series has no short plain form
    inp = _inputs(case, seed)
    if kind == "photo":
        return _exact_photo(case, inp)
    if kind == "inner":
        return _exact_inner(case, inp)
    if kind == "post":
        return _exact_post(case, inp, seed)
    return _exact_sweep(case, inp)
