"""Calls under way on one stream (needs an MI355X) while the program goes on
with another: handles are changed and tensors let go of at once, and results are
those of the call."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def system():
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    w = wl.tiny(n=150, n_poles=4000, M=2048, mesh_lo=2.1, mesh_hi=2.5)
    h = native.load_symmetry(w.syms[0])
    E = torch.as_tensor(w.mesh, device="cuda:0")
    yield torch, native, h, E, torch.cuda.Stream()
    h.free()


@pytest.mark.parametrize("what", ["dipoles", "widths", "sectors"])
def test_handle_changed_while_a_call_is_under_way(system, what):
    torch, native, h, E, side = system
    rng = np.random.default_rng(3)
    d = [rng.normal(size=h.n_poles) for _ in range(2)]
    g = [10.0 ** rng.uniform(-4, -2, h.n_poles) for _ in range(2)]
    native.rm_load_dipoles(h, d[0])
    native.rm_load_widths(h, g[0])
    damped = native.make_opts(flags=native.RM_FLAG_RADIATION_DAMPING)
    load, call = {
        "dipoles": (lambda k: native.rm_load_dipoles(h, d[k]),
                    lambda: native.rm_photoionization([h], E, -0.8)[0]),
        "widths": (lambda k: native.rm_load_widths(h, g[k]),
                   lambda: native.rm_photoionization([h], E, -0.8, damped)[0]),
        "sectors": (lambda k: native.rm_set_propagation(h, 25.0 + 5.0 * k, 2),
                    lambda: native.rm_sweep_energies([h], 150, E[:256])[0])}[what]
    ref = []
    for k in (1, 0):
        load(k)
        ref.insert(0, call().cpu().numpy())
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        first = call()
    load(1)  # from the default stream, which does not wait for the other
    second = call()
    torch.cuda.synchronize()
    assert np.array_equal(first.cpu().numpy(), ref[0])
    assert np.array_equal(second.cpu().numpy(), ref[1])
    assert not np.array_equal(ref[0], ref[1])
    if what == "sectors":
        native.rm_set_propagation(h, 25.0, 0)


@pytest.mark.parametrize("call", ["sweep", "photo", "kmatrix", "rmatrix"])
def test_tensors_of_another_stream_outlive_the_call(system, call):
    torch, native, h, E0, side = system
    native.rm_load_dipoles(h, np.ones(h.n_poles))
    M = 2048 if call in ("sweep", "photo") else 1024
    run = {"sweep": lambda E, o, s: native.rm_sweep_energies([h], 150, E, omega=o,
                                                             status=s),
           "photo": lambda E, o, s: native.rm_photoionization([h], E, -0.8,
                                                              sigma=o, status=s),
           "kmatrix": lambda E, o, s: native.rm_kmatrix(h, E),
           "rmatrix": lambda E, o, s: native.rm_rmatrix(h, E)}[call]
    width = {"sweep": 150 * 151 // 2, "photo": 1}.get(call, 1)
    for warm in (True, False):
        E = E0[:M].clone()
        o = torch.empty(M * width, dtype=torch.float64, device="cuda:0")
        s = torch.empty(M, dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            out = run(E, o, s)
        done = torch.cuda.Event()
        done.record(side)
        used = {E.data_ptr()}
        if call in ("sweep", "photo"):
            used |= {o.data_ptr(), s.data_ptr()}
        del out, E, o, s
        if warm:
            torch.cuda.synchronize()
    again = [torch.empty(M, dtype=torch.float64, device="cuda:0"),
             torch.empty(M * width, dtype=torch.float64, device="cuda:0"),
             torch.empty(M, dtype=torch.int32, device="cuda:0")]
    assert not done.query(), "the call was over before its tensors were looked at"
    assert not used & {t.data_ptr() for t in again}
    torch.cuda.synchronize()
