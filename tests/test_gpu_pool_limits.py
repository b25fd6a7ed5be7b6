"""Calls that need more memory than the device has free beside what the library
keeps between calls (needs an MI355X): they get it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GB = 1 << 30


def _network(native, torch):
    m = native.Mlp(8, 1024, 2)
    # Z and A of 2 x 1024 values a sample, dA and dZ of 1024: 24 kB a sample
    Y = m.forward(torch.zeros((110000, 8), device="cuda:0"))
    assert bool((Y == Y[0]).all())
    m.free()


def _upsilon(native, torch):
    M = 1000000  # a factor for each energy and temperature: 2 GB
    E = torch.linspace(0.1, 1.0, M, dtype=torch.float64, device="cuda:0")
    om = torch.ones((M, 1), dtype=torch.float64, device="cuda:0")
    ups = native.rm_effective_collision_strengths(
        E, om, [0.0], 1, np.linspace(0.01, 0.02, 270))
    assert bool(torch.isfinite(ups).all())


def _inner(native, torch):
    n = 256  # quadrature tables of 256 x 256 x 4096 values: 2.1 GB
    model = dict(e_thr=np.zeros(n), l=np.zeros(n, dtype=np.int32), z=1.0, a=5.0,
                 depth=np.eye(n), range=np.ones((n, n)))
    E, _, _, _ = native.rm_inner_region(model, 1, 4096)
    assert np.allclose(E, E[0], rtol=1e-10)  # n channels that are not coupled


@pytest.mark.parametrize("call", [_network, _upsilon, _inner])
def test_kept_memory_does_not_stand_in_the_way(call):
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    torch.cuda.empty_cache()
    n, M = 100, 16384
    w = wl.tiny(n=n, n_poles=150, M=M)
    h = native.load_symmetry(w.syms[0])
    E = torch.as_tensor(w.mesh, device="cuda:0")
    native.rm_sweep_energies([h], n, E)  # 3.9 GB of workspace, kept
    torch.cuda.synchronize()  # (emptying torch's cache would free the pool)
    fill = []
    try:
        for _ in range(3):  # what is asked for and what goes differ a little
            left = torch.cuda.mem_get_info()[0] - GB
            if left > 0:
                fill.append(torch.empty(left, dtype=torch.uint8, device="cuda:0"))
        assert torch.cuda.mem_get_info()[0] < 2 * GB
        call(native, torch)
        torch.cuda.synchronize()
    finally:
        fill.clear()
        torch.cuda.empty_cache()
        h.free()


def test_network_after_a_batch_that_does_not_fit():
    """The activations of 2^31 - 1 samples (70 TB) are refused, and the network
    still serves the batches it served before."""
    import torch
    from paper_1403_5524_amd import native
    m = native.Mlp(1, 4096, 2)
    X = torch.linspace(-1, 1, 8, device="cuda:0")[:, None].contiguous()
    Y = m.forward(X).cpu()
    with pytest.raises(native.RmError) as ei:
        m.forward(torch.empty((2 ** 31 - 1, 1), device="cuda:0"))
    assert ei.value.code == native.RM_ERR_NOMEM
    assert torch.equal(m.forward(X).cpu(), Y)
    m.free()
    torch.cuda.empty_cache()
