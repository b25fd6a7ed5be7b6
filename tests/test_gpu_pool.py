"""Workspace kept between calls (needs an MI355X): calls from several threads
on their own streams share it, and it goes back with the last handle."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_threads_and_streams_share_the_workspace_pool():
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    work, ref = [], []
    for n, nh, M in ((8, 100, 300), (40, 600, 200), (5, 64, 48)):
        w = wl.tiny(n=n, n_poles=nh, M=M, seed=n)
        h = native.load_symmetry(w.syms[0])
        E = torch.as_tensor(w.mesh, device="cuda:0")
        om, _ = native.rm_sweep_energies([h], n, E)
        torch.cuda.synchronize()
        work.append((h, n, E))
        ref.append(om.cpu().numpy())
    bad = []

    def run(k):
        h, n, E = work[k]
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                om, _ = native.rm_sweep_energies([h], n, E)
                if not np.array_equal(om.cpu().numpy(), ref[k]):
                    bad.append(k)
    threads = [threading.Thread(target=run, args=(k,)) for k in (0, 1, 2, 0)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for h, _, _ in work:
        h.free()


def test_pool_is_given_back_with_the_last_handle():
    import gc
    import torch
    from paper_1403_5524_amd import native, workloads as wl
    gc.collect()  # handles of earlier tests
    torch.cuda.synchronize()
    w = wl.tiny(n=100, n_poles=600, M=2048)
    h = native.load_symmetry(w.syms[0])
    E = torch.as_tensor(w.mesh, device="cuda:0")
    om, _ = native.rm_sweep_energies([h], 100, E)
    torch.cuda.synchronize()
    held = torch.cuda.mem_get_info()[0]
    h.free()
    torch.cuda.synchronize()
    # at least the 3 n^2 doubles of workspace per energy
    assert torch.cuda.mem_get_info()[0] - held > 0.9 * 8 * 3 * 100 ** 2 * 2048
