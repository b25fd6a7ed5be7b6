"""The autotuner's FP64 choice (needs an MI355X) is one per class of mesh: what
was fastest on a coarse mesh is not taken for a fine one, and entries that do not
say which mesh they were timed on are not read."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

_SCRIPT = r"""
import sys, numpy as np, torch
sys.path.insert(0, sys.argv[1])
from paper_1403_5524_amd import native as nat, workloads as wl
s = wl.tiny(n=100, n_poles=3000, M=8, seed=5).syms[0]
h = nat.load_symmetry(s)
for step in (0.06, 1e-5):  # poles near at every energy; all but a few far
    E = torch.as_tensor(2.5 + step * (np.arange(512) + 0.5), device="cuda:0")
    p = nat.Plan([h], 100, E, nat.make_opts(flags=nat.RM_FLAG_AUTOTUNE))
    print("variant", p.info()[2][0])
    p.free()
"""
SCALED_W, PAIRS = 0, 5


@pytest.mark.parametrize("entry,coarse,fine", [
    ("100 3000 0 5 0", [PAIRS], [SCALED_W]),           # a coarse mesh's choice
    ("100 3000 0 5", [SCALED_W, PAIRS], [SCALED_W])])  # of no known mesh
def test_fp64_choice_is_kept_per_mesh_class(tmp_path, entry, coarse, fine):
    cache = tmp_path / "tune.txt"
    cache.write_text(entry + "\n77 999 2 3\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _SCRIPT, root],
                       env=dict(os.environ, RM_TUNE_CACHE=str(cache)),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    got = [int(x.split()[1]) for x in r.stdout.split("\n")
           if x.startswith("variant")]
    assert got[0] in coarse and got[1] in fine
    lines = cache.read_text().split("\n")
    assert "100 3000 0 %d 0" % got[0] in lines      # both classes are kept,
    assert "100 3000 0 %d 3" % got[1] in lines      # and the mixed entry
    assert "77 999 2 3" in lines
