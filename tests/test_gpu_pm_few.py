"""The PM step on either side of the 65536 particles from which the assignment
takes boxes of pieces, and below, where it takes one box or none: uniform and clustered sets, in mesh order, drifted by a
cell of the mesh since their tree was made, and in no order.  Both sides compute
in FP64 with the same formulas and differ by the FFT's and the sums' order:
1e-10 of the force's norm, as for the other PM tests."""
import numpy as np
import pytest
import torch

import paper_1211_4406_amd as srf
from oracle import pm

pytestmark = pytest.mark.gpu
PM_TOL = 1e-10


@pytest.mark.parametrize("n", [40001, 65535, 65536, 70001])
@pytest.mark.parametrize("name", ["uniform", "ball"])
@pytest.mark.parametrize("n_mesh", [16, 32, 64])
@pytest.mark.parametrize("moved", ["no", "drifted", "shuffled"])
def test_pm_few(n, name, n_mesh, moved):
    rng = np.random.default_rng(2310)
    pos = rng.random((n, 3)) if name == "uniform" else np.mod(0.99 + 0.01 * rng.standard_normal((n, 3)), 1.0)
    m = rng.uniform(0.5, 1.5, n) / n
    print(f"[gpu] pm few n={n} {name} n_mesh={n_mesh} moved={moved}", flush=True)
    tree = srf.tree_build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), srf.Params(r_cut=0.1))
    if moved != "no":
        pos = (np.mod(pos + rng.standard_normal((n, 3)) / n_mesh, 1.0) if moved == "drifted"
               else pos[rng.permutation(n)])
        srf.tree_refit(tree, torch.tensor(pos, device="cuda"))
    r_cut = 3.0 / n_mesh
    a = srf.pm_force(tree, 1.0, r_cut, n_mesh).cpu().numpy()
    ref = pm.pm_force(pos[:, 0], pos[:, 1], pos[:, 2], m, 1.0, r_cut, n_mesh)
    assert np.linalg.norm(a - ref) <= PM_TOL * np.linalg.norm(ref)
