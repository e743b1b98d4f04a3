"""The PM step's boxes and runs: workgroups whose particles' mesh points fit a
box in LDS, in one piece or several, and those that do not (sparse sets on a
fine mesh; a refitted tree whose particles are no longer in mesh order); runs
of one particle to thousands in one mesh cell; boxes across the faces; both
parities of log2(n_mesh).  Both sides compute in FP64 with the same formulas
and differ by the FFT's and the sums' order: 1e-10 of the force's norm, as for
the other PM tests."""
import numpy as np
import pytest
import torch

import paper_1211_4406_amd as srf
from oracle import pm

pytestmark = pytest.mark.gpu
PM_TOL = 1e-10


def _positions(name, rng):
    if name == "pair":
        return np.array([[0.999, 0.5, 0.25], [0.02, 0.49, 0.3]])
    if name == "sparse":
        return rng.random((3001, 3))
    if name == "corner":     # across the box's corner, thousands to a mesh cell
        return np.mod(0.01 * rng.standard_normal((9001, 3)), 1.0)
    return np.concatenate([rng.random((4097, 3)), np.mod(0.3 + 0.02 * rng.standard_normal((4096, 3)), 1.0)])


@pytest.mark.parametrize("name", ["pair", "sparse", "corner", "mixed"])
@pytest.mark.parametrize("n_mesh", [16, 32, 64, 128])
@pytest.mark.parametrize("moved", [False, True])
def test_pm_boxes(name, n_mesh, moved):
    rng = np.random.default_rng(2300)
    pos = _positions(name, rng)
    n = len(pos)
    m = rng.uniform(0.5, 1.5, n) / n
    print(f"[gpu] pm boxes {name} n_mesh={n_mesh} moved={moved}", flush=True)
    p = srf.Params(r_cut=0.1)
    tree = srf.tree_build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), p)
    if moved:
        pos = pos[rng.permutation(n)]
        srf.tree_refit(tree, torch.tensor(pos, device="cuda"))
    r_cut = 3.0 / max(n_mesh, 16)
    a = srf.pm_force(tree, 1.0, r_cut, n_mesh).cpu().numpy()
    ref = pm.pm_force(pos[:, 0], pos[:, 1], pos[:, 2], m, 1.0, r_cut, n_mesh)
    assert np.linalg.norm(a - ref) <= PM_TOL * np.linalg.norm(ref)
