"""The quadrupole pass's chunks: cells that reach no target are left out, and
several waves share a group of a small tree.  Group sizes, cutoffs from a
fraction of a spacing to several, fresh and refitted trees: the force with
quadrupole cells against the FP64 oracle.  The monopole force is held to its
element-wise bound elsewhere; the total keeps the tolerances of the other
quadrupole tests, taken of the norm."""
import numpy as np
import pytest
import torch

import oracle
import paper_1211_4406_amd as srf
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_group", [8, 33, 64])
@pytest.mark.parametrize("r_cut", [0.03, 0.08, 0.2])
@pytest.mark.parametrize("refit", [False, True])
def test_quadrupole_of_chunks(n_group, r_cut, refit):
    n = 5003
    rng = np.random.default_rng(2500 + n_group)
    pos = np.concatenate([rng.random((n // 2, 3)), np.mod(0.97 + 0.05 * rng.standard_normal((n - n // 2, 3)), 1.0)])
    m = rng.uniform(0.5, 1.5, n) / n
    params = synth.Params(1.0, r_cut, 3e-4, 0.8, n_group, 4)
    print(f"[gpu] quadrupole chunks n_group={n_group} r_cut={r_cut} refit={refit}", flush=True)
    ref = oracle.OracleTree(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), m, params)
    p = srf.Params.of(params)
    tree = srf.tree_build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), p)
    if refit:
        new = pos + 4e-3 * (2 * rng.random((n, 3)) - 1)
        srf.tree_refit(tree, torch.tensor(new, device="cuda"))
        ref = ref.refitted(new[:, 0], new[:, 1], new[:, 2])
    lists = srf.make_lists(tree, p)
    want = ref.force_quadrupole()
    for precision, tol in ((srf.FP32_REL, 1e-5), (srf.FP64, 1e-12)):
        q = srf.Params.of(params, precision)
        a = srf.short_range_force(tree, lists, q, quadrupole=True).cpu().numpy()
        assert np.linalg.norm(a - want) <= tol * np.linalg.norm(want)
