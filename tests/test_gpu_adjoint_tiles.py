"""The adjoint's tiles: list entries that reach no target are left out, and
target blocks that four entries cannot reach are skipped.  Group sizes at the
edges of the target blocks of 16, cutoffs from a fraction of a spacing (nearly
every entry left out) to several, both forms of the far distance (eps), and
fresh and refitted trees, element-wise against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1211_4406_amd as srf
import synth
from _parity import U32, U64, check, constant, max_list

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_group", [1, 16, 17, 33, 49, 64])
@pytest.mark.parametrize("r_cut,eps", [(0.012, 1e-4), (0.05, 3e-4), (0.05, 5e-3), (0.2, 1e-3)])
@pytest.mark.parametrize("refit", [False, True])
def test_adjoint_of_tiles(n_group, r_cut, eps, refit):
    n = 3001
    rng = np.random.default_rng(2100 + n_group)
    pos = np.concatenate([rng.random((n // 2, 3)), np.mod(0.97 + 0.05 * rng.standard_normal((n - n // 2, 3)), 1.0)])
    w = synth.loss_weights(n, 2101)
    params = synth.Params(1.0, r_cut, eps, 0.6, n_group, min(8, n_group))
    print(f"[gpu] adjoint tiles n_group={n_group} r_cut={r_cut} eps={eps} refit={refit}", flush=True)
    m = rng.uniform(0.5, 1.5, n) / n
    ref = oracle.OracleTree(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), m, params)
    p = srf.Params.of(params)
    tree = srf.tree_build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), p)
    if refit:
        new = pos + 4e-3 * (2 * rng.random((n, 3)) - 1)
        srf.tree_refit(tree, torch.tensor(new, device="cuda"))
        ref = ref.refitted(new[:, 0], new[:, 1], new[:, 2])
    lists = srf.make_lists(tree, p)
    wt = torch.tensor(w, device="cuda")
    rx, rm = ref.adjoint(w)
    for fp64, u in ((False, U32), (True, U64)):
        q = srf.Params.of(params, srf.FP64 if fp64 else srf.FP32_REL)
        gx, gm = srf.short_range_adjoint(tree, lists, q, wt)
        Ex, Em = ref.adjoint_bound(w, u)
        C = constant("adjoint", fp64, max_list(ref))
        check(gx.cpu().numpy(), rx, Ex, C, f"dL/dx fp64={fp64}")
        check(gm.cpu().numpy(), rm, Em, C, f"dL/dm fp64={fp64}")
