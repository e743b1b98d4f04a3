"""The force's tiles: list entries that reach no target
are left out, and several waves share a group of a small tree (whole tiles, or
chunks of them when a list has fewer tiles than waves).  Group sizes on both
sides of every stream count, cutoffs from a fraction of a spacing to several,
both forms of the far distance (eps), plain and compensated FP32 and FP64,
fresh and refitted trees, against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_1211_4406_amd as srf
import synth
from _parity import U32, U64, check, constant, max_list

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_group", [1, 8, 9, 16, 17, 21, 22, 32, 33, 64])
@pytest.mark.parametrize("r_cut,eps", [(0.012, 1e-4), (0.05, 3e-4), (0.05, 5e-3), (0.2, 1e-3)])
@pytest.mark.parametrize("refit", [False, True])
def test_force_of_tiles(n_group, r_cut, eps, refit):
    n = 3001
    rng = np.random.default_rng(2200 + n_group)
    pos = np.concatenate([rng.random((n // 2, 3)), np.mod(0.97 + 0.05 * rng.standard_normal((n - n // 2, 3)), 1.0)])
    params = synth.Params(1.0, r_cut, eps, 0.6, n_group, min(8, n_group))
    print(f"[gpu] force tiles n_group={n_group} r_cut={r_cut} eps={eps} refit={refit}", flush=True)
    m = rng.uniform(0.5, 1.5, n) / n
    ref = oracle.OracleTree(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), m, params)
    p = srf.Params.of(params)
    tree = srf.tree_build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), p)
    if refit:
        new = pos + 4e-3 * (2 * rng.random((n, 3)) - 1)
        srf.tree_refit(tree, torch.tensor(new, device="cuda"))
        ref = ref.refitted(new[:, 0], new[:, 1], new[:, 2])
    lists = srf.make_lists(tree, p)
    a_ref = ref.force()
    for fp64, comp in ((False, 0), (False, 1), (True, 0)):
        q = dataclasses.replace(p, precision=srf.FP64 if fp64 else srf.FP32_REL, compensated=comp)
        a = srf.short_range_force(tree, lists, q).cpu().numpy()
        check(a, a_ref, ref.force_bound(U64 if fp64 else U32), constant("force", fp64, max_list(ref)),
              f"force fp64={fp64} compensated={comp}")


@pytest.mark.parametrize("n_group", [34, 43, 50, 51])
@pytest.mark.parametrize("r_cut", [0.004, 0.03, 0.24])
@pytest.mark.parametrize("n", [49, 130, 2357])
def test_force_of_numbered_pairs_of_chunks_and_targets(n_group, r_cut, n):
    """Groups of 33 to 50 targets take the lanes by (chunk, target) pairs: lists from one short chunk
    to several tiles, and last rounds of fewer pairs than there are chunks."""
    rng = np.random.default_rng(4700 + n_group + n)
    pos = np.mod(0.5 + 0.04 * rng.standard_normal((n, 3)), 1.0)
    params = synth.Params(1.0, r_cut, 1e-3, 0.5, n_group, 8)
    print(f"[gpu] force pairs n={n} n_group={n_group} r_cut={r_cut}", flush=True)
    m = rng.uniform(0.5, 1.5, n) / n
    ref = oracle.OracleTree(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), m, params)
    p = srf.Params.of(params)
    tree = srf.tree_build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), p)
    lists = srf.make_lists(tree, p)
    a_ref = ref.force()
    for fp64 in (False, True):
        q = dataclasses.replace(p, precision=srf.FP64 if fp64 else srf.FP32_REL)
        a = srf.short_range_force(tree, lists, q).cpu().numpy()
        check(a, a_ref, ref.force_bound(U64 if fp64 else U32), constant("force", fp64, max_list(ref)),
              f"force fp64={fp64}")
