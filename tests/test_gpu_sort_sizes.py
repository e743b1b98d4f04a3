"""The sort and its inputs' gather at the sizes where its kernels change: tiles
of 1024 keys, the largest set that takes them, and larger ones; clumps whose
members share the high key word, up to and past the longest run that is ordered
by counting, on both sides; strided inputs; repeated positions.  Keys,
permutation and sorted particles equal a stable sort on the host."""
import numpy as np
import pytest
import torch

import oracle
import paper_1211_4406_amd as srf

pytestmark = pytest.mark.gpu
FEW = 1 << 21


@pytest.mark.parametrize("n,clump", [(1, 0), (2, 2), (63, 0), (64, 64), (1023, 300), (1024, 1024), (1025, 1025),
                                     (4097, 3000), (FEW, 1024), (FEW, 1025), (FEW + 1, 1024), (FEW + 1, 1025)])
@pytest.mark.parametrize("strided", [False, True])
def test_sort_sizes(n, clump, strided):
    print(f"[gpu] sort n={n} clump={clump} strided={strided}", flush=True)
    rng = np.random.default_rng(2400 + n + clump)
    pos = rng.random((n, 3))
    pos[:clump] = (5 + 0.5) / 2 ** 11 + (rng.random((clump, 3)) - 0.5) * 2e-4   # one high key word
    pos[: clump // 3] = pos[clump // 3: 2 * (clump // 3)]                       # repeated positions
    pos = pos[rng.permutation(n)]
    m = rng.uniform(0.5, 1.5, n)
    keys = oracle.morton_keys(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy())
    keys = np.asarray(keys[0] if isinstance(keys, tuple) else keys).astype(np.uint64)
    perm = np.argsort(keys, kind="stable")
    x, mt = torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda")
    if strided:
        wide = torch.zeros((n, 5), dtype=torch.float64, device="cuda")
        wide[:, 1:4] = x
        x, mt = wide[:, 1:4], torch.stack([mt, mt], dim=1)[:, 0]
    tree = srf.tree_build(x, mt, srf.Params())
    ex = tree.export()
    assert np.array_equal(ex["keys"], keys[perm]) and np.array_equal(ex["perm"], perm)
    xs, ms = tree.sorted_particles()
    assert np.array_equal(xs, pos[perm]) and np.array_equal(ms, m[perm])


@pytest.mark.parametrize("n", [1023, 2049, 4095, 4096])
@pytest.mark.parametrize("kind", ["uniform", "one key", "two keys", "descending"])
def test_sort_by_one_workgroup(n, kind):
    """Up to 4096 keys are sorted by one workgroup; 4097 and up are in test_sort_sizes."""
    print(f"[gpu] sort by one workgroup n={n} {kind}", flush=True)
    rng = np.random.default_rng(2900 + n)
    pos = rng.random((n, 3))
    if kind == "one key":
        pos[:] = (5 + 0.5) / 2 ** 11 + (rng.random((n, 3)) - 0.5) * 2e-4
    elif kind == "two keys":   # stable: ties stay in input order
        pos = np.where(rng.random((n, 1)) < 0.5, 0.125, 0.875) * np.ones((1, 3))
    elif kind == "descending":
        pos = np.sort(pos, axis=0)[::-1].copy()
    keys = oracle.morton_keys(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy())
    keys = np.asarray(keys[0] if isinstance(keys, tuple) else keys).astype(np.uint64)
    perm = np.argsort(keys, kind="stable")
    m = rng.uniform(0.5, 1.5, n)
    ex = srf.tree_build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), srf.Params()).export()
    assert np.array_equal(ex["keys"], keys[perm]) and np.array_equal(ex["perm"], perm)
