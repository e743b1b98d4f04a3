"""The two walks that build the interaction lists (one wave per group; one
thread per group for large trees and for lists that a wave's buffer does not
hold) give the oracle's lists bit for bit: single-particle leaves make one
item per entry, so that the groups' item counts spread over every size of the
wave's final sort (up to 256, 512, 1024 and 2048 items) and past its buffer.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1211_4406_amd as srf
import synth

SIZES = [(0.03, 0, 256, 6001), (0.07, 257, 512, 6001), (0.13, 513, 1024, 6001), (0.23, 1025, 2048, 6001),
         (0.245, 2049, 4096, 6001), (0.245, 4097, 20000, 40001)]


def _set(r_cut, n):
    rng = np.random.default_rng(77)
    pos = rng.random((n, 3))
    p = synth.Params(1.0, r_cut, 1e-3, 0.25, 64, 1)
    return synth.ParticleSet(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), np.full(n, 1.0 / n), p)


def _items(lists):
    return np.diff(lists.poff) + np.diff(lists.noff)


@pytest.mark.parametrize("r_cut,lo,hi,n", SIZES)
def test_item_counts_reach_each_size(r_cut, lo, hi, n):
    ps = _set(r_cut, n)
    ot = oracle.OracleTree(ps.x, ps.y, ps.z, ps.m, ps.params)
    assert lo <= _items(ot.lists).max() <= hi, _items(ot.lists).max()


@pytest.mark.gpu
@pytest.mark.parametrize("r_cut,lo,hi,n", SIZES)
@pytest.mark.parametrize("refit", [False, True])
def test_lists_of_every_size(r_cut, lo, hi, n, refit):
    ps = _set(r_cut, n)
    print(f"[gpu] walk r_cut={r_cut} n={n} refit={refit}", flush=True)
    p = srf.Params.of(ps.params)
    x = torch.tensor(ps.positions(), device="cuda")
    tree = srf.tree_build(x, torch.tensor(ps.m, device="cuda"), p)
    ref = oracle.OracleTree(ps.x, ps.y, ps.z, ps.m, ps.params)
    if refit:
        new = ps.positions() + 2e-3 * (2 * np.random.default_rng(78).random((ps.n, 3)) - 1)
        srf.tree_refit(tree, torch.tensor(new, device="cuda"))
        ref = ref.refitted(new[:, 0], new[:, 1], new[:, 2])
    got = srf.make_lists(tree, p)
    L = got.export()
    for k in ("poff", "pidx", "noff", "nidx"):
        assert np.array_equal(L[k], getattr(ref.lists, k)), k
    info = got.info()
    assert info["interactions"] == ref.interactions()
    assert info["n_particle_entries"] == ref.lists.pidx.size and info["n_node_entries"] == ref.lists.nidx.size
