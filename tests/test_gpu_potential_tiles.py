"""The potential's tiles: entries that reach no target are left out, one, four
or eight waves share a group (whole tiles, or chunks of them), and trees of
groups of at most 8 targets take a kernel of their own.  Group sizes on both
sides of every stream count, cutoffs from a fraction of a spacing to several,
both forms of the far distance (eps), fresh and refitted trees, against the
FP64 oracle over the same lists: FP32 element by element, FP64 to 1e-12 of the
norm, as for the other potential tests (the oracle's own rounding is as large
as the FP64 kernel's).

Bound.  With FP32's unit roundoff u, a pair's offset d is the
difference of two rounded offsets p, x from the group's centre: it is off by at
most e = u (|p| + |x| + |d|), plus the FP64 error of a cell's centre of mass,
u64 (2 n_c + 2).  s^2 is off by 3 u relatively, s^-1 by 4 u and by the offset's
r e / s^2; r by at most 10 u (the far form s^2 s^-1 - eps^2 / 2 s^-1, its
truncation below u / 2 included) and by e.  Then
  t = 2 - k r is off by dt = 24 u + k e, and q = t^6 R / 140 by
  ((t + dt)^6 - t^6) R / 140 + 25 u q  (five products, R to 15 u);
  the inner polynomial, of terms c_n xi^n of sum A and derivative sum A', by
  50 u A + k e A'
(both taken within 0.1 % of xi = 1, where either may be chosen), and m q / s by
7 u more.  A lane adds at most 32 terms before FP64, and the oracle its list
in FP64: (32 u + L u64) times the sum of the terms.  A twentieth is added for
the second order."""
import numpy as np
import pytest
import torch

import bench
import oracle
import paper_1211_4406_amd as srf
import synth
from _parity import U32, U64, say

FP64_TOL = 1e-12
GROUPS = [1, 8, 9, 16, 17, 21, 22, 32, 33, 64]
CUTS = [(0.012, 1e-4, 0.6), (0.05, 5e-3, 0.6), (0.2, 1e-3, 0.6)]
SETS = [(1201, g, *c) for g in GROUPS for c in CUTS] + [(1201, 64, 0.004, 1e-4, 0.6)]
# small groups with lists long enough for eight waves
SETS += [(3001, 8, 0.24, 1e-3, 0.2), (2001, 16, 0.2, 1e-3, 0.4), (2001, 21, 0.2, 1e-3, 0.5)]
# more than 700 groups with work for several waves: four
SETS += [(6001, 8, 0.2, 1e-3, 0.3), (12001, 16, 0.1, 1e-3, 0.5), (12001, 21, 0.1, 1e-3, 0.5),
         (20001, 32, 0.1, 3e-4, 0.5), (40001, 64, 0.05, 3e-4, 0.6)]


def _set(n, n_group, r_cut, eps, theta):
    rng = np.random.default_rng(3200 + n_group)
    pos = np.concatenate([rng.random((n // 2, 3)), np.mod(0.97 + 0.05 * rng.standard_normal((n - n // 2, 3)), 1.0)])
    m = rng.uniform(0.5, 1.5, n) / n
    params = synth.Params(1.0, r_cut, eps, theta, n_group, min(8, n_group))
    return pos, m, params, oracle.OracleTree(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), m, params), rng


def _waves(ref):
    L = ref.lists
    return bench.waves_per_group(dict(n_groups=ref.n_groups, n_particle_entries=L.pidx.size,
                                      n_node_entries=L.nidx.size, interactions=ref.interactions()), 26.0)


def _image(d):
    return d - np.rint(d)


def bound(ref, u):
    p, L = ref.params, ref.lists
    k = 2.0 / p.r_cut
    x = np.stack([ref.ux, ref.uy, ref.uz], axis=1)
    out = np.empty(ref.n)
    for g in range(ref.n_groups):
        f, c = int(ref.gfirst[g]), int(ref.gcount[g])
        part, cell = L.pidx[L.poff[g]:L.poff[g + 1]], L.nidx[L.noff[g]:L.noff[g + 1]]
        cen = 0.5 * (ref.lo[g] + ref.hi[g])
        src = _image(np.concatenate([x[part], ref.X[cell]]) - cen)
        m = np.concatenate([ref.m[part], ref.M[cell]])
        com = np.concatenate([np.zeros(part.size), 2.0 * ref.tree.count[cell] + 2.0]) * U64
        me = _image(x[f:f + c] - cen)
        d = src[None] - me[:, None]
        r = np.sqrt((d * d).sum(axis=2))
        e = u * (np.linalg.norm(src, axis=1)[None] + np.linalg.norm(me, axis=1)[:, None] + r) + com[None]
        s = np.sqrt(r * r + p.eps ** 2)
        xi = k * r
        t, dt = np.maximum(2.0 - xi, 0.0), 24 * u + k * e
        R = (xi * xi + 4 * xi + 2) / 140
        outer = np.where(xi < 2 + dt, ((t + dt) ** 6 - t ** 6) * R, 0.0)
        A = 1 + xi * (52 / 35 + xi ** 2 * (4 / 5 + xi ** 2 * (2 / 5 + xi * (1 / 10 + xi * (2 / 35 + 3 / 140 * xi)))))
        dA = 52 / 35 + xi ** 2 * (12 / 5 + xi ** 2 * (2 + xi * (3 / 5 + xi * (2 / 5 + 6 / 35 * xi))))
        inner = 50 * u * A + k * e * dA
        q = np.where(xi < 1, 1 + xi * (-52 / 35 + xi ** 2 * (4 / 5 + xi ** 2 * (-2 / 5 + xi * (1 / 10 + xi * (
            2 / 35 - 3 / 140 * xi))))), t ** 6 * R)
        dq = np.where(xi <= 1.001, inner, 0.0) + np.where(xi >= 0.999, outer + 25 * u * q, 0.0)
        own = np.concatenate([part, np.full(cell.size, -1)])[None] == np.arange(f, f + c)[:, None]
        w = np.where(own, 0.0, m[None] / s)
        out[f:f + c] = (w * (dq + q * (7 * u + r * e / s ** 2))).sum(axis=1) + (32 * u + m.size * U64) * (w * q).sum(axis=1)
    res = np.empty(ref.n)
    res[ref.perm] = 1.05 * abs(p.G) * out
    return res


def test_sets_reach_every_instance():
    """Every stream count with one wave and with several, and four and eight waves."""
    seen = set()
    for s in SETS:
        ref = _set(*s)[3]
        top = int(ref.gcount.max())
        seen.add((_waves(ref), 1 if top > 32 else 2 if top > 21 else 3 if top > 16 else 4 if top > 8 else 8))
    assert seen >= {(w, st) for w in (1, 4, 8) for st in (1, 2, 3, 4, 8)}, sorted(seen)


@pytest.mark.gpu
@pytest.mark.parametrize("case", SETS, ids=lambda c: f"{c[0]}-{c[1]}-{c[2]}-{c[3]}")
@pytest.mark.parametrize("refit", [False, True])
def test_potential_of_tiles(case, refit):
    pos, m, params, ref, rng = _set(*case)
    n = len(pos)
    say(f"[gpu] potential tiles {case} refit={refit}")
    p = srf.Params.of(params)
    tree = srf.tree_build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), p)
    if refit:
        new = pos + 4e-3 * (2 * rng.random((n, 3)) - 1)
        srf.tree_refit(tree, torch.tensor(new, device="cuda"))
        ref = ref.refitted(new[:, 0], new[:, 1], new[:, 2])
    lists = srf.make_lists(tree, p)
    want = ref.potential()
    phi = srf.short_range_potential(tree, lists, p).cpu().numpy()
    B = bound(ref, U32)
    worst = float((np.abs(phi - want) / np.maximum(B, 1e-300)).max())
    say(f"    waves {_waves(ref)}, largest |diff| / bound {worst:.3g}")
    assert np.all(np.abs(phi - want) <= B)
    phi = srf.short_range_potential(tree, lists, srf.Params.of(params, srf.FP64)).cpu().numpy()
    assert np.linalg.norm(phi - want) <= FP64_TOL * np.linalg.norm(want)
