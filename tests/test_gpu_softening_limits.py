"""Softening lengths at the ends of what is accepted (finite and > 0): a square
that overflows makes s^-1 = (r^2 + eps^2)^(-1/2) exactly 0, so that every output
is exactly 0; a square that underflows to 0 leaves s = r, and the potential of
two particles at one point is -infinity, that of the others their r-only sum."""
import numpy as np
import pytest
import torch

import paper_1211_4406_amd as srf

pytestmark = pytest.mark.gpu


def _tree(pos, eps, precision, **kw):
    n = len(pos)
    p = srf.Params(r_cut=0.2, eps=eps, theta=0.8, n_group=16, n_leaf=4, precision=precision, **kw)
    tree = srf.tree_build(torch.tensor(pos, device="cuda"), torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda"), p)
    return p, tree, srf.make_lists(tree, p)


@pytest.mark.parametrize("precision", [srf.FP32_REL, srf.FP64])
@pytest.mark.parametrize("eps", [1e160, 1e300])
def test_softening_whose_square_overflows(precision, eps):
    n = 700
    rng = np.random.default_rng(3100)
    print(f"[gpu] softening eps={eps} precision={precision}", flush=True)
    p, tree, lists = _tree(rng.random((n, 3)), eps, precision)
    w = torch.tensor(rng.standard_normal((n, 3)), device="cuda")
    gx, gm = srf.short_range_adjoint(tree, lists, p, w)
    for name, v in (("force", srf.short_range_force(tree, lists, p)), ("dL/dx", gx), ("dL/dm", gm),
                    ("potential", srf.short_range_potential(tree, lists, p)),
                    ("quadrupole", srf.short_range_force(tree, lists, p, quadrupole=True))):
        assert torch.equal(v, torch.zeros_like(v)), name


def test_softening_whose_square_underflows():
    """FP64; q(xi) / r summed in FP64 on the host: 64 bits' rounding of 300 terms of one sign, a few
    roundings each, stays below 300 * 8 * 2^-53 < 3e-13 of the sum."""
    n = 300
    rng = np.random.default_rng(3101)
    pos = rng.random((n, 3))
    pos[1] = pos[0]
    print("[gpu] softening eps=1e-170", flush=True)
    p, tree, lists = _tree(pos, 1e-170, srf.FP64)
    p0 = srf.Params(r_cut=p.r_cut, eps=p.eps, theta=0.0, n_group=p.n_group, n_leaf=p.n_leaf, precision=srf.FP64)
    phi = srf.short_range_potential(tree, srf.make_lists(tree, p0), p0).cpu().numpy()   # theta = 0: particles only
    assert phi[0] == -np.inf and phi[1] == -np.inf
    d = pos[:, None, :] - pos[None, :, :]
    r = np.sqrt(((d - np.rint(d)) ** 2).sum(axis=2))
    xi = 2.0 * r / p.r_cut
    q = np.where(xi <= 1,
                 1 - 52 / 35 * xi + 4 / 5 * xi ** 3 - 2 / 5 * xi ** 5 + xi ** 6 / 10 + 2 / 35 * xi ** 7 - 3 / 140 * xi ** 8,
                 np.where(xi < 2, (2 - xi) ** 6 * (xi * xi + 4 * xi + 2) / 140, 0.0))
    with np.errstate(divide="ignore", invalid="ignore"):
        pair = np.where(r > 0, q / r, 0.0)
    want = -pair.sum(axis=1) / n
    np.testing.assert_allclose(phi[2:], want[2:], rtol=3e-13, atol=1e-13 * np.abs(want).max())
