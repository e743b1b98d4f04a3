"""The work that users of the short-range TreePM step have it do, as timed cases.

A case is one call sequence of a user's program over the public entry points:

* ``force``: one PP cycle of a simulation: tree, lists, accelerations (``quadrupole`` and
  ``mac`` = 1 are the accuracy variants of the same cycle);
* ``grad``: one training step through ``short_range`` (forward, and the backward that
  rebuilds tree and lists and runs the adjoint), with the accelerations and both gradients;
* ``potential``: an energy diagnostic over the tree and lists of the force;
* ``pm``: one long-range (PM) evaluation on the tree of the last PP cycle;
* ``step``: one step of the multiple-stepsize integrator (one PM and two PP cycles).

The particle sets are those of the repository's workloads (uniform; uniform background plus
Plummer halos; Zel'dovich-displaced lattice), with every length in mean interparticle
spacings, so that one recipe serves every size: r_cut from 1.6 spacings (4096 particles at
r_cut = 0.1) to 7.5 (the paper's run), softening 0.005 to 0.03 spacings.

``exact`` evaluates the same tree approximation in plain torch, FP64 throughout.
"""
from __future__ import annotations

import math

import torch

import paper_1211_4406_amd as srf

DEFAULTS = dict(task="force", kind="clustered", n=0, rc=6.0, eps=0.0256, theta=0.5, n_group=64, n_leaf=16, mac=0,
                fp64=False, compensated=False, quadrupole=False, n_mesh=0)
HALO_FRACTION = 0.5      # share of the particles in halos
PER_HALO = 2048
HALO_RADII = (0.125, 1.25)   # Plummer scale radii, spacings, log-uniform
ZELDOVICH_RMS = 0.3      # rms displacement, spacings
DEVICE = "cuda"


def _case(name=None, **kw):
    c = dict(DEFAULTS, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest calls: 4096 uniform particles, where launches and the host count
        _case("force-uniform-4096", kind="uniform", n=4096, rc=1.6, eps=0.016),
        # a small gradient step (a fitting loop on a small box), odd size
        _case("grad-clustered-10007", task="grad", n=10007, rc=4.5),
        # ordinary simulation boxes: ragged, and the 2^21 clustered workload
        _case("force-clustered-131071", n=131071),
        _case("force-clustered-2097152", n=1 << 21),
        # the largest clustered set: the per-node share of a large run, short cutoff
        _case("force-clustered-13000000", n=13_000_000, rc=2.75, eps=0.0047),
        # training steps: the 2^20 clustered workload, and the 256^3 lattice of the benchmark
        _case("grad-clustered-1048576", task="grad", n=1 << 20, rc=4.75, eps=0.02),
        _case("grad-zeldovich-16777216", task="grad", kind="zeldovich", n=256 ** 3, eps=0.0128),
        # all-FP64 gradients: reference trajectories and gradient checks
        _case("grad-fp64-clustered-200003", task="grad", n=200_003, fp64=True),
        # accuracy variants: quadrupole cells with the centre-of-mass criterion
        _case("quadrupole-com-clustered-524287", n=524_287, mac=1, quadrupole=True),
        # energy diagnostics over the lists in hand
        _case("potential-zeldovich-2097152", task="potential", kind="zeldovich", n=128 ** 3, eps=0.0128),
        # the long-range half on the mesh of the paper's ratio (N_PM = N / 8)
        _case("pm-zeldovich-16777216-mesh-128", task="pm", kind="zeldovich", n=256 ** 3, n_mesh=128),
        # one whole step of the integrator
        _case("step-zeldovich-2097152-mesh-64", task="step", kind="zeldovich", n=128 ** 3, eps=0.0128, n_mesh=64),
    ]


def draw(rng):
    task = rng.choice(["force", "force", "force", "grad", "grad", "potential", "pm", "step"])
    kind = rng.choice(["uniform", "clustered", "clustered", "zeldovich"])
    fp64 = task in ("force", "grad", "potential") and rng.random() < 0.2
    hi = 17 if fp64 else (20 if task in ("grad", "step") else 21)
    n = int(2.0 ** rng.uniform(10, hi))
    if kind == "zeldovich":
        n = round(n ** (1.0 / 3.0)) ** 3
    spacing = n ** (-1.0 / 3.0)
    rc = min(rng.uniform(1.6, 7.5), 0.24 / spacing)
    theta = rng.choice([0.3, 0.5, 0.5, 0.5, 0.7]) if n <= 1 << 19 else rng.choice([0.5, 0.6, 0.7])
    n_group, n_leaf = rng.choice([(64, 16), (64, 16), (64, 16), (64, 8), (32, 8)])
    n_mesh = 0
    if task in ("pm", "step"):   # about N / 8 mesh points, a power of two per axis
        n_mesh = min(256, max(16, 2 ** round(math.log2(0.5 / spacing) + rng.choice([0, 0, 1]))))
    return _case(task=task, kind=kind, n=n, rc=rc, eps=rng.uniform(0.005, 0.03), theta=theta, n_group=n_group,
                 n_leaf=n_leaf, mac=int(rng.random() < 0.2), fp64=fp64,
                 compensated=task == "force" and not fp64 and rng.random() < 0.15,
                 quadrupole=task == "force" and rng.random() < 0.2, n_mesh=n_mesh)


# ------------------------------------------------------------------ inputs
def _params(case):
    s = case["n"] ** (-1.0 / 3.0)
    return srf.Params(G=1.0, r_cut=case["rc"] * s, eps=case["eps"] * s, theta=case["theta"], n_group=case["n_group"],
                      n_leaf=case["n_leaf"], precision=srf.FP64 if case["fp64"] else srf.FP32_REL,
                      compensated=int(case["compensated"]), mac=case["mac"])


def _zeldovich(grid, gen):
    """Lattice and displacement [N,3] (lattice spacings) of a Gaussian field with P(k) ~ k^-2."""
    noise = torch.randn((grid,) * 3, dtype=torch.float64, device=DEVICE, generator=gen)
    nk = torch.fft.rfftn(noise)
    kf = torch.fft.fftfreq(grid, 1.0 / grid, dtype=torch.float64, device=DEVICE)
    kr = torch.fft.rfftfreq(grid, 1.0 / grid, dtype=torch.float64, device=DEVICE)
    ks = (kf[:, None, None], kf[None, :, None], kr[None, None, :])
    k2 = ks[0] ** 2 + ks[1] ** 2 + ks[2] ** 2
    k2[0, 0, 0] = 1.0
    nk = nk / k2 ** 1.5
    nk[0, 0, 0] = 0.0
    for a in range(3):
        nk = nk * (ks[a].abs() * 2 != grid)
    psi = torch.stack([torch.fft.irfftn(1j * k * nk, s=(grid,) * 3).reshape(-1) for k in ks], dim=1)
    psi *= ZELDOVICH_RMS / (psi ** 2).sum(dim=1).mean().sqrt()
    idx = torch.arange(grid, dtype=torch.float64, device=DEVICE) + 0.5
    q = torch.stack(torch.meshgrid(idx, idx, idx, indexing="ij"), dim=-1).reshape(-1, 3)
    return q, psi


def _positions(case, gen):
    """Positions [N,3] in [0,1) and, for the lattice, the displacement (box units)."""
    n, kind = case["n"], case["kind"]
    spacing = n ** (-1.0 / 3.0)
    rand = lambda *s: torch.rand(s, dtype=torch.float64, device=DEVICE, generator=gen)  # noqa: E731
    if kind == "zeldovich":
        grid = round(n ** (1.0 / 3.0))
        q, psi = _zeldovich(grid, gen)
        return torch.remainder((q + psi) / grid, 1.0), psi / grid
    if kind == "uniform":
        return rand(n, 3), None
    nh = max(1, round(n * HALO_FRACTION / PER_HALO))
    in_halos = int(n * HALO_FRACTION)
    centres = rand(nh, 3)
    a = spacing * torch.exp(math.log(HALO_RADII[0]) + rand(nh) * math.log(HALO_RADII[1] / HALO_RADII[0]))
    h = torch.arange(in_halos, device=DEVICE) * nh // max(in_halos, 1)
    inside = (1.0 + (a[h] / 0.5) ** 2) ** -1.5       # mass within r = 1/2, where the spheres end
    u = (1.0 - rand(in_halos)) * inside
    r = a[h] / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
    d = torch.randn((in_halos, 3), dtype=torch.float64, device=DEVICE, generator=gen)
    d /= d.norm(dim=1, keepdim=True)
    halos = torch.remainder(centres[h] + r[:, None] * d, 1.0)
    return torch.cat([rand(n - in_halos, 3), halos]), None


def _inputs(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    x, psi = _positions(case, gen)
    n = case["n"]
    m = torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEVICE)
    w = torch.randn((n, 3), dtype=torch.float32, device=DEVICE, generator=gen).double() if case["task"] == "grad" else None
    return x, m, w, psi


def prepare(case, seed):
    x, m, w, psi = _inputs(case, seed)
    p = _params(case)
    s = dict(case=case, x=x, m=m, w=w, p=p)
    if case["task"] == "grad":
        x.requires_grad_(True)
        m.requires_grad_(True)
    elif case["task"] in ("potential", "pm"):
        s["tree"] = srf.tree_build(x, m, p)
        if case["task"] == "potential":
            s["lists"] = srf.make_lists(s["tree"], p)
    elif case["task"] == "step":
        # a simulation under way: the growing mode (or small random velocities), one step taken
        s["v"] = 25.0 * psi if psi is not None else 10.0 * case["n"] ** (-1.0 / 3.0) * (x - 0.5)
        s["dt"] = 2e-4
        s["integ"] = srf.TreePMIntegrator(p, case["n_mesh"])
        s["integ"].step(x, s["v"], m, s["dt"])
    return s


def run(s):
    task, x, m, p = s["case"]["task"], s["x"], s["m"], s["p"]
    if task == "grad":
        a = srf.short_range(x, m, p)
        gx, gm = torch.autograd.grad(a, (x, m), s["w"])
        return {"a": a, "gx": gx, "gm": gm}
    if task == "potential":
        return {"phi": srf.short_range_potential(s["tree"], s["lists"], p)}
    if task == "pm":
        return {"a": srf.pm_force(s["tree"], p.G, p.r_cut, s["case"]["n_mesh"])}
    if task == "step":
        s["integ"].step(x, s["v"], m, s["dt"])
        return {"x": x, "v": s["v"]}
    tree = srf.tree_build(x, m, p)
    lists = srf.make_lists(tree, p)
    return {"a": srf.short_range_force(tree, lists, p, quadrupole=s["case"]["quadrupole"])}


def work(case):
    """Inputs read once, outputs written once; 51 flops per source of a particle (the count of the
    paper's force loop), 1.5 times that for the adjoint, over the sources a uniform density gives
    it: the particles of unaccepted leaves (nearer than a leaf's side over theta) and one cell per
    half-full leaf between there and r_cut."""
    n, half = case["n"], case["n_leaf"] / 2.0
    ball = 4.0 / 3.0 * math.pi
    near = ball * min(case["rc"], half ** (1.0 / 3.0) / case["theta"]) ** 3
    cells = max(0.0, ball * case["rc"] ** 3 - near) / half
    pairs = n * (near + cells)
    mesh = case["n_mesh"] ** 3
    pm = 2 * 27 * 8 * n + 2 * 5 * mesh * math.log2(max(mesh, 2)) + 33 * mesh
    task = case["task"]
    if task == "grad":   # x, m, w -> a, dL/dx, dL/dm
        return {"bytes": 8.0 * n * 14, "flops": 2.5 * 51 * pairs}
    if task == "potential":
        return {"bytes": 8.0 * n * 5, "flops": 40 * pairs}
    if task == "pm":
        return {"bytes": 8.0 * n * 7, "flops": float(pm)}
    if task == "step":   # x, v, m and both accelerations in, x, v and both accelerations out
        return {"bytes": 8.0 * n * 25, "flops": 2 * 51 * pairs + pm}
    return {"bytes": 8.0 * n * 7, "flops": 51 * pairs + (80 * n * cells if case["quadrupole"] else 0.0)}


# ------------------------------------------------- the same in plain torch
MAX_LEVEL = 21
PAIR_CHUNK = 1 << 24


def _spread(v):
    for shift, mask in ((32, 0x1F00000000FFFF), (16, 0x1F0000FF0000FF), (8, 0x100F00F00F00F00F),
                        (4, 0x10C30C30C30C30C3), (2, 0x1249249249249249)):
        v = (v | (v << shift)) & mask
    return v


def _image(d):
    return d - torch.round(d)


def _tree(x, case):
    """Cells, groups and the sorted order of the octree over wrapped positions x [N,3]."""
    u = x - torch.floor(x)
    u = torch.where(u == 1.0, torch.zeros_like(u), u)
    k = torch.clamp((u * 2.0 ** MAX_LEVEL).long(), max=2 ** MAX_LEVEL - 1)
    key = (_spread(k[:, 0]) << 2) | (_spread(k[:, 1]) << 1) | _spread(k[:, 2])
    key, order = torch.sort(key, stable=True)
    n, dev, n_group, n_leaf = x.shape[0], x.device, case["n_group"], case["n_leaf"]
    one = lambda v: torch.tensor([v], device=dev)  # noqa: E731
    first, count, level, ijk, parent = [one(0)], [one(n)], [one(0)], [torch.zeros(1, 3, device=dev).long()], [one(-1)]
    cell_of = torch.zeros(n, dtype=torch.long, device=dev)   # the deepest cell of each particle so far
    inside, total = torch.arange(n, device=dev), 1
    split = [one(True)]
    g_first, g_count = [], []
    for lv in range(1, MAX_LEVEL + 1):
        if inside.numel() == 0:
            break
        pre = key[inside] >> (3 * (MAX_LEVEL - lv))
        _, inv, cnt = torch.unique_consecutive(pre, return_inverse=True, return_counts=True)
        start = torch.cumsum(cnt, 0) - cnt
        f = inside[start]
        par = cell_of[f]
        g = torch.zeros((cnt.numel(), 3), dtype=torch.long, device=dev)
        for b in range(lv):
            for ax in range(3):
                g[:, ax] |= ((pre[start] >> (3 * b + 2 - ax)) & 1) << b
        first.append(f), count.append(cnt), level.append(torch.full_like(f, lv)), ijk.append(g), parent.append(par)
        sp = (cnt > n_leaf) & (lv < MAX_LEVEL)
        split.append(sp)
        cell_of[inside] = total + inv
        _groups(lv, f, cnt, par, torch.cat(count)[par], n_group, g_first, g_count)
        total += cnt.numel()
        inside = inside[sp[inv]]
    gf, gc = torch.cat(g_first), torch.cat(g_count)
    gf, o = torch.sort(gf)
    cat = torch.cat
    return dict(order=order, u=u[order], first=cat(first), count=cat(count), level=cat(level), ijk=cat(ijk),
                parent=cat(parent), leaf=~cat(split), leaf_of=cell_of, nc=total, gf=gf, gc=gc[o])


def _groups(lv, first, count, par, pcount, n_group, g_first, g_count):
    """Groups among one level's cells: candidates (at most n_group particles, under the root or a
    cell of more than n_group) merged greedily with the candidates before them under one parent
    (not under the root); level-21 cells of more than n_group in chunks."""
    cand = (count <= n_group) & ((pcount > n_group) | (lv == 1))
    if lv == 1:
        g_first.append(first[cand]), g_count.append(count[cand])
    elif cand.any():
        idx = torch.arange(first.numel(), device=first.device)
        new_par = torch.ones_like(cand)
        new_par[1:] = par[1:] != par[:-1]
        rank = idx - torch.cummax(torch.where(new_par, idx, 0), 0).values   # place among the siblings
        run, opened, start = torch.zeros_like(count), torch.zeros_like(cand), cand.clone()
        for r in range(8):   # the run that is open after each sibling
            at = idx[rank == r]
            prev_run = run[at - 1] if r else torch.zeros_like(at)
            prev_open = opened[at - 1] if r else torch.zeros_like(at).bool()
            joins = cand[at] & prev_open & (prev_run + count[at] <= n_group)
            start[at] = cand[at] & ~joins
            run[at] = torch.where(joins, prev_run + count[at], count[at])
            opened[at] = cand[at]
        number = torch.cumsum(start, 0) - 1
        g_first.append(first[start])
        g_count.append(torch.zeros_like(g_first[-1]).index_add_(0, number[cand], count[cand]))
    if lv == MAX_LEVEL:
        for f, c in zip(first[count > n_group].tolist(), count[count > n_group].tolist()):
            at = torch.arange(f, f + c, n_group, device=first.device)
            g_first.append(at), g_count.append(torch.clamp(f + c - at, max=n_group))


def _upward(t, own):
    """Sums of own [cells, ...] over each cell and its descendants (children come after parents,
    level by level)."""
    for lv in range(int(t["level"][-1]), 0, -1):
        at = torch.nonzero(t["level"] == lv)[:, 0]
        own = own.index_add(0, t["parent"][at], own[at])
    return own


def _moments(t, u, m):
    """Mass and centre of mass of every cell, differentiable in u [N,3] and m [N] (sorted)."""
    own = torch.zeros((t["nc"], 4), dtype=u.dtype, device=u.device)
    s = _upward(t, own.index_add(0, t["leaf_of"], torch.cat([u * m[:, None], m[:, None]], dim=1)))
    return s[:, 3], s[:, :3] / s[:, 3:]


def _second_moments(t, u, m, M, X):
    """sum_k m_k (x_k - X)(x_k - X)^T of every cell about its centre of mass: a leaf's from its
    particles, an inner cell's from its children's by the parallel-axis theorem."""
    outer = lambda w, d: w[:, None, None] * d[:, :, None] * d[:, None, :]  # noqa: E731
    S = torch.zeros((t["nc"], 3, 3), dtype=u.dtype, device=u.device)
    S.index_add_(0, t["leaf_of"], outer(m, u - X[t["leaf_of"]]))
    for lv in range(int(t["level"][-1]), 0, -1):
        at = torch.nonzero(t["level"] == lv)[:, 0]
        up = t["parent"][at]
        S.index_add_(0, up, S[at] + outer(M[at], X[at] - X[up]))
    return S


def _lists(t, X, p):
    """(group, source) pairs: sources < N are sorted particles, N + c cells."""
    n, dev = t["u"].shape[0], X.device
    member = torch.repeat_interleave(torch.arange(t["gf"].numel(), device=dev), t["gc"])
    lo = torch.full((t["gf"].numel(), 3), math.inf, dtype=torch.float64, device=dev)
    hi = -lo
    at = member[:, None].expand(-1, 3)
    lo = lo.scatter_reduce(0, at, t["u"], "amin")
    hi = hi.scatter_reduce(0, at, t["u"], "amax")
    cg, hg = (lo + hi) * 0.5, (hi - lo) * 0.5
    side = torch.pow(2.0, -t["level"].double())
    centre = (t["ijk"].double() + 0.5) * side[:, None]
    kids = torch.argsort(t["parent"], stable=True)[1:]        # the root comes first
    nkids = torch.bincount(t["parent"][1:], minlength=t["nc"])
    kid0 = torch.cumsum(nkids, 0) - nkids

    def gap2(c, h, g):
        d = (c - cg[g]).abs()
        d = torch.minimum(d, 1.0 - d)
        e = torch.clamp(d - (h + hg[g]), min=0.0) ** 2
        return (e[:, 0] + e[:, 1]) + e[:, 2]

    def spread_over(lengths):
        rep = torch.repeat_interleave(torch.arange(lengths.numel(), device=dev), lengths)
        return rep, torch.arange(rep.numel(), device=dev) - (torch.cumsum(lengths, 0) - lengths)[rep]

    g = torch.arange(t["gf"].numel(), device=dev)
    c = torch.zeros_like(g)
    out_g, out_s = [], []
    while g.numel():
        keep = gap2(centre[c], (side[c] * 0.5)[:, None], g) < p.r_cut * p.r_cut
        g, c = g[keep], c[keep]
        d2 = gap2(X[c] if p.mac else centre[c], 0.0, g)
        acc = side[c] * side[c] < (p.theta * p.theta) * d2
        out_g.append(g[acc]), out_s.append(n + c[acc])
        leaf = ~acc & t["leaf"][c]
        rep, k = spread_over(t["count"][c[leaf]])
        out_g.append(g[leaf][rep]), out_s.append(t["first"][c[leaf]][rep] + k)
        opened = ~acc & ~t["leaf"][c]
        rep, k = spread_over(nkids[c[opened]])
        g, c = g[opened][rep], kids[kid0[c[opened]][rep] + k]
    return torch.cat(out_g), torch.cat(out_s)


def _cutoff(xi):
    inner = 1 + xi ** 3 * (-8 / 5 + xi ** 2 * (8 / 5 + xi * (-1 / 2 + xi * (-12 / 35 + 3 / 20 * xi))))
    outer = (2 - xi) ** 5 * (7 * xi ** 3 + 22 * xi ** 2 + 10 * xi + 4) / 140
    return torch.where(xi <= 1, inner, torch.where(xi < 2, outer, 0.0))


def _pairs(t, eg, es):
    """The pairs of the lists in chunks of whole targets: the targets' range, their numbers of
    sources, and the pairs (target, source), each target's consecutive."""
    ng, n = t["gf"].numel(), t["u"].shape[0]
    es = es[torch.argsort(eg, stable=True)]
    length = torch.bincount(eg, minlength=ng)
    e0 = torch.cumsum(length, 0) - length
    member = torch.repeat_interleave(torch.arange(ng, device=eg.device), t["gc"])
    per = length[member]
    ends = torch.cumsum(per, 0)
    i0 = 0
    while i0 < n:
        done = int(ends[i0 - 1]) if i0 else 0
        i1 = max(i0 + 1, int(torch.searchsorted(ends, done + PAIR_CHUNK)))
        i = torch.repeat_interleave(torch.arange(i0, i1, device=eg.device), per[i0:i1])
        k = torch.arange(i.numel(), device=eg.device) - (ends - per)[i] + done
        yield i0, i1, per[i0:i1], i, es[e0[member[i]] + k]
        i0 = i1


def _sums(v, per):
    """Sums of v [pairs, ...] over each target's pairs."""
    return torch.segment_reduce(v, "sum", lengths=per, axis=0, unsafe=True)


def _pair_accel(p, ui, sj, mj):
    d = sj - ui
    d = d - torch.round(d.detach())
    r2 = (d * d).sum(dim=1)
    r = torch.sqrt(torch.clamp(r2, min=1e-300))
    s2 = r2 + p.eps * p.eps
    return d * (mj * _cutoff(2 * r / p.r_cut) / (s2 * torch.sqrt(s2)))[:, None]


def _pair_potential(p, ui, sj, mj):
    r2 = (_image(sj - ui) ** 2).sum(dim=1)
    xi = 2 * torch.sqrt(r2) / p.r_cut
    q = torch.where(
        xi <= 1,
        1 + xi * (-52 / 35 + xi ** 2 * (4 / 5 + xi ** 2 * (-2 / 5 + xi * (1 / 10 + xi * (2 / 35 - 3 / 140 * xi))))),
        torch.where(xi < 2, (2 - xi) ** 6 * (xi * xi + 4 * xi + 2) / 140, 0.0))
    return -mj * q / torch.sqrt(r2 + p.eps * p.eps)


def _pair_quadrupole(p, ui, xc, S):
    """1/2 S_ab d_a d_b F(D) for second moments S [.,3,3], F the pair force of a unit source."""
    D = _image(xc - ui)
    D = torch.where(((D * D).sum(dim=1) < p.r_cut * p.r_cut)[:, None], D, 0.5 * p.r_cut * 3 ** 0.5)   # xi = 3: no term
    r2 = (D * D).sum(dim=1)
    r, k = torch.sqrt(r2), 2.0 / p.r_cut
    xi, s2 = k * r, r2 + p.eps * p.eps
    s = torch.sqrt(s2)
    g = _cutoff(xi)
    P = 2 * xi * xi + 4 * xi - 1
    t = 2 - xi
    g1 = torch.where(xi <= 1, xi ** 2 * (-24 / 5 + 8 * xi ** 2 - 3 * xi ** 3 - 12 / 5 * xi ** 4 + 6 / 5 * xi ** 5),
                     -xi * t ** 4 * P / 5)
    g2 = torch.where(xi <= 1, xi * (-48 / 5 + 32 * xi ** 2 - 15 * xi ** 3 - 72 / 5 * xi ** 4 + 42 / 5 * xi ** 5),
                     -t ** 3 * (t * P - 4 * xi * P + xi * t * (4 * xi + 4)) / 5)
    psi = k * g1 / (r * s ** 3) - 3 * g / s ** 5
    chi = k * k * g2 / (r2 * s ** 3) - k * g1 / (r2 * r * s ** 3) - 6 * k * g1 / (r * s ** 5) + 15 * g / s ** 7
    SD = (S @ D[:, :, None])[:, :, 0]
    c = 0.5 * psi * (S[:, 0, 0] + S[:, 1, 1] + S[:, 2, 2]) + 0.5 * chi * (D * SD).sum(dim=1)
    return torch.where(xi[:, None] < 2, psi[:, None] * SD + c[:, None] * D, 0.0)


def _exact_pp(case, x, m, w):
    p, n = _params(case), case["n"]
    t = _tree(x, case)
    u, ms = t["u"], m[t["order"]]
    back = torch.empty_like(t["order"])
    back[t["order"]] = torch.arange(n, device=x.device)
    M, X = _moments(t, u, ms)
    eg, es = _lists(t, X, p)
    S, mu = torch.cat([u, X]), torch.cat([ms, M])
    if case["task"] == "potential":
        phi = torch.zeros(n, dtype=torch.float64, device=x.device)
        for i0, i1, per, i, j in _pairs(t, eg, es):
            phi[i0:i1] = _sums(_pair_potential(p, u[i], S[j], torch.where(i == j, 0.0, mu[j])), per)
        return {"phi": p.G * phi[back]}
    a = torch.zeros((n, 3), dtype=torch.float64, device=x.device)
    second = None
    if case["quadrupole"]:
        second = _second_moments(t, u, ms, M, X)
    gu, gS, gmu = torch.zeros_like(u), torch.zeros_like(S), torch.zeros_like(mu)
    ws = w[t["order"]] if w is not None else None
    for i0, i1, per, i, j in _pairs(t, eg, es):
        ui, sj, mj = u[i], S[j], torch.where(i == j, 0.0, mu[j])   # the target itself is left out
        if w is None:
            f = _pair_accel(p, ui, sj, mj)
        else:
            for v in (ui, sj, mj):
                v.requires_grad_(True)
            f = _pair_accel(p, ui, sj, mj)
            gi, gj, gm = torch.autograd.grad(f, (ui, sj, mj), ws[i])
            gu[i0:i1] = _sums(gi, per)
            gS.index_add_(0, j, gj)
            gmu.index_add_(0, j, gm)
            f = f.detach()
        if second is not None:
            cell = torch.nonzero(j >= n)[:, 0]
            c = j[cell] - n
            f.index_add_(0, cell, _pair_quadrupole(p, u[i[cell]], X[c], second[c]))
        a[i0:i1] = _sums(f, per)
    out = {"a": p.G * a[back]}
    if w is not None:   # the cells' gradients through their moments
        uu, mm = u.clone().requires_grad_(True), ms.clone().requires_grad_(True)
        M, X = _moments(t, uu, mm)
        cu, cm = torch.autograd.grad((X, M), (uu, mm), (gS[n:], gmu[n:]))
        out["gx"] = p.G * (gu + gS[:n] + cu)[back]
        out["gm"] = p.G * (gmu[:n] + cm)[back]
    return out


def _tsc(x, n):
    c = torch.floor(x * n + 0.5)
    d = x * n - c
    w = torch.stack([0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2], dim=-1)      # [N,3 axes,3]
    i = (c.long()[..., None] + torch.arange(-1, 2, device=x.device)) % n
    for a in range(3):
        for b in range(3):
            for e in range(3):
                yield (i[:, 0, a] * n + i[:, 1, b]) * n + i[:, 2, e], w[:, 0, a] * w[:, 1, b] * w[:, 2, e]


def _exact_pm(case, x, m):
    p, n = _params(case), case["n_mesh"]
    rho = torch.zeros(n ** 3, dtype=torch.float64, device=x.device)
    for i, w in _tsc(x, n):
        rho.index_add_(0, i, m * w * float(n) ** 3)
    k1 = 2 * math.pi * torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=x.device)
    k2 = k1[:, None, None] ** 2 + k1[None, :, None] ** 2 + k1[None, None, :] ** 2
    sinc = torch.sinc(k1 / (2 * math.pi * n)) ** 3
    window = sinc[:, None, None] * sinc[None, :, None] * sinc[None, None, :]
    s = torch.sqrt(k2) * p.r_cut / 2
    v = torch.clamp(s, max=0.5) ** 2
    series = 1 + v * (-1 / 15 + v * (1 / 560 + v * (-1 / 37800 + v / 3991680)))
    b = torch.clamp(s, min=0.5)
    shape = torch.where(s < 0.5, series, 12 * (2 - 2 * torch.cos(b) - b * torch.sin(b)) / b ** 4)
    k2[0, 0, 0] = 1.0
    green = -4 * math.pi * p.G * shape ** 2 / (k2 * window ** 2)
    green[0, 0, 0] = 0.0
    phi = torch.fft.ifftn(torch.fft.fftn(rho.reshape(n, n, n)) * green).real
    field = torch.stack([(-2 / 3 * (phi.roll(-1, a) - phi.roll(1, a)) + (phi.roll(-2, a) - phi.roll(2, a)) / 12) * n
                         for a in range(3)], dim=-1).reshape(-1, 3)
    out = torch.zeros((x.shape[0], 3), dtype=torch.float64, device=x.device)
    for i, w in _tsc(x, n):
        out += w[:, None] * field[i]
    return {"a": out}


def exact(case, seed):
    if case["task"] == "step" or (case["task"] != "pm" and case["n"] > 1 << 21):
        return None      # a step follows many others; the largest sets have too many pairs
    x, m, w, _ = _inputs(case, seed)
    return _exact_pm(case, x, m) if case["task"] == "pm" else _exact_pp(case, x, m, w)
