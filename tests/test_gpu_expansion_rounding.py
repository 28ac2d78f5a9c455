"""The kernels' own errors: the FMM of order p on the GPU against the same
truncated sums in extended precision, target by target, within the roundings of
the sums that enter each.  All orders, both tree forms, charges and dipoles; a
term of an expansion that is lost, or a child or box of a list, is many orders of
magnitude above that.  The highest order counts most for points at the corners of boxes of
shallow trees: left out, it makes there an error of two to ten times the bound at
order 31, and of hundreds at order 24."""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.fixture(scope="module")
def yk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1007_5335_amd.yk as yk
    yk.load_library()
    return yk


def _tree(yk, ctx, slot, adaptive):
    t = yk.yk_plan_tree_export(ctx, slot)   # (checked against oracle.tree elsewhere)
    if adaptive:
        t.update(yk.yk_plan_adaptive_export(ctx, slot))
    return t


def _corners(rng, xy, m):
    """The points moved to the corners of an m x m grid, to a thousandth of its spacing."""
    return np.clip((np.round(m * xy) + 0.002 * (rng.random(xy.shape) - 0.5)) / m, 0.0, 1.0 - 2.0 ** -40)


def _check(sums, got, perm, sample, roundings=8):
    """Per target: at most 8 (or `roundings`) roundings of the terms' absolute values (a sum of many terms of either sign rounds by
    about one rounding of its absolute sum; some 30 such stages, P2M, shifts at up to 11 levels each way, M2L, L2P and
    the near field, each of either sign: the root of their number, and a little) and 4 of a position (a centre's
    coordinate rounds twice, at both ends of a translation: the root of four, and the 1.7 sides^-1 by which that
    changes K_0 or K_1 at the closest points)."""
    worst = 0.0
    for j in sample:
        v, mag, pos = sums.at_sorted(int(j))
        tol = U * (roundings * mag + 4 * pos)
        worst = max(worst, float(abs(got[perm[j]] - v) / tol))
    print(f"  largest error: {worst:.1e} of the bound", flush=True)
    assert worst <= 1.0


# alpha against the box sides 2^-l: M2L by sibling groups at sides of at most 4 alpha
CHARGES = [
    dict(n=700, leaf=16, alpha=0.3),                          # every level by groups, 16 + 4 parents
    dict(n=20011, leaf=16, alpha=0.02),                       # two coarser levels, box by box
    dict(n=60013, leaf=16, alpha=0.0045),                     # more than 512 coarser boxes: dense tiles
    dict(n=9001, leaf=8, alpha=0.1, strip=True),              # a thin set: most groups incomplete
    dict(n=5003, leaf=16, alpha=0.1, p=24),
    dict(n=5003, leaf=16, alpha=0.1, p=28),
    # no groups; the shifts' other padded orders, by subtrees and level by level
    dict(n=700, leaf=16, alpha=0.3, p=8),
    dict(n=40009, leaf=16, alpha=0.2, p=12),
    dict(n=3001, leaf=8, alpha=0.2, p=16),
    dict(n=5003, leaf=16, alpha=0.1, p=20),
    dict(n=3001, leaf=8, alpha=0.2, p=16, cache=0),           # P2M and the near field uncached
    dict(n=5003, leaf=16, alpha=0.1, p=31, cache=0),
    dict(n=60013, leaf=4, alpha=0.1, p=8),                    # P2M in two halves of the orders
    dict(n=600, leaf=16, alpha=0.1, corners=8),
    dict(n=600, leaf=16, alpha=0.3, corners=8),
    dict(n=1200, leaf=16, alpha=0.03, corners=16),            # the coarsest level by box
    dict(n=1200, leaf=16, alpha=0.1, corners=16, p=28),
    dict(n=1200, leaf=16, alpha=0.1, corners=16, p=24, cache=0),
    dict(n=1200, leaf=16, alpha=0.1, corners=16, p=20),
]


@pytest.mark.parametrize("c", CHARGES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_charges_uniform(yk, c):
    import torch
    from oracle import expansions as E
    rng = np.random.default_rng(41)
    n, p = c["n"], c.get("p", 31)
    xy = rng.random((n, 2))
    if c.get("strip"):
        xy[:, 1] = 0.3 + 0.06 * xy[:, 1]
    if "corners" in c:
        xy = _corners(rng, xy, c["corners"])
    q = rng.standard_normal(n)
    print(f"rounding, charges: {c}", flush=True)
    kw = {} if "cache" not in c else dict(near_cache_mb=c["cache"])
    ctx = yk.yk_create(leaf_size=c["leaf"], p=p, tree=yk.YK_TREE_UNIFORM, **kw)
    try:
        out = torch.empty(n, dtype=torch.float64, device="cuda")
        yk.yk_volume_potential(ctx, dev(xy), dev(q), None, c["alpha"], out)
        t = _tree(yk, ctx, 2, False)
    finally:
        yk.yk_destroy(ctx)
    _check(E.Sums(t, c["alpha"], p, xy, q), host(out), t["perm"], rng.choice(n, 60, replace=False))


BOTH = [
    dict(n=900, nodes=64, leaf=4, alpha=0.5, p=8),
    dict(n=5003, nodes=257, leaf=16, alpha=0.05, p=12),
    dict(n=9001, nodes=1024, leaf=260, alpha=0.02, p=16),     # leaves of several wavefronts
    dict(n=20011, nodes=512, leaf=32, alpha=0.004, p=20),
    dict(n=20011, nodes=4096, leaf=16, alpha=0.01, p=24),
    dict(n=9001, nodes=333, leaf=100, alpha=0.1, p=28),
    dict(n=12007, nodes=1000, leaf=32, alpha=0.03, p=31),
    dict(n=60017, nodes=2048, leaf=4, alpha=0.02, p=8),       # more leaves than go by a wavefront each
    dict(n=60017, nodes=2048, leaf=4, alpha=0.02, p=31),
    dict(n=1500, nodes=100, leaf=16, alpha=0.1, p=31, corners=64),
    dict(n=1500, nodes=100, leaf=16, alpha=0.1, p=24, corners=64),
    # uniform trees: P2M of few leaves, and of many with dipoles in some
    dict(n=5003, nodes=257, leaf=16, alpha=0.05, p=12, tree=0),
    dict(n=5003, nodes=257, leaf=16, alpha=0.05, p=31, tree=0),
    dict(n=60017, nodes=9000, leaf=4, alpha=0.05, p=20, tree=0),
    dict(n=60017, nodes=300, leaf=4, alpha=0.05, p=31, tree=0),
    dict(n=1200, nodes=100, leaf=16, alpha=0.03, p=31, tree=0, corners=16),
    dict(n=1200, nodes=100, leaf=16, alpha=0.03, p=24, tree=0, corners=16),
]


@pytest.mark.parametrize("c", BOTH, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_charges_and_dipoles(yk, c):
    import torch
    from oracle import expansions as E
    rng = np.random.default_rng(43)
    n, nodes, alpha, p, tree = c["n"], c["nodes"], c["alpha"], c["p"], c.get("tree", 1)
    xy = rng.random((n, 2))
    if tree:
        half = n // 2   # graded towards a corner of the circle below
        xy[:half] = np.clip(0.7 + 0.3 * (rng.random((half, 2)) - 0.5) ** 3 * 8, 0, 1)
    if "corners" in c:
        xy = _corners(rng, xy, c["corners"])
    q = rng.standard_normal(n)
    th = 2 * np.pi * np.sort(rng.random(nodes) ** 2)
    nrm = np.stack([np.cos(th), np.sin(th)], 1)
    bxy, ones, d = 0.5 + 0.2 * nrm, np.ones(nodes), rng.standard_normal(nodes)
    print(f"rounding, charges and dipoles: {c}", flush=True)
    ctx = yk.yk_create(leaf_size=c["leaf"], p=p, tree=tree, direct=0)
    try:
        bd = yk.Boundary(bxy, nrm, ones, ones, [0, nodes])
        ov = torch.empty(n, dtype=torch.float64, device="cuda")
        ob = torch.empty(nodes, dtype=torch.float64, device="cuda")
        yk.yk_fmm_potential(ctx, dev(xy), dev(q), bd, dev(d), alpha, ov, ob)
        t = _tree(yk, ctx, 0, tree == 1)
    finally:
        yk.yk_destroy(ctx)
    print(f"  {len(t['leaf_range'])} leaves", flush=True)
    _check(E.Sums(t, alpha, p, xy, q, bxy, nrm, d), host(ov), t["perm"], rng.choice(n, 60, replace=False))


@pytest.mark.parametrize("ratio", [1.0, 2.0, 3.99])
def test_siblings_shares_stay_apart(yk, ratio):
    """Charges in one box of level 5 alone, box sides of `ratio` alpha there (groups serve sides up to four alpha):
    the targets that this box reaches by M2L at its own level, each relative to its own sum.  What a sibling's share
    leaves in it is at most exp(2.24 ratio) roundings of that (the centres' distances of the shares: 2 and 3 sqrt(2)
    sides), times 64: the products of 256 terms at M2L and
    at two shifts, without the allowance for their signs that _check makes."""
    import torch
    from oracle import expansions as E
    rng = np.random.default_rng(47)
    n, lev, p = 16384, 5, 31
    alpha = 2.0 ** -lev / ratio
    xy = rng.random((n, 2))
    xy[0], xy[1] = 0.0, 1.0 - 2.0 ** -40   # (the square is the unit one, to 1e-9)
    cell = np.floor(xy * 2 ** lev).astype(int)
    q = np.where((cell == 14).all(axis=1), 1.0, 0.0)
    print(f"siblings' shares: side {ratio} alpha", flush=True)
    ctx = yk.yk_create(leaf_size=32, p=p, tree=yk.YK_TREE_UNIFORM)
    try:
        out = torch.empty(n, dtype=torch.float64, device="cuda")
        yk.yk_volume_potential(ctx, dev(xy), dev(q), None, alpha, out)
        t = _tree(yk, ctx, 2, False)
    finally:
        yk.yk_destroy(ctx)
    assert t["leaf_level"] >= lev
    got = host(out)
    # V lists of the box's neighbours' parents' children: two or three boxes away
    far = np.abs(cell - 14).max(axis=1)
    parent = np.abs(cell // 2 - 7).max(axis=1)
    idx = np.flatnonzero((far >= 2) & (parent <= 1))
    idx = rng.choice(idx, min(150, len(idx)), replace=False)
    place = np.argsort(t["perm"][:n])
    sums = E.Sums(t, alpha, p, xy, q)
    err = []
    for i in idx:
        v, _, _ = sums.at_sorted(int(place[i]))
        err.append(float(abs(got[i] - v) / v))
    print(f"  largest error {max(err):.1e} of the target's own sum, median {np.median(err):.1e}", flush=True)
    assert max(err) <= 64 * U * np.exp(2.24 * ratio)


# leaves (4^level, all filled) on either side of the items that choose the kernel (4,608 for boxes of up to alpha,
# 12,288 for others); items of a few targets and of several wavefronts'
@pytest.mark.parametrize("n,leaf,level,ratio", [(300, 16, 3, 1.2), (900, 200, 2, 4.0), (40000, 16, 6, 0.9),
                                                (40000, 16, 6, 3.0), (200000, 16, 7, 0.9), (200000, 16, 7, 3.0),
                                                (200000, 16, 7, 12.0)])
def test_near_field_beyond_the_series(yk, n, leaf, level, ratio):
    """The near field evaluated on the fly at arguments beyond its series, coincident points among the pairs.  An
    argument of z rounds to z roundings of exp(-z), and the pairs reach z = 2 sqrt(2) ratio <= 34."""
    import torch
    from oracle import expansions as E
    rng = np.random.default_rng(53)
    alpha = 2.0 ** -level / ratio
    xy = rng.random((n, 2))
    xy[10:20] = xy[:10]
    nodes = 200
    th = 2 * np.pi * np.arange(nodes) / nodes
    nrm = np.stack([np.cos(th), np.sin(th)], 1)
    bxy, ones = 0.5 + 0.3 * nrm, np.ones(nodes)
    q, d = rng.standard_normal(n), rng.standard_normal(nodes)
    print(f"rounding, large arguments: {n} {leaf} {ratio}", flush=True)
    ctx = yk.yk_create(leaf_size=leaf, p=31, tree=yk.YK_TREE_UNIFORM, near_cache_mb=0, direct=0)
    try:
        bd = yk.Boundary(bxy, nrm, ones, ones, [0, nodes])
        ov = torch.empty(n, dtype=torch.float64, device="cuda")
        ob = torch.empty(nodes, dtype=torch.float64, device="cuda")
        yk.yk_fmm_potential(ctx, dev(xy), dev(q), bd, dev(d), alpha, ov, ob)
        t = _tree(yk, ctx, 0, False)
    finally:
        yk.yk_destroy(ctx)
    print(f"  level {t['leaf_level']}, {len(t['leaf_range'])} leaves", flush=True)
    assert t["leaf_level"] == level and (len(t["leaf_range"]) > 12288) == (n > 100000)
    place = np.argsort(t["perm"][:n])
    sample = np.concatenate([place[:20], rng.choice(n, 40, replace=False)])
    _check(E.Sums(t, alpha, 31, xy, q, bxy, nrm, d), host(ov), t["perm"], sample, roundings=8 + 34)
