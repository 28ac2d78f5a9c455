"""A pass over strengths that are not finite leaves nothing behind: the same
context, evaluated again on finite data, gives bit for bit what a fresh one
gives.  Every plan keeps its expansions between calls; the trees here have
several levels of M2L by sibling groups and of parent-child shifts, the dense
products by box beside them, and the padded orders whose expansions are cleared
before every pass."""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def yk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1007_5335_amd.yk as yk
    yk.load_library()
    return yk


def _points(n, clustered):
    rng = np.random.default_rng(5)
    xy = rng.random((n, 2))
    if clustered:
        xy[:n // 2] = np.clip(0.4 + 0.01 * rng.standard_normal((n // 2, 2)), 0, 1)
    return xy, rng.standard_normal(n), rng.standard_normal(n)


def _bad(q, value, at):
    b = q.copy()
    b[at] = value
    return b


def _check(yk, opts, call, good, bad):
    """call(ctx, data) -> outputs: fresh on good; then, elsewhere, bad and good again."""
    ref = None
    for seq in ([good], [bad, good], [bad, bad, good]):
        ctx = yk.yk_create(**opts)
        try:
            for data in seq:
                out = call(ctx, data)
        finally:
            yk.yk_destroy(ctx)
        assert np.all(np.isfinite(out))
        if ref is None:
            ref = out
        assert np.array_equal(ref, out)


TREES = [
    dict(n=20011, leaf=16, alpha=0.1),                            # every level by groups
    dict(n=20011, leaf=16, alpha=0.02),                           # coarser levels by box in the same launch
    dict(n=60013, leaf=16, alpha=0.0045),                         # coarser levels by the dense tiles
    dict(n=20011, leaf=16, alpha=0.1, p=24),
    dict(n=20011, leaf=16, alpha=0.1, p=16),                      # no groups
    dict(n=30011, leaf=32, alpha=0.03, clustered=True, tree=1),   # adaptive, with X lists
]


@pytest.mark.parametrize("value", [np.nan, np.inf, 1e308], ids=["nan", "inf", "overflow"])
@pytest.mark.parametrize("c", TREES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_charges_after_nonfinite_charges(yk, c, value):
    import torch
    n = c["n"]
    xy, q, q2 = _points(n, c.get("clustered"))
    dxy = dev(xy)
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    print(f"nonfinite charges: {c} {value}", flush=True)

    def call(ctx, data):
        yk.yk_volume_potential(ctx, dxy, dev(data), None, c["alpha"], out)
        return host(out)
    bad = np.full(n, value) if value == 1e308 else _bad(q2, value, n // 3)
    _check(yk, dict(leaf_size=c["leaf"], p=c.get("p", 31), tree=c.get("tree", 0)), call, q, bad)


@pytest.mark.parametrize("tree", [0, 1])
def test_charges_and_dipoles_after_nonfinite_ones(yk, tree):
    """One context, a pass over charges and dipoles: either of them not finite."""
    import torch
    n, nodes, alpha = 20011, 2048, 0.05
    xy, q, _ = _points(n, tree == 1)
    rng = np.random.default_rng(6)
    th = 2 * np.pi * np.arange(nodes) / nodes
    nrm = np.stack([np.cos(th), np.sin(th)], 1)
    ones = np.ones(nodes)
    bd = yk.Boundary(0.5 + 0.3 * nrm, nrm, 0.3 * ones, ones / 0.3, [0, nodes])
    d = rng.standard_normal(nodes)
    dxy = dev(xy)
    ov = torch.empty(n, dtype=torch.float64, device="cuda")
    ob = torch.empty(nodes, dtype=torch.float64, device="cuda")
    print(f"nonfinite dipoles: tree {tree}", flush=True)

    def call(ctx, data):
        yk.yk_fmm_potential(ctx, dxy, dev(data[0]), bd, dev(data[1]), alpha, ov, ob)
        return np.concatenate([host(ov), host(ob)])
    for bad in ((_bad(q, np.nan, 7), d), (q, _bad(d, np.nan, 1000))):
        _check(yk, dict(leaf_size=16, p=31, tree=tree), call, (q, d), bad)


def test_box_grid_after_nonfinite_cells(yk):
    import torch
    m = 256
    rng = np.random.default_rng(9)
    B = rng.standard_normal(m * m)
    V = torch.empty(m * m, dtype=torch.float64, device="cuda")
    grid = yk.make_grid(0.0, 0.0, 1.0 / m, m, m)
    print("nonfinite cells: grid", flush=True)

    def call(ctx, data):
        yk.yk_box_potential(ctx, grid, dev(data), 0.0316, V)
        return host(V)
    _check(yk, {}, call, B, _bad(B, np.nan, 12345))


def test_box_leaves_after_nonfinite_cells(yk):
    import torch
    # leaves of level 4 inside a ring of level 5 about them: 2:1 balanced
    lev, ix, iy = [], [], []
    for j in range(16):
        for i in range(16):
            if 4 <= i < 12 and 4 <= j < 12:
                for k in range(4):
                    lev.append(5), ix.append(2 * i + (k & 1)), iy.append(2 * j + (k >> 1))
            else:
                lev.append(4), ix.append(i), iy.append(j)
    leaves = [np.array(a, dtype=np.int32) for a in (lev, ix, iy)]
    n = 16 * len(lev)
    rng = np.random.default_rng(11)
    B = rng.standard_normal(n)
    V = torch.empty(n, dtype=torch.float64, device="cuda")
    print("nonfinite cells: leaves", flush=True)

    def call(ctx, data):
        yk.yk_box_potential_adaptive(ctx, (0.0, 0.0, 1.0), *leaves, dev(data), 0.0316, V)
        return host(V)
    _check(yk, {}, call, B, _bad(B, np.nan, n // 2))
