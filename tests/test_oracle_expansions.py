"""The truncated FMM sums in extended precision (oracle/expansions.py): their
Bessel functions against scipy, and at order 31 against direct sums, within the
truncation, on uniform and adaptive trees with charges and dipoles."""
import numpy as np
import pytest

import oracle
from oracle import expansions as E
from oracle import tree as T


def test_bessel_functions():
    sp = pytest.importorskip("scipy.special")
    x = np.array([1e-6, 1e-3, 0.1, 0.7, 2.0, 9.5, 40.0])
    n = np.arange(33)[:, None]
    with np.errstate(over="ignore"):
        I, K = sp.iv(n, x), sp.kv(n, x)
    ok = np.isfinite(K) & (I > 1e-290)
    assert np.max(np.abs(E.bessel_i(x, 32).astype(float)[ok] / I[ok] - 1)) < 1e-13
    assert np.max(np.abs(E.bessel_k(x, 32).astype(float)[ok] / K[ok] - 1)) < 1e-13


@pytest.mark.parametrize("adaptive", [False, True])
@pytest.mark.parametrize("alpha", [0.4, 0.03])
def test_truncated_sums_approach_direct_sums(adaptive, alpha):
    rng = np.random.default_rng(2)
    n, nodes = 1500, 200
    xy = rng.random((n, 2))
    if adaptive:
        xy[:1000] = 0.4 + 0.01 * rng.standard_normal((1000, 2))
    th = 2 * np.pi * np.arange(nodes) / nodes
    nrm = np.stack([np.cos(th), np.sin(th)], 1)
    bxy = 0.5 + 0.3 * nrm
    q, d = rng.standard_normal(n), rng.standard_normal(nodes)
    square = (0.0, 0.0, 1.0)
    build = T.build_adaptive if adaptive else T.build
    t = build([xy, bxy], square, 8, alpha)
    t["square"] = square
    err = {}
    for p in (12, 31):
        s = E.Sums(t, alpha, p, xy, q, bxy, nrm, d)
        j = rng.choice(n, 25, replace=False)
        got = np.array([s.at_sorted(int(k)) for k in j])
        x = s.xy[j].astype(float)
        ref = oracle.volume_sum(xy, q, alpha, tgt_xy=x) + oracle.dl_sum(bxy, nrm, d, alpha, x)
        assert np.all(np.abs(ref) <= got[:, 1] * (1 + 1e-10))
        err[p] = np.max(np.abs(got[:, 0] - ref) / got[:, 1])
    # each order takes at least a factor 0.547 off the terms left out
    print(adaptive, alpha, err)
    assert err[31] < 1e-9 and 1e-14 < err[12] < (12 + 2) * 0.547 ** 12 / 0.453 ** 2
