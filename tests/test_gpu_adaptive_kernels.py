"""The adaptive tree's kernels on the GPU (P2M by wavefront and by quads, P2L,
M2P, the near field by kinds of series) for charges and dipoles, against the
oracle's direct sums at sampled points: leaves of one point and of more than a
wavefront, few leaves and more than the quads' threshold, scales at which every
kind of near-field series occurs."""
import numpy as np
import pytest

import oracle
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


CASES = [
    dict(n=900, nodes=64, leaf=4, alpha=0.5, p=8),
    dict(n=5003, nodes=257, leaf=16, alpha=0.05, p=12),
    dict(n=9001, nodes=1024, leaf=260, alpha=0.02, p=16),      # leaves of several wavefronts
    dict(n=20011, nodes=512, leaf=32, alpha=0.004, p=20),
    dict(n=20011, nodes=4096, leaf=16, alpha=0.01, p=24),
    dict(n=9001, nodes=333, leaf=100, alpha=0.1, p=28),
    dict(n=12007, nodes=1000, leaf=32, alpha=0.03, p=31),
    dict(n=90017, nodes=2048, leaf=16, alpha=0.02, p=31),      # more than 8,192 leaves
    dict(n=90017, nodes=2048, leaf=16, alpha=0.003, p=8),
    # uniform trees of more than 8,192 leaves: the leaves with dipoles by
    # themselves, several points per lane or a few
    dict(n=90017, nodes=9000, leaf=8, alpha=0.05, p=31, tree=0),
    dict(n=90017, nodes=300, leaf=8, alpha=0.05, p=12, tree=0),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_adaptive_kernels_match_direct_sums(yk, c):
    import torch
    rng = np.random.default_rng(23)
    n, nodes, alpha, p = c["n"], c["nodes"], c["alpha"], c["p"]
    # half the points graded towards a corner of the circle below
    xy = rng.random((n, 2))
    half = n // 2
    xy[:half] = np.clip(0.7 + 0.3 * (rng.random((half, 2)) - 0.5) ** 3 * 8, 0, 1)
    q = rng.standard_normal(n)
    th = 2 * np.pi * np.sort(rng.random(nodes) ** 2)   # dense near angle 0
    nrm = np.stack([np.cos(th), np.sin(th)], 1)
    bxy, ones = 0.5 + 0.2 * nrm, np.ones(nodes)
    d = rng.standard_normal(nodes)
    print(f"adaptive kernels: {c}", flush=True)
    ctx = yk.yk_create(leaf_size=c["leaf"], p=p, tree=c.get("tree", yk.YK_TREE_ADAPTIVE), direct=0)
    try:
        bd = yk.Boundary(bxy, nrm, ones, ones, [0, nodes])
        ov = torch.empty(n, dtype=torch.float64, device="cuda")
        ob = torch.empty(nodes, dtype=torch.float64, device="cuda")
        yk.yk_fmm_potential(ctx, dev(xy), dev(q), bd, dev(d), alpha, ov, ob)
        got = host(ov)
        info = yk.yk_plan_info_get(ctx, 0)
    finally:
        yk.yk_destroy(ctx)
    print(f"  {info.n_leaves} leaves", flush=True)
    assert (info.n_leaves > 8192) == (n > 90000)
    idx = rng.choice(n, size=150, replace=False)
    ref = oracle.volume_sum(xy, q, alpha, tgt_xy=xy[idx]) + oracle.dl_sum(bxy, nrm, d, alpha, xy[idx])
    # truncation: the terms left out decay by 0.547 per order (a box's points
    # within sqrt(2)/2 sides of its centre, the centres of a pair two sides
    # apart; W and X pairs 0.471), and a dipole's are their derivative:
    # sum over n > p of n 0.547^(n-1) <= (p + 2) 0.547^p / (1 - 0.547)^2
    assert np.max(np.abs(got[idx] - ref)) <= (p + 2) * 0.547 ** p / 0.453 ** 2 * np.max(np.abs(ref))
