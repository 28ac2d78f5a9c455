"""The fused passes of the warm-start network (256 hidden units) on the GPU
against the FP64 reference: one row, the edges of a workgroup's 16, 32 and 64
rows and of the runs that the weights' gradients are summed in, features at an
odd float offset."""
import numpy as np
import pytest

import workloads as W
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


@pytest.mark.parametrize("rows,offset", [(1, 0), (15, 1), (17, 0), (65, 3), (4111, 0), (8193, 2), (16385, 0)])
def test_fused_passes_vs_fp64(yk, rows, offset):
    import torch
    from oracle import mlp
    cfg = W.config_c0(n_nodes=64, m=8)
    ctx = yk.yk_create()
    bd = yk.Boundary.from_workload(cfg["bnd"])
    ws = yk.yk_ws_create(ctx, bd, hidden=256)
    try:
        n, H, Fp = yk.yk_ws_num_params(ws)
        rng = np.random.default_rng(rows)
        p = (rng.standard_normal(n) * 0.08).astype(np.float32)
        X = rng.standard_normal((rows, Fp)).astype(np.float32)
        t = rng.standard_normal(rows).astype(np.float32)
        yk.yk_ws_set_params(ws, dev(p, torch.float32))
        buf = torch.empty(rows * Fp + 4, dtype=torch.float32, device="cuda")
        Xd = buf[offset:offset + rows * Fp].view(rows, Fp)
        Xd.copy_(torch.as_tensor(X))
        print(f"fused passes rows={rows} offset={offset}", flush=True)
        g = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
        loss = yk.yk_ws_loss_grad(ws, Xd, dev(t, torch.float32), g)
        y = torch.full((rows,), float("nan"), dtype=torch.float32, device="cuda")
        yk.yk_ws_forward(ws, Xd, y)
        g, y = host(g).astype(np.float64), host(y).astype(np.float64)
    finally:
        yk.yk_ws_destroy(ws)
        yk.yk_destroy(ctx)
    p, X, t = p.astype(np.float64), X.astype(np.float64), t.astype(np.float64)
    ref, _ = mlp.forward(p, H, Fp, X)
    ref_loss, ref_g = mlp.loss_grad(p, H, Fp, X, t)
    # FP32 sums of 80 + 256 + 256 terms: below 600 roundings of the terms' size
    # (2^-24 each), random in sign: 600^(1/2) of them, and 16 for the largest of many
    tol = 16 * 600 ** 0.5 * 2.0 ** -24
    assert np.max(np.abs(y - ref)) <= tol * max(1.0, np.max(np.abs(ref)))
    assert abs(loss - ref_loss) <= 2 * tol * max(1.0, ref_loss)
    # the gradient's sums over the rows are of terms of random sign: the sum of
    # their sizes is the scale
    o = np.cumsum([0, H * Fp, H, H * H, H, H, 1])
    for a, b in zip(o[:-1], o[1:]):
        scale = max(np.max(np.abs(ref_g[a:b])), 1e-3)
        assert np.max(np.abs(g[a:b] - ref_g[a:b])) <= 4 * tol * scale * rows ** 0.5
