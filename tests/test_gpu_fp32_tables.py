"""The FP32 copy of the M2L operators, made by the first pass that reads it: a
context that changes precision or order between passes gives bit for bit what
fresh contexts give."""
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


# dense lists below 64 padded coefficients; sparse lists (points along a curve)
@pytest.mark.parametrize("curve,orders", [(False, (16, 12)), (False, (8, 20)), (True, (31, 24))])
def test_fp32_operators_follow_the_plan(yk, curve, orders):
    import torch
    rng = np.random.default_rng(13)
    n, alpha = 6007, 0.1
    xy = rng.random((n, 2))
    if curve:
        th = 2 * np.pi * xy[:, 0]
        xy = 0.5 + 0.4 * np.stack([np.cos(th), np.sin(th)], 1)
    dxy, q = dev(xy), dev(rng.standard_normal(n))
    print(f"fp32 operators: curve {curve}, orders {orders}", flush=True)

    def passes(seq):
        """Outputs of the passes (order, precision) of one context."""
        outs = []
        ctx = yk.yk_create(leaf_size=16, p=seq[0][0], precision=seq[0][1])
        try:
            for p, prec in seq:
                opt = yk.yk_default_options()
                opt.leaf_size, opt.p, opt.precision = 16, p, prec
                yk.yk_set_options(ctx, opt)
                out = torch.empty(n, dtype=torch.float64, device="cuda")
                yk.yk_volume_potential(ctx, dxy, q, None, alpha, out)
                outs.append(host(out))
            if curve:
                assert yk.yk_plan_info_get(ctx, 2).m2l_sparse == 1
        finally:
            yk.yk_destroy(ctx)
        return outs
    a, b = orders
    seq = [(a, yk.YK_PREC_FP64), (a, yk.YK_PREC_FP32), (b, yk.YK_PREC_FP32), (a, yk.YK_PREC_FP64),
           (a, yk.YK_PREC_FP32)]
    for got, one in zip(passes(seq), seq):
        assert np.array_equal(got, passes([one])[0])
