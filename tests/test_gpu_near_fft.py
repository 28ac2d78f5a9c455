"""The curve FFTs of the near-boundary evaluation (three stages to a pass, after
one of one or two when their number is not a multiple of three) at sizes of
every remainder, the largest included: one grid step against a closed form."""
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


@pytest.mark.parametrize("outer,inner", [(8192, 512), (4096, 2048), (2048, 1024)])
def test_curve_ffts_closed_form(yk, outer, inner):
    import torch
    b = W.make_boundary([W.circle((0.0, 0.0), 0.4, outer), W.circle((0.0, 0.0), 0.1, inner, ccw=False)])
    grid, pts = W.grid_box(-0.5, 0.5, 512)
    uf = lambda p: np.sin(3 * p[:, 0]) * np.sin(2 * p[:, 1]) + 1.0
    a2 = 1e-3
    B = (1 + 13 * a2) * uf(pts) - 13 * a2
    inside = b.region(pts) < 0
    print(f"curve FFTs {outer} + {inner}", flush=True)
    ctx = yk.yk_create()
    try:
        bd = yk.Boundary.from_workload(b)
        sig = torch.zeros(b.n, dtype=torch.float64, device="cuda")
        u = torch.empty(pts.shape[0], dtype=torch.float64, device="cuda")
        yk.yk_heat_step_grid(ctx, bd, yk.make_grid(*grid), dev(B), yk.HEAT_ZERO_GUESS, dev(uf(b.xy)), a2, 1e-12, sig, u)
        n_near, _ = yk.yk_near_info(ctx)
        got = host(u)
    finally:
        yk.yk_destroy(ctx)
    assert n_near > 0
    # the grid's quadrature errs by less than 1e-6 here with 1,024 + 512 nodes;
    # no curve has fewer, and the boundary's error falls with its nodes
    assert np.max(np.abs(got - uf(pts))[inside]) < 1e-6
