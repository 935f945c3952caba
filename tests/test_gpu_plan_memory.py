"""Buffers that share a place: chunk partials with the shell layers or in phi, the
adjoint's shell layers with the forward solve's or in the slice stack. Solves and
adjoints in turn in memory that starts as NaN, against the FP64 oracle."""
import numpy as np
import pytest

from oracle import poisson as P
from paper_2108_11871_amd import inputs as I

pytestmark = pytest.mark.gpu


# partials: every family in the workspace, one of them in phi (2D and 3D, equal and
# unequal panel counts), and tiles widened to fit; the adjoint's shell layers of thin,
# flat and cubic boxes larger and smaller than the slice stack, both orders
@pytest.mark.parametrize("adjoint", [True, False])
@pytest.mark.parametrize("shape,order", [((33, 33, 33), 6), ((33, 33, 33), 4), ((65, 70, 61), 4), ((27, 64, 31), 4),
                                         ((25, 25, 25), 4), ((8, 40, 47), 6), ((9, 8, 70), 6), ((3, 20, 21), 4),
                                         ((65, 65), 4), ((65, 65), 6), ((9, 200), 4), ((257, 200), 6), ((8, 9), 6)])
def test_shared_buffers(shape, order, adjoint):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, rel_err, to_dev

    banner("shape=%s order=%d adjoint=%s" % (shape, order, adjoint))
    rho, h, _ = I.workload_bumps(shape, seed=41, scale=[1.0, 1.2, 0.9][:len(shape)])
    w = np.random.default_rng(7).standard_normal(shape)
    plan = api.Plan(shape, h, order=order, adjoint=adjoint, no_workspace=True)
    buf = torch.full((plan.workspace_bytes // 8 + 1,), float("nan"), dtype=torch.float64, device="cuda:0")
    plan.set_workspace(buf)
    phi = torch.full(shape, float("nan"), dtype=torch.float64, device="cuda:0")
    grad = torch.full(shape, float("nan"), dtype=torch.float64, device="cuda:0")
    ref, ref_adj = P.solve(rho, h, order), P.adjoint(w, h, order)
    rho_d, w_d = to_dev(rho), to_dev(w)
    for _ in range(2):
        plan(rho_d, phi)
        plan.adjoint(w_d, grad)
        torch.cuda.synchronize()
        assert rel_err(phi.cpu().numpy(), ref) < 1e-12
        assert rel_err(grad.cpu().numpy(), ref_adj) < 1e-12
    plan.close()
