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


def test_partials_in_phi_under_capture_and_in_static_scratch():
    """Order-4 boxes whose chunk partials lie in phi: graph replays over outputs that hold
    NaN, with eager work between, extended solves and the static scratch, bit for bit."""
    import ctypes

    import torch
    from paper_2108_11871_amd import _lib, api
    from gpu_util import banner, to_dev

    banner("partials in phi: batch graph, static scratch, extended")
    shapes = [(33, 33, 33), (25, 25, 25), (65, 70, 61), (65, 65), (9, 200)]
    cases = [I.workload_bumps(s, seed=45 + b, scale=[1.0, 1.2, 0.9][:len(s)])[:2] for b, s in enumerate(shapes)]
    rhos = [to_dev(r) for r, _ in cases]
    plans = [api.Plan(s, h, order=4) for s, (_, h) in zip(shapes, cases)]
    refs = [p(r) for p, r in zip(plans, rhos)]
    batch = api.Batch(shapes, [h for _, h in cases], order=4)
    outs = [torch.empty_like(r) for r in rhos]
    for _ in range(4):  # eager and captured, then replays
        for o in outs:
            o.fill_(float("nan"))
        batch(rhos, outs)
        eager = plans[0](rhos[0])
        torch.cuda.synchronize()
        assert all(torch.equal(o, r) for o, r in zip(outs, refs)) and torch.equal(eager, refs[0])
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for p, r, ref in zip(plans, rhos, refs):
        out = torch.full_like(r, float("nan"))
        rc = _lib.lib().ips_execute_static(p._h, ctypes.c_void_p(r.data_ptr()), ctypes.c_void_p(out.data_ptr()), stream)
        torch.cuda.synchronize()
        assert rc == 0 and torch.equal(out, ref)
    ext = api.Plan((27, 27, 27), cases[0][1], order=4, margin=3)  # solves on 33^3
    inner = rhos[0][3:30, 3:30, 3:30].contiguous()
    grown = torch.zeros_like(rhos[0])
    grown[3:30, 3:30, 3:30] = inner
    got = ext(inner)
    torch.cuda.synchronize()
    assert torch.equal(got, plans[0](grown)[3:30, 3:30, 3:30])
