"""The HIP adjoint rho_bar = A^T phi_bar (ips_execute_adjoint) and the
autograd function built on it.

Bars:
* parity with the oracle's adjoint (a separate transposed chain, itself
  pinned by dot-product and dense-transpose tests): 1e-12 relative, max norm;
* dot-product identity <A v, w> = <v, A^T w> between the HIP forward and the
  HIP adjoint at sizes the oracle cannot reach: 1e-12 relative;
* gradients of J(rho) = 1/2 |phi(rho) - phi_target|^2 through SolveFn
  against central differences, which are exact for a quadratic J
  (rounding only): 1e-10 relative in FP64.
"""
import numpy as np
import pytest

from oracle import poisson as P
from paper_2108_11871_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _gpu_adjoint(w, h, order, precision="fp64", flag=False):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import to_dev

    plan = api.Plan(w.shape, h, order=order, precision=precision, adjoint=flag)
    out = plan.adjoint(to_dev(w))
    torch.cuda.synchronize()
    res = out.cpu().numpy()
    plan.close()
    return res


@pytest.mark.parametrize("shape,h,order", [
    ((17,), (0.1,), 4), ((64,), (0.03,), 4), ((257,), (2.0 / 256,), 4),
    ((9, 11), (0.2, 0.13), 4), ((9, 11), (0.2, 0.13), 6), ((12, 13), (0.1, 0.07), 6),
    ((33, 41), (0.06, 0.05), 6), ((50, 38), (0.04, 0.05), 4), ((3, 5), (0.5, 0.3), 4),
    ((8, 9, 10), (0.2, 0.17, 0.11), 4), ((8, 9, 10), (0.2, 0.17, 0.11), 6),
    ((10, 11, 12), (0.1, 0.12, 0.09), 6), ((17, 21, 19), (0.1, 0.08, 0.09), 6),
    ((24, 17, 31), (0.05, 0.07, 0.04), 4), ((3, 4, 5), (0.4, 0.3, 0.2), 4),
])
def test_adjoint_matches_oracle(shape, h, order):
    from gpu_util import banner, rel_err

    banner("adjoint shape=%s order=%d" % (shape, order))
    rng = np.random.default_rng(sum(shape) * 7 + order)
    w = rng.standard_normal(shape)
    ref = P.adjoint(w, h, order)
    got = _gpu_adjoint(w, h, order)
    err = rel_err(got, ref)
    print("  rel err %.3e" % err, flush=True)
    assert err < TOL
    assert np.all(got[P.boundary_mask(shape)] == 0.0)


def test_adjoint_33_cube_order6():
    from gpu_util import banner, rel_err

    banner("adjoint 33^3 order 6")
    n = 33
    rho, h, _ = I.workload_bumps_3d(n, seed=11)
    w = rho + 0.1 * np.random.default_rng(2).standard_normal(rho.shape)
    ref = P.adjoint(w, h, 6)
    got = _gpu_adjoint(w, h, 6)
    err = rel_err(got, ref)
    print("  rel err %.3e" % err, flush=True)
    assert err < TOL


def test_adjoint_preallocation_and_mixed_precision():
    """The workspace flag changes only when the adjoint's buffers are
    allocated (bitwise the same result).  The mixed modes run the volume
    transforms in FP32 tiles with FP64 data in memory: the result stays
    within a few FP32 roundings of the FP64 adjoint (1e-6 relative, max
    norm), the bar of the mixed forward solve."""
    from gpu_util import rel_err

    for shape, h in (((20, 18, 22), (0.1, 0.11, 0.09)), ((33, 41), (0.06, 0.05))):
        w = np.random.default_rng(5).standard_normal(shape)
        ref = _gpu_adjoint(w, h, 6)
        assert np.array_equal(_gpu_adjoint(w, h, 6, flag=True), ref)
        for prec in ("mixed_fp32", "mixed_fp32_slices"):
            err = rel_err(_gpu_adjoint(w, h, 6, precision=prec), ref)
            print("  %s %s rel err %.3e" % (shape, prec, err), flush=True)
            assert err < 1e-6


@pytest.mark.parametrize("shape,order,precision", [
    ((65, 65, 65), 6, "fp64"), ((129, 97, 113), 6, "fp64"), ((129, 129, 129), 4, "fp64"),
    ((513, 385), 6, "fp64"), ((129, 129, 129), 6, "mixed_fp32_slices")])
def test_dot_product_identity_large(shape, order, precision):
    """FP64: 1e-12 of the scale; the mixed modes (FP32 transforms in both
    directions): 1e-6."""
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner

    banner("dot product shape=%s order=%d %s" % (shape, order, precision))
    tol = 1e-12 if precision == "fp64" else 1e-6
    h = tuple(2.0 / (s - 1) for s in shape)
    plan = api.Plan(shape, h, order=order, precision=precision)
    g = torch.Generator(device="cuda:0").manual_seed(7)
    v = torch.randn(shape, dtype=torch.float64, device="cuda:0", generator=g)
    w = torch.randn(shape, dtype=torch.float64, device="cuda:0", generator=g)
    Av = plan(v)
    Atw = plan.adjoint(w)
    inner = tuple(slice(1, -1) for _ in shape)
    lhs = float((Av * w).sum())
    rhs = float((v[inner] * Atw[inner]).sum())
    # scale of the sums: sum |Av| |w|
    scale = float((Av.abs() * w.abs()).sum())
    plan.close()
    print("  <Av,w> %.15e  <v,A^T w> %.15e  rel %.2e" % (lhs, rhs, abs(lhs - rhs) / scale), flush=True)
    assert abs(lhs - rhs) <= tol * scale


@pytest.mark.parametrize("shape,precision", [((33, 33, 33), "fp64"), ((65, 49, 57), "fp64"),
                                             ((65, 65), "fp64"), ((33, 33, 33), "mixed_fp32_slices")])
def test_autograd_gradient_matches_central_differences(shape, precision):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, to_dev

    banner("autograd shape=%s %s" % (shape, precision))
    d = len(shape)
    rho_np, h, _ = I.workload_bumps(shape, seed=4)
    tgt_np, _, _ = I.workload_bumps(shape, seed=5)
    plan = api.Plan(shape, h, order=6, precision=precision)
    target = plan(to_dev(tgt_np)).detach()
    rho = to_dev(rho_np).requires_grad_(True)
    phi = api.SolveFn.apply(rho, plan)
    J = 0.5 * ((phi - target) ** 2).sum()
    J.backward()
    grad = rho.grad.detach()

    def Jof(r):
        with torch.no_grad():
            p = plan(r)
            return 0.5 * float(((p - target) ** 2).sum())

    rng = np.random.default_rng(6)
    inner = tuple(slice(1, -1) for _ in range(d))
    worst = 0.0
    for t in range(4):
        if t % 2 == 0:
            v_np, _, _ = I.workload_bumps(shape, seed=100 + t)
        else:
            v_np = np.zeros(shape)
            v_np[inner] = rng.standard_normal(tuple(s - 2 for s in shape))
        v = to_dev(v_np)
        tau = float(rho.detach().abs().max() / v.abs().max())
        fd = (Jof(rho.detach() + tau * v) - Jof(rho.detach() - tau * v)) / (2.0 * tau)
        an = float((grad * v).sum())
        rel = abs(fd - an) / max(abs(fd), abs(an), 1e-300)
        worst = max(worst, rel)
        print("  direction %d: <grad,v> %.12e  FD %.12e  rel %.2e" % (t, an, fd, rel), flush=True)
    plan.close()
    # FP64: only rounding separates the two; the mixed forward perturbs J by ~1e-7 relative
    assert worst < (1e-10 if precision == "fp64" else 1e-4)


@pytest.mark.parametrize("precision", ["fp64", "mixed_fp32_slices"])
def test_autograd_257_cube_sixteen_directions(precision):
    """J = 1/2 |phi(rho) - phi_target|^2 on 257^3 (rho seed 4, phi_target the
    FP64 solve of the bump sum with seed 5): <dJ/drho, v> against central
    differences along 8 bump-sum and 8 white-noise directions."""
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, to_dev

    banner("autograd 257^3 %s" % precision)
    n = 257
    rho_np, h, _ = I.workload_bumps_3d(n, seed=4)
    tgt_np, _, _ = I.workload_bumps_3d(n, seed=5)
    ref_plan = api.Plan(rho_np.shape, h, order=6)
    target = ref_plan(to_dev(tgt_np)).detach()
    ref_plan.close()
    del tgt_np
    plan = api.Plan(rho_np.shape, h, order=6, precision=precision)
    rho = to_dev(rho_np).requires_grad_(True)
    phi = api.SolveFn.apply(rho, plan)
    J = 0.5 * ((phi - target) ** 2).sum()
    J.backward()
    grad = rho.grad.detach()
    r0 = rho.detach()

    def Jof(r):
        with torch.no_grad():
            return 0.5 * float(((plan(r) - target) ** 2).sum())

    gen = torch.Generator(device="cuda:0").manual_seed(6)
    worst = 0.0
    for t in range(16):
        if t < 8:
            c, w, a = I.bump_params(600 + t, 3)
            v = to_dev(I.bump_sum((n, n, n), c, w, a, 10))
        else:
            v = torch.zeros_like(r0)
            v[1:-1, 1:-1, 1:-1] = torch.randn((n - 2,) * 3, dtype=torch.float64, device="cuda:0",
                                              generator=gen)
        tau = float(r0.abs().max() / v.abs().max())
        fd = (Jof(r0 + tau * v) - Jof(r0 - tau * v)) / (2.0 * tau)
        an = float((grad * v).sum())
        rel = abs(fd - an) / max(abs(fd), abs(an), 1e-300)
        worst = max(worst, rel)
        print("  direction %2d: <grad,v> %.12e  FD %.12e  rel %.2e" % (t, an, fd, rel), flush=True)
    plan.close()
    assert worst < (1e-10 if precision == "fp64" else 1e-4)


# shell form of the FP64 adjoint: the smallest grids (core layers of both sides share
# nodes up to M = 9), layers of one node, one and several splits of the sums, rows
# shorter and longer than a wave
@pytest.mark.parametrize("shape,order", [((8, 8, 8), 6), ((8, 9, 13), 6), ((11, 10, 66), 6), ((70, 8, 9), 6),
                                         ((9, 131, 10), 6), ((3, 4, 5), 4), ((40, 3, 6), 4), ((8, 8), 6), ((9, 12), 6),
                                         ((257, 9), 6), ((10, 300), 6), ((3, 7), 4)])
def test_shell_adjoint_small(shape, order):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, rel_err, to_dev

    banner("adjoint shape=%s order=%d" % (shape, order))
    h = I.grid_spacing(shape, -1.0, 1.3)
    w = np.random.default_rng(5).standard_normal(shape)
    got = api.Plan(shape, h, order=order, adjoint=True).adjoint(to_dev(w))
    torch.cuda.synchronize()
    assert rel_err(got.cpu().numpy(), P.adjoint(w, h, order)) < 1e-12


# register tiles of the expansion: slices as columns (ragged, one more than whole tiles)
# and, with fewer slices than a tile's columns, the other slots; every family, 2M = 256 .. 2048
@pytest.mark.parametrize("shape,order", [((129, 18, 257), 6), ((20, 129, 12), 4), ((129, 9, 130), 6), ((10, 257, 129), 6),
                                         ((257, 129, 9), 4), ((1025, 9, 10), 4), ((8, 513, 19), 6), ((130, 129), 6),
                                         ((1025, 300), 4)])
def test_expand_register_tiles(shape, order):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, rel_err, to_dev

    banner("adjoint shape=%s order=%d" % (shape, order))
    h = I.grid_spacing(shape, -1.0, 1.3)
    w = np.random.default_rng(6).standard_normal(shape)
    got = api.Plan(shape, h, order=order, adjoint=True).adjoint(to_dev(w))
    torch.cuda.synchronize()
    assert rel_err(got.cpu().numpy(), P.adjoint(w, h, order)) < 1e-12


# the tile budget of a plan does not reach the expansion's register tiles (the budget is
# read once per process: each runs in one of its own)
@pytest.mark.parametrize("work", ["1024", "4096"])
def test_adjoint_at_other_tile_budgets(work):
    import os
    import subprocess
    import sys
    from gpu_util import banner

    banner("adjoint, tile budget " + work)
    code = """
import numpy as np, torch
from oracle import poisson as P
from paper_2108_11871_amd import api, inputs as I
for shape in ((129, 20, 257), (8, 257, 129), (257, 130)):
    h = I.grid_spacing(shape, -1.0, 1.3)
    w = np.random.default_rng(8).standard_normal(shape)
    got = api.Plan(shape, h, order=6, adjoint=True).adjoint(torch.from_numpy(w).cuda()).cpu().numpy()
    ref = P.adjoint(w, h, 6)
    err = np.abs(got - ref).max() / np.abs(ref).max()
    assert err < 1e-12, (shape, err)
print("adjoint budgets ok")
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, env=dict(os.environ, IPS_TILE_WORK=work), text=True,
                       capture_output=True, timeout=110)
    assert r.returncode == 0 and "adjoint budgets ok" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
