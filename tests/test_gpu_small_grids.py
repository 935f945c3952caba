"""Small and uneven grids at the edges of the launch-shape rules (tile widths
narrowed to fill the GPU, the row groups of the final pass), of the prime radices
and of the register tiles, against the FP64 oracle (1e-12 in FP64 and 1e-6 in the mixed modes,
the bars of every parity test)."""
import pytest

from oracle import poisson as P
from paper_2108_11871_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 1e-12


# row groups of the final pass: n0 - 2 rows, doubled while they fit 256 threads
# (1, 2, 64, 65, 127, 128, 129 rows); the other axes leave one ragged tile,
# exactly one tile, or many
@pytest.mark.parametrize("shape,order", [((3, 9), 4), ((4, 21), 4), ((66, 66), 6), ((67, 9), 6), ((129, 35), 6),
                                         ((130, 18), 4), ((131, 67), 6), ((3, 9, 8), 4), ((66, 9, 8), 6),
                                         ((67, 19, 8), 6), ((130, 10, 9), 6), ((9, 131, 10), 6)])
def test_row_groups_and_narrow_tiles(shape, order):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, rel_err, to_dev

    banner("shape=%s order=%d" % (shape, order))
    rho, h, _ = I.workload_bumps(shape, seed=33, scale=[1.0, 1.2, 0.9][:len(shape)])
    phi = api.Plan(shape, h, order=order)(to_dev(rho))
    torch.cuda.synchronize()
    assert rel_err(phi.cpu().numpy(), P.solve(rho, h, order)) < TOL


# prime factors 7, 11, 13 (registers); 17 .. 509 (matrix cores: one row block,
# 16 frequencies exactly, one more than 48, the most blocks per wave); 521 (direct
# sums: too many blocks); squares and products of them, with and without powers
# of two, in full and narrowed tiles; in 3D both transforms of a face
@pytest.mark.parametrize("mode,tol", [("fp64", TOL), ("mixed_fp32_slices", 1e-6)])
@pytest.mark.parametrize("panels", [(7, 11), (13, 49), (17, 31), (37, 97), (121, 56), (143, 66), (169, 23), (289, 29),
                                    (323, 13), (257, 181), (502, 11), (509, 7), (521, 19), (13, 17, 22),
                                    (74, 31, 11), (62, 34, 58)])
def test_prime_radices(panels, mode, tol):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, rel_err, to_dev

    shape = tuple(m + 1 for m in panels)
    banner("shape=%s %s" % (shape, mode))
    rho, h, _ = I.workload_bumps(shape, seed=34, scale=[1.0, 1.2, 0.9][:len(shape)])
    phi = api.Plan(shape, h, order=6, precision=mode)(to_dev(rho))
    torch.cuda.synchronize()
    assert rel_err(phi.cpu().numpy(), P.solve(rho, h, 6, boundary="fft")) < tol


# register tiles: every length 2M = 256 .. 4096 (8192: test_gpu_long.py), the columns
# one ragged tile, one more than whole tiles, and many
@pytest.mark.parametrize("mode,tol", [("fp64", TOL), ("mixed_fp32", 1e-6), ("mixed_fp32_slices", 1e-6)])
@pytest.mark.parametrize("shape", [(129, 257), (257, 19), (513, 129), (1025, 257), (2049, 12), (130, 2049),
                                   (129, 9, 257), (257, 129, 20)])
def test_register_tiles(shape, mode, tol):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, rel_err, to_dev

    banner("shape=%s %s" % (shape, mode))
    rho, h, _ = I.workload_bumps(shape, seed=35, scale=[1.0, 1.2, 0.9][:len(shape)])
    phi = api.Plan(shape, h, order=6, precision=mode)(to_dev(rho))
    torch.cuda.synchronize()
    assert rel_err(phi.cpu().numpy(), P.solve(rho, h, 6, boundary="fft")) < tol


# wider register tiles: rho along z and along y at 2M = 512 and 1024 (enough blocks for
# twice and, in FP32, four times the default, ragged columns), contractions of two
# chunks per tile at 2M = 1024
# with an odd number of chunks and an even one
@pytest.mark.parametrize("mode,tol", [("fp64", TOL), ("mixed_fp32", 1e-6), ("mixed_fp32_slices", 1e-6)])
@pytest.mark.parametrize("shape", [(131, 131, 257), (131, 257, 132), (129, 75, 513), (129, 150, 513),
                                   (513, 37, 65), (513, 34, 66)])
def test_double_width_tiles(shape, mode, tol):
    import torch
    from paper_2108_11871_amd import api
    from gpu_util import banner, rel_err, to_dev

    banner("shape=%s %s" % (shape, mode))
    rho, h, _ = I.workload_bumps(shape, seed=36, scale=[1.0, 1.2, 0.9])
    phi = api.Plan(shape, h, order=6, precision=mode)(to_dev(rho))
    torch.cuda.synchronize()
    assert rel_err(phi.cpu().numpy(), P.solve(rho, h, 6, boundary="fft")) < tol
