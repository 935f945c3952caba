"""Small and uneven grids at the edges of the launch-shape rules: tile widths
narrowed to fill the GPU and the row groups of the final pass, against the
FP64 oracle (1e-12, the bar of every FP64 parity test)."""
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
