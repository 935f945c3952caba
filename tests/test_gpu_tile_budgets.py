"""Solves of plans with other tile budgets than the default (read once per process, so
each runs in a process of its own): tiles of 4 and of 16 elements a thread, against the
FP64 oracle."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CODE = """
import numpy as np, torch
from oracle import poisson as P
from paper_2108_11871_amd import api, inputs as I
for shape in ((129, 20, 65), (33, 257, 40), (513, 12, 70), (46, 61, 35), (129, 513), (1025, 99)):
    rho, h, _ = I.workload_bumps(shape, seed=43, scale=[1.0, 1.2, 0.9][:len(shape)])
    ref = P.solve(rho, h, 6, boundary="fft")
    for mode, tol in (("fp64", 1e-12), ("mixed_fp32", 1e-6), ("mixed_fp32_slices", 1e-6)):
        phi = api.Plan(shape, h, order=6, precision=mode)(torch.from_numpy(rho).cuda()).cpu().numpy()
        err = np.abs(phi - ref).max() / np.abs(ref).max()
        print(shape, mode, err, flush=True)
        assert err < tol, (shape, mode, err)
print("budget ok")
"""


@pytest.mark.parametrize("work", ["1024", "4096"])
def test_solve_at_other_tile_budgets(work):
    from gpu_util import banner

    banner("solve, tile budget " + work)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CODE], cwd=root, env=dict(os.environ, IPS_TILE_WORK=work), text=True,
                       capture_output=True, timeout=110)
    assert r.returncode == 0 and "budget ok" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
