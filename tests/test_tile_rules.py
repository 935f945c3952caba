"""The rules by which a kernel picks the form of a direct DFT stage, checked on the
host over all radices, lengths and widths (tests/tile_rules.hip; no GPU)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_direct_stage_rules(tmp_path):
    from paper_2108_11871_amd import build as B

    try:
        cc = B.hipcc()
    except RuntimeError:
        pytest.skip("hipcc is needed")
    exe = str(tmp_path / "tile_rules")
    subprocess.check_call([cc] + B.compile_flags() + ["-O1", os.path.join(HERE, "tile_rules.hip"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "tile rules hold" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
