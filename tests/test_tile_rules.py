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


def test_wide_contractions_keep_four_waves(tmp_path):
    """The FP32 contractions of 16 elements a thread (a tile budget of 4096) stay within 128
    registers, the most at which four waves of a SIMD are resident."""
    import re

    from paper_2108_11871_amd import build as B

    try:
        cc = B.hipcc()
    except RuntimeError:
        pytest.skip("hipcc is needed")
    r = subprocess.run([cc] + B.compile_flags() + ["--offload-device-only", "-c", os.path.join(B.CSRC, "conv_f32.hip"),
                                                  "-o", str(tmp_path / "x.o"), "-Rpass-analysis=kernel-resource-usage"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    use = re.findall(r"Function Name: (\S+).*?VGPRs: (\d+)", r.stderr, re.S)
    wide = {n: int(v) for n, v in use if "4k_ccIffLi16E" in n}
    assert len(wide) > 10
    # (any length, 4 NT < N <= 8 NT: eight slot rows a thread)
    assert all(v <= 128 for n, v in wide.items() if "ELi0ELi8E" not in n), wide
