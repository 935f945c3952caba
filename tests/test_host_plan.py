"""What plans decide on the host -- workspace sizes, kernels -- through the library on a
stand-in runtime (tests/stub_runtime.cpp): no GPU needed."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ADJOINT = 2
SCRATCH = 64 << 20


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ is needed for the stand-in runtime")
    from paper_2108_11871_amd import _lib

    _lib.lib()  # raises if the library is not built
    from paper_2108_11871_amd import build as B

    exe = str(tmp_path_factory.mktemp("stub") / "stub")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-rdynamic", "-I" + os.path.join(ROOT, "include"),
                           os.path.join(HERE, "stub_runtime.cpp"), B.LIB, "-Wl,--allow-shlib-undefined",
                           "-Wl,-rpath," + os.path.dirname(B.LIB), "-o", exe])

    def run(requests, **env):
        text = "".join("%d %s %d %d %d %s\n" % (len(n), " ".join(map(str, n)), order, precision, flags, call)
                       for n, order, precision, flags, call in requests)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=300, env=dict(os.environ, **env))
        assert r.returncode == 0, r.stderr
        return r.stdout.split("\n")

    return run


# The workspace of a plan with whole contraction tiles, volume-form adjoint and separate
# areas: (shape, order, precision, flags, bytes). Buffers of these sizes are in use, and
# the ones below 64 MiB run in the static scratch.
SIZES = [
    ((8, 257, 257), 6, 0, ADJOINT, 64503040),
    ((12, 257, 257), 6, 0, ADJOINT, 91075840),
    ((8, 129, 129), 6, 0, ADJOINT, 16522496),
    ((122, 84, 88), 4, 0, ADJOINT, 67027712),
    ((163, 13, 237), 6, 0, ADJOINT, 66737728),
    ((146, 12, 276), 6, 0, ADJOINT, 65961216),
    ((27, 64, 31), 4, 0, 0, 2095008),
    ((27, 64, 31), 4, 0, ADJOINT, 3907392),
    ((33, 33, 33), 6, 0, 0, 2000944),
    ((33, 33, 33), 4, 0, 0, 1493296),
    ((65, 65, 65), 4, 0, 0, 9948720),
    ((65, 65, 65), 6, 0, 0, 12044592),
    ((8, 8, 8), 6, 0, ADJOINT, 89088),
    ((65, 1025, 1025), 4, 0, ADJOINT, 4178249216),
    ((237, 241, 8), 6, 0, 0, 39909616),
    ((9, 14), 6, 0, ADJOINT, 13824),
    ((63, 60), 4, 0, 0, 54096),
    ((8, 3966), 6, 0, ADJOINT, 2926560),
    ((97, 97, 97), 6, 0, 0, 41339440),
    ((129, 129, 129), 6, 0, ADJOINT, 212927744),
    ((65, 65, 65), 6, 2, ADJOINT, 24462336),
    ((65, 65, 65), 6, 1, 0, 11044400),
]


def test_workspace_needs_no_more_than_whole_tiles_did(stub):
    out = stub([(n, order, precision, flags, "size") for n, order, precision, flags, _ in SIZES])
    for (n, order, precision, flags, was), now in zip(SIZES, out):
        assert 0 < int(now) <= was, (n, order, precision, flags, was, now)


def test_static_scratch_still_holds_these_plans(stub):
    fit = [s for s in SIZES if s[4] <= SCRATCH]
    assert len(fit) > 10
    for s, now in zip(fit, stub([s[:4] + ("size",) for s in fit])):
        assert int(now) <= SCRATCH, (s, now)


# lengths with register tiles: 3D the transformed axes are 1 and 0, with and without
# enough slices for a tile's columns; 2D both axes
@pytest.mark.parametrize("work", ["1024", "2048", "4096"])
@pytest.mark.parametrize("n", [(129, 257, 20), (129, 513, 200), (257, 129, 12), (1025, 257, 40), (129, 257), (2049, 1025)])
def test_expansion_takes_register_tiles_at_every_budget(stub, n, work):
    out = stub([(n, 6, 0, ADJOINT, "adjoint")], IPS_TILE_WORK=work)
    exp = [line.split()[0] for line in out if "k_expand" in line]
    assert len(exp) == len(n)
    assert all(e.startswith("k_expand_rt<") for e in exp), exp


# powers of two, 5-smooth and other panel counts in one block of 256 or 1024 threads
@pytest.mark.parametrize("n,kind", [(65, 1), (1025, 1), (4097, 1), (61, 2), (1001, 2), (3001, 2), (50, 0), (2047, 0)])
def test_1d_kernels_hold_the_radices_of_their_length_only(stub, n, kind):
    out = stub([((n,), 4, 0, 0, "execute"), ((n,), 4, 0, ADJOINT, "adjoint")])
    names = [line.split()[0] for line in out if line.startswith("k_")]
    assert [x.split("<")[0] for x in names] == ["k_1d", "k_adj_1d"]
    assert all(x.split(",")[1] == str(kind) for x in names), names


# the launches of the volume-form adjoint (two and three axes, orders 6 and 4), which the
# shell form must not exceed on grids that launches bound
@pytest.mark.parametrize("n,order,most", [((14, 14), 6, 20), ((14, 14), 4, 13), ((33, 40), 6, 20), ((14, 15, 16), 6, 38),
                                          ((14, 15, 16), 4, 24), ((33, 33, 33), 6, 38), ((257, 257, 257), 6, 38)])
def test_fp64_adjoint_launches(stub, n, order, most):
    out = stub([(n, order, 0, ADJOINT, "adjoint")])
    assert 0 < len([line for line in out if line.startswith("k_")]) <= most


@pytest.mark.parametrize("precision", [0, 2])
def test_tiny_lines_are_not_split_below_a_wave(stub, precision):
    # 2M = 26: a tile of two columns would hold 26 elements, of four 52
    out = stub([((14, 14), 6, precision, ADJOINT, call) for call in ("execute", "adjoint")])
    passes = [line.split() for line in out if line.startswith("k_pass<")]
    assert len(passes) > 8
    assert all(int(blocks) <= 5 for _, blocks, _ in passes), passes
