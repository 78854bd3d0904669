"""Which kernel a call goes to and how many workgroups and pool units its launch has: the host arithmetic of
csrc/attn_route.h, compiled without HIP."""
import ctypes
import os
import subprocess

import pytest

import paper_2603_24517_amd as A

HERE = os.path.dirname(os.path.abspath(__file__))
WHOLE, SHARED, SPLIT = range(3)
NCU = 256


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("route") / "route.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "route_shim.cpp")], check=True)
    lib = ctypes.CDLL(so)

    def call(B, Hq, Hkv, Sq, Skv, causal=True, ncu=NCU):
        out = (ctypes.c_longlong * 4)()
        rc = lib.route(B, Hq, Hkv, Sq, Skv, int(causal), ncu, out)
        assert rc == A.ATTN_OK
        return dict(zip(("kind", "items", "wgs", "units"), out))
    return call


@pytest.mark.parametrize("shape,causal,kind", [
    ((1, 4, 4, 512, 512), False, SPLIT),            # few rows in all
    ((1, 32, 8, 1, 32768), True, SPLIT), ((16, 32, 8, 1, 4000), True, SPLIT),
    ((1, 32, 8, 512, 16384), True, SHARED), ((1, 4, 4, 16384, 16384), True, SHARED),
    ((8, 16, 16, 4096, 4096), False, WHOLE), ((24, 16, 16, 200, 200), True, WHOLE), ((2, 16, 16, 1500, 1500), False, WHOLE),
])
def test_kind(route, shape, causal, kind):
    assert route(*shape, causal)["kind"] == kind


def test_grid_of_few_row_calls_stays_launchable(route):
    """HIP takes no grid of 2^32 threads or more: calls of more items than that allows, one workgroup of 512 threads
    each, run in the 256-row kernel, whose grid follows the number of compute units."""
    below, at = route(65535, 128, 128, 1, 1), route(65536, 128, 128, 1, 1)
    assert (below["kind"], below["items"]) == (SPLIT, 2 ** 23 - 128)
    assert (at["kind"], at["items"], at["wgs"]) == (WHOLE, 2 ** 23, NCU)
    for shape in ((1048576, 32, 8, 1, 1), (2 ** 24, 4, 4, 1, 7), (2 ** 20, 64, 8, 3, 1)):
        r = route(*shape)
        assert r["wgs"] * 512 < 2 ** 32, (shape, r)
