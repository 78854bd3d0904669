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
