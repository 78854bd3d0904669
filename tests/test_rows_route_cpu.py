"""Which calls go to the kernel with workgroups of four wavefronts, in which items, and the windows that these are dealt in: the
host arithmetic of csrc/attn_route.h."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "%s/paper_2603_24517_amd/csrc/attn_route.h"
extern "C" int rows(int B, int Hq, int Hkv, int Sq, int Skv, int causal, int ncu, int *out)
{
    attn::Route r = {};
    const int rc = attn::make_shape(B, Hq, Hkv, Sq, Skv, r.shape, r.sched);
    if (rc != ATTN_OK) return rc;
    attn::make_route(B, Hkv, Skv, causal, ncu, r);
    const attn::Rows &w = r.rows;
    const int all[] = {(int)r.kind, w.kgroups, w.tile_pos, w.ntile, w.nrest, w.window, w.window0};
    for (int i = 0; i < 7; ++i) out[i] = all[i];
    return rc;
}
"""
WHOLE, SHARED, SPLIT = range(3)


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "rows.cpp").write_text(SHIM % ROOT)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(d / "rows.so"), str(d / "rows.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "rows.so"))

    def call(B, Hq, Hkv, Sq, Skv, causal, ncu=256):
        out = (ctypes.c_int * 7)()
        assert lib.rows(B, Hq, Hkv, Sq, Skv, int(causal), ncu, out) == 0
        return dict(zip(("kind", "kgroups", "tile_pos", "ntile", "nrest", "window", "window0"), out))
    return call


@pytest.mark.parametrize("shape,causal,kgroups", [
    ((1, 32, 8, 1111, 1111), True, 2), ((1, 16, 16, 2000, 2000), True, 2), ((24, 16, 16, 200, 200), True, 1), ((300, 4, 4, 150, 150), True, 2),
    ((5, 4, 4, 1200, 1200), False, 1), ((32, 40, 40, 123, 123), True, 1),
    ((2, 16, 16, 1500, 1500), False, 0), ((8, 16, 16, 4096, 4096), False, 0), ((8, 16, 16, 4096, 4096), True, 0),
    ((1, 64, 8, 32768, 32768), True, 0), ((1, 32, 8, 512, 16384), True, 0), ((1, 4, 4, 512, 512), False, 0), ((16, 32, 8, 1, 4000), True, 0),
])
def test_which_calls(rows, shape, causal, kgroups):
    r = rows(*shape, causal)
    assert r["kgroups"] == kgroups and (kgroups == 0 or r["kind"] == WHOLE), r


@pytest.mark.parametrize("shape,causal", [
    ((2, 64, 8, 104, 5599), True), ((4, 64, 8, 35, 4426), False), ((2, 40, 40, 105, 5604), True), ((1, 40, 40, 293, 3978), False),     # shared
    ((9, 6, 2, 517, 4612), True), ((20, 12, 3, 269, 2017), True), ((2, 4, 4, 2300, 2300), True), ((1, 16, 16, 3222, 3222), True),             # shared
    ((20, 32, 8, 63, 6726), True), ((9, 40, 40, 148, 2876), True), ((4, 40, 40, 218, 2809), True), ((4, 32, 4, 264, 3506), True),       # far keys
    ((22, 40, 40, 391, 391), True), ((91, 16, 16, 242, 242), False), ((59, 16, 16, 400, 400), True), ((162, 4, 4, 221, 221), False), ((57, 32, 8, 694, 694), True),      # many items
    ((4, 16, 16, 1607, 63), True), ((4, 32, 4, 2481, 34), True),                                                                        # rows without keys
])
def test_calls_that_smaller_workgroups_made_slower(rows, shape, causal):
    """Measured 3 to 56 % slower there than in 256-row items, with K and V from memory or from the last cache."""
    assert rows(*shape, causal)["kgroups"] == 0


def _item(r, bid):
    """Workgroup -> (tile, rest), as the kernel does it."""
    if bid < r["window0"] * r["ntile"]:
        tile_r, rest = divmod(bid, r["window0"])
    else:
        win, inside = divmod(bid - r["window0"] * r["ntile"], r["window"] * r["ntile"])
        tile_r, k = divmod(inside, r["window"])
        rest = r["window0"] + win * r["window"] + k
    return r["ntile"] - 1 - tile_r, rest


@pytest.mark.parametrize("shape,ncu", [((24, 16, 16, 200, 200), 256), ((24, 16, 16, 150, 150), 80), ((1, 32, 8, 1111, 1111), 256), ((11, 4, 4, 998, 998), 256),
                                       ((11, 4, 4, 998, 998), 80), ((35, 4, 4, 150, 150), 256), ((7, 12, 3, 600, 700), 256),
                                       ((1, 3, 3, 5000, 90), 80), ((13, 40, 40, 133, 135), 256)])
def test_every_item_once(rows, shape, ncu):
    r = rows(*shape, True, ncu)
    assert r["kgroups"] != 0, r
    n = r["ntile"] * r["nrest"]
    assert 1 <= r["window0"] <= r["window"] <= r["nrest"] and (r["nrest"] - r["window0"]) % r["window"] == 0
    assert r["window"] == r["nrest"] or r["window"] % 8 == 0
    assert sorted(_item(r, b) for b in range(n)) == [(t, k) for t in range(r["ntile"]) for k in range(r["nrest"])]
