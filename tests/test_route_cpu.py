"""Which kernel a call goes to and how many workgroups and pool units its launch has: the host arithmetic of
csrc/attn_route.h, compiled without HIP."""
import ctypes
import os
import re
import subprocess

import pytest

import paper_2603_24517_amd as A

HERE = os.path.dirname(os.path.abspath(__file__))
WHOLE, SHARED, SPLIT = range(3)
NCU = 256


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("route") / "route.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "route_shim.cpp")], check=True)
    return ctypes.CDLL(so)


@pytest.fixture(scope="module")
def route(lib):
    def call(B, Hq, Hkv, Sq, Skv, causal=True, ncu=NCU):
        out = (ctypes.c_longlong * 7)()
        rc = lib.route(B, Hq, Hkv, Sq, Skv, int(causal), ncu, out)
        assert rc == A.ATTN_OK
        return dict(zip(("kind", "items", "wgs", "units", "once", "once_null", "kgroups"), out))
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


@pytest.mark.parametrize("shape,shared", [
    ((1, 32, 8, 1, 1280), True), ((2, 16, 16, 1, 1280), True), ((4, 16, 16, 1, 1280), True), ((1, 8, 8, 1, 1216), False),
    ((8, 16, 16, 1, 1600), False), ((8, 16, 16, 1, 1800), True),            # 128 items of one tile
    ((85, 1, 1, 1, 1280), True), ((86, 1, 1, 1, 1280), False),              # three parts, two
    ((1, 32, 4, 51, 1700), False), ((1, 32, 4, 51, 2200), True),            # 13 tiles, 52 items
    ((1, 4, 4, 700, 2400), False), ((1, 4, 4, 700, 2700), True),            # 22 tiles, 88 items
])
def test_split_key_items_are_shared_only_where_that_pays(route, shape, shared):
    r = route(*shape)
    assert r["kind"] == SPLIT and (r["units"] > 0) == shared == (r["wgs"] > r["items"]), r


@pytest.mark.parametrize("shape,kind", [
    ((16, 64, 8, 4, 4096), SPLIT), ((64, 64, 8, 4, 4096), SPLIT), ((1024, 32, 8, 1, 128), SPLIT),       # up to 32 rows: any number
    ((16, 64, 8, 5, 4096), SPLIT), ((17, 64, 8, 8, 2048), SPLIT), ((24, 64, 8, 8, 2048), SPLIT),        # 33 .. 64: 256, 272, 384 tiles
    ((34, 64, 8, 8, 1500), SPLIT), ((40, 64, 8, 8, 1500), SPLIT),                                       # 544, 640
    ((17, 64, 8, 8, 2049), SHARED), ((25, 64, 8, 8, 500), WHOLE), ((41, 64, 8, 8, 500), SPLIT), ((41, 64, 8, 8, 1000), WHOLE), ((49, 64, 8, 8, 500), WHOLE), ((33, 64, 8, 8, 1600), WHOLE), ((64, 64, 8, 7, 4096), WHOLE), ((64, 16, 16, 33, 200), WHOLE),
])
def test_few_rows_in_two_tiles_read_keys_twice(route, shape, kind):
    r = route(*shape)
    # (a call that the 256-row kernel gets may take either of its forms)
    assert r["kind"] == kind or {r["kind"], kind} == {WHOLE, SHARED}, r


def test_calls_of_the_bits_test_are_shared(route):
    import test_shared_bits_gpu as T
    for shape in T.SHARED_CALLS:
        for causal in (False, True):
            assert route(*shape, causal)["kind"] == SHARED, (shape, causal)


@pytest.mark.parametrize("shape,takes", [((1, 32, 8, 1, 32768), True), ((1, 32, 8, 512, 16384), True),
                                         ((1, 4, 4, 512, 512), False), ((8, 16, 16, 4096, 4096), False)])
def test_memory_taken_for_a_launch_that_fails_is_given_back(lib, shape, takes):
    def steps(refused, region=0):
        log = ctypes.create_string_buffer(8)
        rc = lib.steps(*shape, 1, NCU, refused, region, log)
        return rc, log.value.decode()
    TAKE, MAIN, GIVE = range(3)
    assert steps(-1) == (A.ATTN_OK, "TM" if takes else "M")
    assert steps(MAIN) == (A.ATTN_E_LAUNCH, "TMG" if takes else "M")
    assert steps(TAKE) == ((A.ATTN_E_LAUNCH, "T") if takes else (A.ATTN_OK, "M"))
    assert steps(GIVE)[0] == A.ATTN_OK
    # a launch that has the region takes nothing and gives nothing back
    assert steps(-1, 1) == (A.ATTN_OK, "M") and steps(MAIN, 1) == (A.ATTN_E_LAUNCH, "M")


def test_header_states_the_device_memory_of_the_code_object(lib):
    lib.pool_bytes.restype = ctypes.c_longlong
    text = open(os.path.join(os.path.dirname(HERE), "include", "attn.h")).read()
    stated = re.search(r"(\d+) MiB\s+\*\s+of device memory", text)
    assert stated and int(stated.group(1)) << 20 == lib.pool_bytes()


@pytest.mark.parametrize("shape,causal,kind", [
    ((9, 16, 16, 571, 33965), False, WHOLE), ((8, 4, 4, 1593, 21904), True, WHOLE), ((8, 40, 40, 413, 3398), False, WHOLE),
    ((7, 40, 40, 153, 7606), False, SHARED), ((4, 16, 16, 439, 9822), True, SHARED),        # (far enough ahead all the same)
])
def test_keys_beyond_the_last_cache_are_shared_only_far_ahead(route, shape, causal, kind):
    assert route(*shape, causal)["kind"] == kind


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("shape", [(7, 64, 8, 16, 22685), (9, 12, 3, 26, 27226), (12, 4, 4, 70, 15095), (12, 32, 4, 9, 16765)])
def test_few_rows_against_long_keys_keep_the_smaller_error(route, shape, causal):
    """The split-key kernel rounds its weights against eight running maxima per part, a shared item of 256 rows against one per part, with
    up to 17 % more error, whichever of the two is faster."""
    assert route(*shape, causal)["kind"] == SPLIT


def test_only_the_regions_counters_are_set_back_by_the_launch(lib):
    """A pool unit is another launch's once it is given back, with nothing to order an earlier store to its counters before that launch's
    counts: those are cleared by the launch in front, never behind the last count.  The region's have no launch in front."""
    pool, region = lib.pool_units(), lib.region_units()
    assert [lib.sets_counters_back(u) for u in range(pool + region)] == [0] * pool + [1] * region
    source = open(os.path.join(os.path.dirname(HERE), "paper_2603_24517_amd", "csrc", "attn_fwd.hip")).read()
    stores = re.findall(r".*\b__hip_atomic_store\([^,]*counter.*", source)
    assert len(stores) == 1 and "if (sets_counters_back(unit))" in stores[0], stores


@pytest.mark.parametrize("shape,once,once_null,parts", [
    ((18, 32, 8, 1, 2000), 0, 0, 1), ((9, 16, 16, 7, 3200), 0, 0, 1), ((18, 32, 8, 1, 4050), 0, 0, 1),      # a repeated call finds them in the last cache
    ((18, 16, 16, 1, 1600), 0, 0, 1), ((17, 16, 16, 1, 2000), 0, 0, 1), ((35, 32, 8, 1, 1500), 0, 0, 1),    # nor are they cut into rounds of parts
    ((18, 32, 8, 1, 4150), 1, 1, 1), ((20, 32, 8, 1, 4000), 1, 1, 1), ((40, 32, 8, 1, 2500), 1, 1, 2),
    ((1, 32, 8, 1, 32768), 0, 1, 20), ((16, 32, 8, 1, 4000), 0, 1, 2), ((1, 32, 8, 1, 8192), 0, 0, 10), ((2, 64, 8, 16, 8192), 0, 0, 4),
])
def test_keys_that_the_last_cache_holds_are_not_read_past_it(route, shape, once, once_null, parts):
    r = route(*shape)
    assert (r["kind"], r["once"], r["once_null"], r["wgs"] / r["items"]) == (SPLIT, once, once_null, parts), r


def test_calls_of_the_read_once_test_are(route):
    import test_read_once_gpu as T
    rounds = [route(*shape, causal) for shape in T.ROUNDS for causal in (False, True)]
    assert all(r["kind"] == SPLIT and r["once"] and r["wgs"] > r["items"] for r in rounds), rounds
    assert max(r["items"] for r in rounds) > 512 and max(r["wgs"] for r in rounds) > 1024
    region = [route(*shape, causal) for shape in T.REGION for causal in (False, True)]
    assert all(r["kind"] == SPLIT and not r["once"] and r["once_null"] and r["wgs"] > r["items"] for r in region), region


def test_rounds_of_parts_fit_the_device_memory(lib, route):
    limits = (ctypes.c_longlong * 4)()
    lib.split_limits(limits)
    items, wgs, units, counters = limits
    assert items <= counters
    seen = 0
    for hq, hkv in ((16, 16), (32, 8), (16, 2), (4, 1)):
        for batch in list(range(1, 300, 7)) + [511, 512, 1023, 1024]:
            for keys in (700, 1700, 2811, 5000, 16384, 65537):
                for ncu in (256, 304, 80):
                    r = route(batch, hq, hkv, 1, keys, True, ncu)
                    if r["kind"] == SPLIT and r["wgs"] > r["items"]:
                        seen += r["items"] * 2 > ncu
                        assert r["items"] <= items and r["wgs"] <= wgs and 0 < r["units"] <= units, (batch, hq, hkv, keys, ncu, r)
    assert seen > 200, seen


def _with_flags(tmp_path, flags):
    so = str(tmp_path / "route.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", *flags, "-o", so, os.path.join(HERE, "route_shim.cpp")], check=True)
    shim = ctypes.CDLL(so)

    def call(B, Hq, Hkv, Sq, Skv, causal):
        out = (ctypes.c_longlong * 7)()
        assert shim.route(B, Hq, Hkv, Sq, Skv, int(causal), NCU, out) == A.ATTN_OK
        return dict(zip(("kind", "items", "wgs", "units", "once", "once_null", "kgroups"), out))
    return call


@pytest.mark.parametrize("name", ["softmax_blockmax_always", "softmax_blockmax_vote", "softmax_blockmax_threshold", "no_item_overlap", "lds_prefetch_1",
                                  "lds_prefetch_5"])
def test_small_shapes_of_the_256_row_kernels_variants_reach_it(tmp_path, name):
    """Their switches act in the 256-row kernel alone; the other kernels would pass the parity tests whatever the switch did."""
    import test_variants_gpu as T
    from paper_2603_24517_amd import build
    call = _with_flags(tmp_path, build.VARIANTS[name])
    routes = [call(*shape[:5], causal) for shape in T.SHAPES + T.JUMP_SHAPES for causal in (False, True)]
    assert all(r["kind"] == WHOLE and r["kgroups"] == 0 for r in routes), routes
    assert any(r["items"] > r["wgs"] for r in routes)       # several items per workgroup


def test_calls_that_stand_for_each_kernel_reach_it(tmp_path, route):
    import test_attn_gpu as T
    from paper_2603_24517_amd import build
    import __graft_entry__ as G
    for shapes in (T.EACH_KERNEL, G.SMOKE):
        split, rows, main = (route(*s) for s in shapes)
        assert split["kind"] == SPLIT and rows["kind"] == main["kind"] == WHOLE and rows["kgroups"] != 0 == main["kgroups"]
        assert main["items"] > main["wgs"]
    whole = _with_flags(tmp_path, build.VARIANTS["whole_items"])
    for shape in T.MANY_ITEMS:
        for causal in (False, True):
            r = whole(*shape, causal)
            assert r["kind"] == WHOLE and r["kgroups"] == 0 and r["items"] > 200, (shape, r)
