"""Build the gfx950 shared libraries in-tree with hipcc.

    python -m paper_2603_24517_amd.build            the attention library (C ABI of include/attn.h) and the binding's native part
    python -m paper_2603_24517_amd.build --all      that, the measurement-aid library (include/attn_probe.h)
                                                     and every variant of the attention kernel

The variants are builds of the same source with one compile-time switch each (see the heads of
csrc/attn_fwd.hip and csrc/attn_route.h); they exist to measure the shipped choices against their alternatives and are
never loaded by the product path.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "attn_fwd.hip")
LIB = os.path.join(HERE, "libattn_mi355x.so")
PROBE_SRC = os.path.join(HERE, "csrc", "attn_probe.hip")
PROBE_LIB = os.path.join(HERE, "libattn_probe.so")
VARIANT_DIR = os.path.join(HERE, "variants")
CALL_SRC = os.path.join(HERE, "csrc", "attn_call.cpp")
CALL_LIB = os.path.join(HERE, "_attn_call.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed FP32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

# every launch through the 256-row kernel, in whole items: for switches that act there
ALL_256_ROWS = ["-DATTN_SMALL_PATH=0", "-DATTN_SHARE=0"]
# name -> extra compiler flags; what each stands for is described where the switches are defined
VARIANTS = {
    "softmax_blockmax_always": ["-DATTN_SOFTMAX=1", *ALL_256_ROWS],
    "softmax_blockmax_vote": ["-DATTN_SOFTMAX=2", *ALL_256_ROWS],
    "softmax_blockmax_threshold": ["-DATTN_SOFTMAX=3", *ALL_256_ROWS],
    "no_item_overlap": ["-DATTN_ITEM_OVERLAP=0", *ALL_256_ROWS],
    # every launch through the 256-row kernel / every launch through the split-key kernel for small problems
    "no_small_path": ["-DATTN_SMALL_PATH=0"],
    "always_small_path": ["-DATTN_SMALL_PATH=2"],
    # no device memory for partial results (what a launch does that finds it in use)
    "no_pool": ["-DATTN_POOL=0"],
    # the 256-row kernel with whole items only / with items shared among workgroups wherever the device memory for it
    # serves / the same, finding that memory in use
    "whole_items": ["-DATTN_SHARE=0"],
    "always_share": ["-DATTN_SHARE=2", "-DATTN_SMALL_PATH=0"],
    "always_share_no_pool": ["-DATTN_SHARE=2", "-DATTN_SMALL_PATH=0", "-DATTN_POOL=0"],
    # every launch through the kernel with workgroups of four wavefronts, in items of 128 rows / of 64
    "always_rows128": ["-DATTN_ROWS=2"],
    "always_rows64": ["-DATTN_ROWS=3"],
    "lds_prefetch_1": ["-DATTN_LDS_PREFETCH=1", *ALL_256_ROWS],
    "lds_prefetch_5": ["-DATTN_LDS_PREFETCH=5", *ALL_256_ROWS],
    # the shipped kernel plus clock stamps of its first workgroup (exports attn_clocks_read as well)
    "clocks": ["-DATTN_CLOCKS"],
    # the same plus cycle sums per phase of one work item (exports attn_phases_read as well)
    "phases": ["-DATTN_CLOCKS=2"],
}


def variant_path(name):
    return os.path.join(VARIANT_DIR, f"libattn_{name}.so")


def _hipcc(flags, out, src, verbose):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *flags, "-o", out, src]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return out


def build_library(extra_flags=(), out=LIB, verbose=False):
    return _hipcc(list(extra_flags), out, SRC, verbose)


def build_probe(verbose=False):
    return _hipcc([], PROBE_LIB, PROBE_SRC, verbose)


def build_call(verbose=False):
    """The Python binding's native part: host code against torch's headers and libraries."""
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f"-I{root}/include", f"-I{root}/include/torch/csrc/api/include",
           "-I/opt/rocm/include", f"-I{sysconfig.get_paths()['include']}", "-o", CALL_LIB, CALL_SRC, f"-L{root}/lib", f"-Wl,-rpath,{root}/lib",
           "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return CALL_LIB


def build_variants(names=None, verbose=False):
    os.makedirs(VARIANT_DIR, exist_ok=True)
    return [build_library(VARIANTS[n], variant_path(n), verbose) for n in (names or VARIANTS)]


def build_all(verbose=False, jobs=4):
    """Everything, a few compilations at a time (each is a single-threaded hipcc run of about ten seconds)."""
    from concurrent.futures import ThreadPoolExecutor
    os.makedirs(VARIANT_DIR, exist_ok=True)
    tasks = [lambda: build_call(verbose=verbose), lambda: build_library(verbose=verbose), lambda: build_probe(verbose=verbose)]
    tasks += [lambda n=n: build_library(VARIANTS[n], variant_path(n), verbose) for n in VARIANTS]
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        for f in [pool.submit(t) for t in tasks]:
            f.result()


if __name__ == "__main__":
    if sys.argv[1:] == ["--all"]:
        build_all(verbose=True)
    else:
        print(build_library(extra_flags=sys.argv[1:], verbose=True))
        print(build_call(verbose=True))
