"""The built code objects keep every kernel inside the register file and out of scratch memory.

The key-block loop counts its own outstanding tile loads (s_waitcnt vmcnt(n) written by hand); a
register spill would put reloads of the compiler's own into that loop, each behind a wait for every
tile request in flight, so "no scratch, no spilled vector register" is a rule of the shipped library
and of every variant that the GPU tests run.  Read from the metadata notes of the code object."""
import pytest

from paper_2603_24517_amd import build as B
from paper_2603_24517_amd import codeobj

LIBS = [("shipped", B.LIB)] + [(n, B.variant_path(n)) for n in B.VARIANTS]


@pytest.mark.parametrize("name,path", LIBS, ids=[n for n, _ in LIBS])
def test_attention_kernels_have_no_scratch_and_fit_the_register_file(name, path):
    meta = codeobj.kernel_metadata(path)
    # kernel, its forms and the threads that it is launched with: 256-row (masked or not, whole or shared items), rows (items of 128, of 64), split-key (shared
    # items or not)
    kinds = [("attn_fwd_kernelI", 4, 512), ("attn_fwd_kernel_rowsI", 2, 256), ("attn_fwd_split_kernelI", 2, 512)]
    assert len(meta) == sum(n for _, n, _ in kinds), sorted(meta)
    for kind, n, threads in kinds:
        kernels = {k: f for k, f in meta.items() if kind in k}
        assert len(kernels) == n, (kind, sorted(meta))
        for k, f in kernels.items():
            assert f["private_segment_fixed_size"] == 0, (name, k, f)
            assert f["vgpr_spill_count"] == 0, (name, k, f)
            # two wavefronts per SIMD: one workgroup of 512 threads on a compute unit, or two of 256
            assert f["vgpr_count"] + f.get("agpr_count", 0) <= 256, (name, k, f)
            assert f["group_segment_fixed_size"] == 0, (name, k, f)                 # LDS is dynamic
            assert f["max_flat_workgroup_size"] == threads, (name, k, f)


def test_probe_kernels_have_no_scratch():
    meta = codeobj.kernel_metadata(B.PROBE_LIB)
    assert len(meta) == 8
    for k, f in meta.items():
        assert f["private_segment_fixed_size"] == 0 and f["vgpr_spill_count"] == 0, (k, f)
        assert f["vgpr_count"] + f.get("agpr_count", 0) <= 128, (k, f)         # up to four wavefronts per SIMD
