"""CPU-only: the build refuses assembly in which the compiler uses accumulation registers that a kernel names by itself."""
import pytest

from paper_2602_04879_amd import build

KERNEL = "dppo_gemm_nt_kernel"
ASM = """_Z12other_kernelv:
\tv_accvgpr_write_b32 a0, v1
.Lfunc_end0:
_Z19dppo_gemm_nt_kernelILi0EEvv:
\ts_load_dwordx2 s[0:1], s[4:5], 0x0
\tv_add_u32_e32 v1, v2, v3                ; a4 in a comment
\t;;#ASMSTART
\tv_mfma_f32_16x16x32_bf16 a[0:0x3], v[8:11], v[4:7], 0
\t;;#ASMEND
\tscratch_load_dword v0, off, off
\t;;#ASMSTART
\tv_accvgpr_read_b32 v2, a[0x2]
\t;;#ASMEND
.LBB1_2:
\ts_cbranch_scc1 .LBB1_2
\ts_endpgm
.Lfunc_end1:
amdhsa.kernels:
  - .agpr_count:     4
    .name:           _Z12other_kernelv
    .private_segment_fixed_size: 64
    .vgpr_spill_count: 3
  - .agpr_count:     256
    .name:           _Z19dppo_gemm_nt_kernelILi0EEvv
    .private_segment_fixed_size: 0
    .vgpr_spill_count: 0
amdhsa.version:
  - 1
  - 2
"""


def test_accumulators_in_the_kernels_own_statements_pass():
    build.check_named_accumulators(ASM, KERNEL)


@pytest.mark.parametrize("old,new", [
    ("\tscratch_load_dword v0, off, off", "\tv_accvgpr_write_b32 a7, v0"),                   # a spilled vector register
    ("\tscratch_load_dword v0, off, off", "\tv_accvgpr_mov_b32 a1, a0"),                     # a copy
    ("\tscratch_load_dword v0, off, off", "\tv_accvgpr_read_b32 v0, a255"),
    ("\tscratch_load_dword v0, off, off", "\tglobal_load_dwordx4 a[4:7], v[0:1], off"),
    ("\ts_endpgm", "\tds_read_b64 a[0:1], v3\n\ts_endpgm"),                                 # behind a label inside the kernel
    (".agpr_count:     256", ".agpr_count:     128"),
    (".vgpr_spill_count: 0", ".vgpr_spill_count: 1"),
    (".private_segment_fixed_size: 0", ".private_segment_fixed_size: 16"),
    ("_Z19dppo_gemm_nt_kernelILi0EEvv:", "_Z5renamev:"),                                     # a body without its entry is not read
    ("    .name:           _Z19dppo_gemm_nt_kernelILi0EEvv", "    .name:           _Z5renamev"),
])
def test_accumulators_used_by_the_compiler_are_refused(old, new):
    assert ASM.count(old) == 1
    with pytest.raises(RuntimeError, match="accumulation registers"):
        build.check_named_accumulators(ASM.replace(old, new), KERNEL)


def test_no_kernel_of_that_name_is_refused():
    with pytest.raises(RuntimeError, match="0 bodies"):
        build.check_named_accumulators(ASM, "dppo_gone_kernel")


def test_every_source_that_names_accumulators_is_looked_through():
    named = [s for s in build.sources() if "DPPO_ALL_ACCUMULATORS()" in open(s).read()]
    assert [s.rsplit("/", 1)[1] for s in named] == list(build.NAMED_ACCUMULATORS)
