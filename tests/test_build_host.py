"""The build refuses a forward kernel in whose named accumulation registers the compiler has a value of its own (no GPU)."""
import pytest

from paper_2509_01085_amd.build import foreign_accumulators

ASSEMBLY = """_ZN3bsa15fwd_walk_kernelILi64ELi0EEEvNS_7FwdArgsE: ; @_ZN3bsa15fwd_walk_kernelILi64ELi0EEEvNS_7FwdArgsE
\tv_mov_b32_e32 v1, v2 ; a name like a1
\ts_cbranch_scc1 .LBB0_2
{0}
\t;;#ASMSTART
\tv_mfma_f32_32x32x16_bf16 a[0:15], v[2:5], v[6:9], a[0:15]
{1}
\t;;#ASMEND
\tglobal_load_dwordx4 v[2:5], v0, s[2:3] offset:16
.Lfunc_end0:
{2}
_ZN3bsa18fwd_combine_kernelILi64ELi0EEEvNS_4GeomE:
{3}
.Lfunc_end1:
"""
TOUCHES = ["\tv_accvgpr_write_b32 a17, v3", "\tv_mfma_f32_32x32x16_bf16 a[16:31], v[2:5], v[6:9], 0", "\tscratch_store_dword off, a3, off"]


@pytest.mark.parametrize("line", TOUCHES)
def test_an_instruction_of_the_compilers_is_found(line):
    found = lambda at: foreign_accumulators(ASSEMBLY.format(*[line if k == at else "" for k in range(4)]), "fwd_walk_kernel")
    assert found(0) == ([line.strip()], 1)
    for elsewhere in (1, 2, 3):  # inline assembly, data, another kernel
        assert found(elsewhere) == ([], 1)
