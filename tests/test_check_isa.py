"""Host logic of the build's assembly checks (paper_2603_02188_amd/check_isa.py)."""
from paper_2603_02188_amd.check_isa import find_overlaps, find_reserved_acc_uses, find_scratch_in_loops

ASM = """
_ZN4mlra12_GLOBAL__N_118decode_mfma_kernelILi6ELi0EEEvNS_9mfma_tile10MfmaParamsE:
\tv_mov_b32_e32 v1, v0
\t;;#ASMSTART
\tv_mfma_f32_32x32x16_bf16 a[0:15], v[2:5], v[6:9], a[0:15]
\t;;#ASMEND
.LBB0_1:
\tv_accvgpr_write_b32 a200, v3
\tv_accvgpr_read_b32 v4, a135
\tds_read_b128 a[140:143], v7
\tv_accvgpr_mov_b32 a120, a210
\ts_endpgm
_ZN4mlra5otherEv:
\tv_accvgpr_write_b32 a3, v3
"""


def test_reserved_accumulation_registers_outside_inline_asm_are_reported():
    bad = find_reserved_acc_uses(ASM, r"decode_mfma_kernel", 136)
    assert [text for _, text in bad] == ["v_accvgpr_read_b32 v4, a135", "v_accvgpr_mov_b32 a120, a210"]
    # nothing reserved, nothing reported; another kernel's registers are its own
    assert find_reserved_acc_uses(ASM, r"decode_mfma_kernel", 0) == []
    assert find_reserved_acc_uses(ASM, r"no_such_kernel", 136) == []


def test_mfma_destination_over_a_source_is_reported():
    ok = "\tv_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], a[0:3], v[0:15]\n"
    bad = "\tv_mfma_f32_32x32x16_bf16 v[0:15], v[12:15], a[0:3], 0\n"
    narrow = "\tv_mfma_f32_16x16x32_bf16 v[0:3], v[0:3], v[4:7], 0\n"
    assert find_overlaps(ok) == [] and find_overlaps(narrow) == []
    assert len(find_overlaps(bad)) == 1


def test_scratch_accesses_in_a_loop_are_reported():
    asm = """
_ZN4mlra15mla_mfma_kernelILi2EEEv: ; @mla
\tscratch_store_dword off, v1, off ; 4-byte Folded Spill
.LBB0_1:                                ; =>This Inner Loop Header: Depth=1
\tds_read_b128 v[0:3], v4
; %%bb.2:                               ;   in Loop: Header=BB0_1 Depth=1
\tglobal_load_lds_dwordx4 v7, s[0:1]
.LBB0_3:                                ;   in Loop: Header=BB0_1 Depth=1
\t%s
\ts_cbranch_scc1 .LBB0_1
; %%bb.4:
\tscratch_load_dword v1, off, off ; 4-byte Folded Reload
\ts_endpgm
_ZN4mlra5otherEv:
.LBB1_1:                                ; =>This Inner Loop Header: Depth=1
\tscratch_load_dword v1, off, off
"""
    clean, spill = asm % "v_mov_b32_e32 v1, v2", asm % "scratch_load_dword v9, off, off offset:4"
    assert find_scratch_in_loops(clean, r"mla_mfma_kernel") == []
    assert [text for _, text in find_scratch_in_loops(spill, r"mla_mfma_kernel")] == ["scratch_load_dword v9, off, off offset:4"]
