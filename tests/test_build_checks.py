"""The build's own check of the prefill kernels' register use (host logic, no GPU)."""
from paper_2410_09615_amd.build import compiler_agpr_uses, lane_reads_too_early

ASM = """\t.text
_ZN4slim5cleanE:
\ts_load_dwordx2 s[0:1], s[4:5], 0x0
\t;;#ASMSTART
\tv_accvgpr_write_b32 a[5], v1
\tv_mfma_f32_32x32x16_f16 a[0:15], v[2:5], v[6:9], a[0:15]
\tv_smfmac_f32_32x32x32_f16 a[16:31], v[2:5], v[6:13], v14 abid:1
\tv_accvgpr_read_b32 v3, a[17]
\t;;#ASMEND
\tbuffer_load_dwordx4 v[24:27], v26, s[20:23], 0 offen ; a5 in a comment does not count
\ts_endpgm
.Lfunc_end0:
_ZN4slim6parkedE:
\tv_accvgpr_write_b32 a14, v30
\tbuffer_load_dwordx4 a[24:27], v26, s[20:23], 0 offen
\tv_mfma_f32_32x32x16_f16 a[0:15], v[2:5], v[6:9], a[0:15]
\tv_accvgpr_read_b32 v21, a7
\ts_endpgm
"""


def test_compiler_uses_of_accumulation_registers_are_found():
    """Kernels that address the accumulation registers by number lose whatever the register allocator
    parks there (a store index, once: an out-of-bounds store).  The build reads the device assembly and
    refuses such a library; here the reader itself, on a clean kernel and on one with three parked values."""
    assert compiler_agpr_uses(ASM) == {"_ZN4slim6parkedE": 3}


LANES = """_ZN4slim5cleanE:
\tv_mov_b32_e32 v9, v64
\tv_mov_b32_e32 v3, v7
\t;;#ASMSTART
\tv_mul_f32 v4, v5, v6
\tv_mul_f32 v5, v4, v6
\tv_fmac_f32_dpp v9, v9, v4 row_newbcast:0 row_mask:0xf bank_mask:0xf
\tv_fmac_f32_dpp v8, v8, v4 row_newbcast:0 row_mask:0xf bank_mask:0xf
\tv_permlane16_swap_b32 v2, v3
\ts_nop 1
\tv_permlane32_swap_b32 v2, v3
\t;;#ASMEND
\ts_nop 1
\tv_mov_b32_dpp v7, v2 row_newbcast:0 row_mask:0xf bank_mask:0xf bound_ctrl:1
\ts_endpgm
_ZN4slim4copyE:
\tv_mov_b32_e32 v9, v64
\t;;#ASMSTART
\ts_nop 0
\tv_fmac_f32_dpp v9, v9, v7 row_newbcast:0 row_mask:0xf bank_mask:0xf
\tv_fmac_f32_dpp v8, v8, v7 row_newbcast:0 row_mask:0xf bank_mask:0xf
\t;;#ASMEND
\tv_mov_b32_dpp v7, v8 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf
\ts_endpgm
_ZN4slim5startE:
\ts_nop 7
\t;;#ASMSTART
\tv_fmac_f32_dpp v53, v53, v7 row_newbcast:1 row_mask:0xf bank_mask:0xf
\t;;#ASMEND
\ts_endpgm
"""


def test_reads_of_other_lanes_right_after_a_write_are_found():
    """A register that another lane reads has to have been written two wait states before, and asm cannot know what the compiler
    places before it: a copy right before a block that begins with such a read, the read itself, and one right behind the
    block are found, in a kernel each; blocks that begin with two other instructions are not."""
    assert lane_reads_too_early(LANES) == {"_ZN4slim4copyE": 2, "_ZN4slim5startE": 1}


def test_counts_that_hand_results_over_order_memory():
    """A workgroup that learns from a count that others have ended reads what they stored: where the result of an
    atomic add is compared, the add releases what came before it, and an acquire follows before anything is read."""
    import glob
    import os
    import re
    from paper_2410_09615_amd.build import CSRC
    found = 0
    for path in glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h")):
        with open(path) as fh:
            text = fh.read()
        for call in re.finditer(r"__hip_atomic_fetch_add\(((?:[^();]|\([^()]*\))*)\)\s*==", text):
            found += 1
            after = text[call.end():].split(";")[0]
            assert "__ATOMIC_RELEASE" in call.group(1) and "fence(__ATOMIC_ACQUIRE" in after, (path, call.group(0))
    assert found == 2


def test_asm_that_writes_m0_says_so():
    """The compiler keeps values of its own in m0 (indexed registers, its own loads to LDS): asm that writes it
    names it among what it clobbers."""
    import glob
    import os
    import re
    from paper_2410_09615_amd.build import CSRC
    found = 0
    for path in glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h")):
        with open(path) as fh:
            text = fh.read()
        for block in re.findall(r'asm volatile\(\s*"[^;]*;', text):
            if re.search(r'"[^"]*\bs_mov_b32 m0\b', block):
                found += 1
                assert '"m0"' in block.split(":")[-1], (path, block)
    assert found == 2
