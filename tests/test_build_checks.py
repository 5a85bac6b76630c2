"""The build's own check of the prefill kernels' register use (host logic, no GPU)."""
from paper_2410_09615_amd.build import compiler_agpr_uses

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
