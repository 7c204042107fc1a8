"""The built device code: no matrix instruction reads a register sooner after a vector write than the hardware allows (the
compiler does not see writes in inline assembly, so nothing else would notice), and no kernel that counts its outstanding
memory operations by hand may spill registers unnoticed."""
import os
import re

from paper_2305_14152_amd import build, peqa

LISTING = """
0000000000001000 <kernel>:
	v_and_or_b32 v9, v1, s2, v3                                // 000000001000: 00000000
	s_nop 0                                                    // 000000001004: 00000000
	v_mfma_f32_16x16x32_bf16 v[20:23], v[4:7], v[8:11], v[20:23]// 000000001008: 00000000 00000000
	v_mov_b32_e32 v14, 0                                       // 000000001010: 00000000
	s_nop 1                                                    // 000000001014: 00000000
	v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[12:15], a[0:3]  // 000000001018: 00000000 00000000
	v_lshrrev_b32_e32 v4, 3, v5                                // 000000001020: 00000000
	s_cbranch_scc1 65530                                       // 000000001024: 00000000 <kernel+0x8>
	ds_read_b128 v[8:11], v2                                   // 000000001028: 00000000 00000000
	v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], a[0:3] // 000000001030: 00000000 00000000
	s_endpgm                                                   // 000000001038: 00000000
"""


def test_the_check_sees_what_it_is_for():
    """One wait state in straight-line code; one over a backward branch; two, and writes of other registers, pass."""
    found = build.early_matrix_reads(LISTING)
    assert len(found) == 2
    assert "1008 reads what v_and_or_b32 at 1000 wrote, after 1 wait" in found[0]
    assert "1008 reads what v_lshrrev_b32_e32 at 1020 wrote, after 1 wait" in found[1]


def test_no_matrix_instruction_reads_too_early():
    peqa.lib()
    assert os.path.exists(build.LIB)
    listings = build.device_listings(build.LIB)
    assert sum("v_mfma" in text for text in listings) >= 3           # the tiled, the token and the T <= 16 contraction
    assert [b for text in listings for b in build.early_matrix_reads(text)] == []


def test_spills_are_refused_in_every_kernel_that_counts():
    """Every kernel with a ring of DMAs (dynamic LDS and matrix instructions) is among those the build looks at."""
    peqa.lib()
    kernels = set()
    for text in build.device_listings(build.LIB):
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            if "global_load_lds" in part:
                kernels.add(re.match(r"[0-9a-f]+ <(.+)>:", part).group(1))
    assert len(kernels) >= 20
    remark = "f.hip:1:1: remark: Function Name: %s [-R]\nf.hip:1:1: remark:     ScratchSize [bytes/lane]: 8 [-R]\n"
    assert [k for k in kernels if not build.check_no_scratch(remark % k)] == []
