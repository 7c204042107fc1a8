"""The built device code: no instruction reads a register sooner after it was written than the hardware allows (the compiler
does not see reads and writes in inline assembly, so nothing else would notice), and no kernel that counts its outstanding
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
	v_readfirstlane_b32 s5, v5                                 // 000000001038: 00000000
	v_readfirstlane_b32 s8, v6                                 // 00000000103C: 00000000
	s_mov_b32 m0, s11                                          // 000000001040: 00000000
	s_nop 2                                                    // 000000001044: 00000000
	global_load_lds_dwordx4 v82, s[4:5]                        // 000000001048: 00000000 00000000
	global_load_lds_dwordx4 v82, s[8:9]                        // 000000001050: 00000000 00000000
	v_mov_b32_e32 v1, v2                                       // 000000001058: 00000000
	s_nop 0                                                    // 00000000105C: 00000000
	v_mov_b32_dpp v3, v1 quad_perm:[1,0,3,2]                   // 000000001060: 00000000 00000000
	s_endpgm                                                   // 000000001068: 00000000
"""


def test_the_check_sees_what_it_is_for():
    """Matrix operands: one wait state of two, in straight-line code and over a backward branch.  A lane exchange: one of two.
    A memory instruction's scalar address: five, and four once the s_nop is shorter.  What waits long enough passes."""
    found = build.early_reads(LISTING)
    expected = ["1008 reads what v_and_or_b32 at 1000 wrote, after 1", "1008 reads what v_lshrrev_b32_e32 at 1020 wrote, after 1",
                "1060 reads what v_mov_b32_e32 at 1058 wrote, after 1"]
    assert len(found) == len(expected), found
    for text, want in zip(found, expected):
        assert want in text
    closer = build.early_reads(LISTING.replace("s_nop 2 ", "s_nop 1 "))
    assert [f for f in closer if f not in found and "1048 reads what v_readfirstlane_b32 at 1038 wrote, after 4" in f]


def test_no_instruction_reads_too_early():
    peqa.lib()
    assert os.path.exists(build.LIB)
    listings = build.device_listings(build.LIB)
    assert sum("v_mfma" in text for text in listings) >= 3           # the tiled, the token and the T <= 16 contraction
    assert [b for text in listings for b in build.early_reads(text)] == []


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


def test_three_workgroups_of_64_row_tiles_fit_a_unit():
    """Per-channel tiles of 64 rows have 48 KB of LDS, so that three four-wave workgroups fit a unit if their kernel, with whatever
    side work is compiled into it, takes no more than a third of a SIMD's 512 registers (in steps of eight)."""
    peqa.lib()
    found = {name: regs for name, regs in build.kernel_registers(build.LIB).items()
             if re.search(r"gemm_multi_kernelILi[34]ELin1ELi4E|gemm_bwd_pair_kernelILi[34]ELi4E|gemm_kernelILi[34]ELi[012]ELb0ELi1ELi4E", name)}
    assert len(found) == 10, found
    assert {name: regs for name, regs in found.items() if regs > 512 // 3 // 8 * 8} == {}


def test_memory_is_read_and_written_by_global_instructions():
    """FLAT loads and stores, which the compiler takes for pointers whose memory it cannot tell, count as LDS operations too: it waits
    for every operation in flight before the use of what one brings."""
    peqa.lib()
    assert [line for text in build.device_listings(build.LIB) for line in text.splitlines()
            if re.match(r"\s+flat_(load|store|atomic)", line)] == []


def test_token_tiles_wait_for_what_they_use_only():
    """The loop of the token contraction, in every kernel that has it: operands by global loads, and no wait that empties the
    memory queue (which the compiler puts where it believes a FLAT operation is pending, and which drains the ring)."""
    peqa.lib()
    loops = {}
    for text in build.device_listings(build.LIB):
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            name = re.match(r"[0-9a-f]+ <(.+)>:", part)
            if not name or "dw_" not in name.group(1):
                continue
            code = [line.split("//")[0].strip() for line in part.splitlines()[1:]]
            barriers = [i for i, op in enumerate(code) if op.startswith("s_barrier")]
            for a, b in zip(barriers, barriers[1:]):
                step = code[a:b]
                if sum(op.startswith("v_mfma") for op in step) == 32 and sum("global_load_lds" in op for op in step) == 2 and \
                        sum("s_waitcnt vmcnt(18)" in op for op in step) == 1:
                    assert not [op for op in step if op.startswith("flat_") or "vmcnt(0)" in op], name.group(1)
                    assert sum(op.startswith("global_load_dwordx4") for op in step) == 4
                    loops[name.group(1)] = loops.get(name.group(1), 0) + 1
    assert len(loops) == 12 and set(loops.values()) == {2}, loops   # alone and of several layers, beside dX of four heights; 3, 4 bits
