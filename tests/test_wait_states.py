"""The wait states that gfx950 leaves to the program, in the assembly of this build (no GPU needed)."""
import pytest

from paper_2107_08170_amd import build
from tests import wait_states


@pytest.mark.parametrize("source", build.SOURCES)
def test_inline_assembly_keeps_the_wait_states(tmp_path, source):
    """No instruction of inline assembly reads what an instruction just before it wrote, or the other way round, without the
    wait states between: the compiler inserts those only between instructions that it has made itself."""
    text = build.assembly(source, str(tmp_path / "device.s"))
    kernels = source.endswith("mv_kernels.hip")
    assert ("#ASMSTART" in text) == kernels and (not kernels or "v_readlane_b32" in text)
    wrong = wait_states.violations(text)
    assert not wrong, "\n".join(f"{found} of {need} wait states: {a.line}: {a.text}  ->  {b.line}: {b.text}" for need, found, a, b in wrong[:20])


INLINE = "\t;;#ASMSTART\n\t{}\n\t;;#ASMEND\n"


@pytest.mark.parametrize("before,between,after,found", [
    ("v_readlane_b32 s2, v56, 0", "", "v_mov_b32 v1, s2", True),
    ("v_readlane_b32 s2, v56, 0", "s_nop 0", "v_mov_b32 v1, s2", True),
    ("v_readlane_b32 s2, v56, 0", "s_nop 1", "v_mov_b32 v1, s2", False),
    ("v_readlane_b32 s2, v56, 0", "s_mov_b32 s2, s7", "v_mov_b32 v1, s2", False),
    ("v_readlane_b32 s2, v56, 0", "", "v_mov_b32 v1, s3", False),
    ("v_readlane_b32 s7, v56, 0", "s_nop 3", "global_store_dword v1, v2, s[6:7]", True),
    ("v_readlane_b32 s7, v56, 0", "s_nop 4", "global_store_dword v1, v2, s[6:7]", False),
    ("v_readlane_b32 s7, v56, 0", "s_addc_u32 s7, s7, 0", "global_store_dword v1, v2, s[6:7]", False),
    ("v_cmp_lt_f32_e32 vcc, v1, v2", "s_nop 0", "v_cndmask_b32_e64 v3, 0, 1.0, vcc", True),
    ("v_rcp_f32_e32 v1, v2", "", "v_max_f32 v3, v1, v1", True),
    ("v_rcp_f32_e32 v1, v2", "v_add_f32_e32 v4, v4, v4", "v_max_f32 v3, v1, v1", False),
    ("v_max_f32 v1, v2, v2", "", "v_mov_b32_dpp v3, v1 quad_perm:[1,2,3,3] row_mask:0xf bank_mask:0xf", True),
])
def test_the_scan_finds_what_it_looks_for(before, between, after, found):
    for text in (f"\t{before}\n\t{between}\n" + INLINE.format(after), INLINE.format(before) + f"\t{between}\n\t{after}\n"):
        assert bool(wait_states.violations(text)) == found
    assert not wait_states.violations(f"\t{before}\n\t{between}\n\t{after}\n")        # the compiler's own business
