"""The build step that checks the generated code of the four-wave GEMM (csrc/check_w4_asm.py), on synthetic
assembly: the kernel counts its own memory waits, so the checker has to notice a register that is used while
its load is still in flight, a scratch access inside the loop and a load issued behind the loop."""
import importlib.util
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_03283_amd", "csrc")


def _checker():
    spec = importlib.util.spec_from_file_location("check_w4_asm", os.path.join(CSRC, "check_w4_asm.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _kernel(loop_extra="", first_wait="s_waitcnt vmcnt(1)", tail_extra=""):
    """A miniature of the kernel's shape: two loads in flight per register set, five barriers, a drain."""
    return f"""
\tbuffer_load_dwordx4 v[0:3], v20, s[0:3], s8 offen
\tbuffer_load_dwordx4 v[4:7], v20, s[0:3], s9 offen
\ts_waitcnt vmcnt(1)
\tds_write_b128 v21, v[0:3]
\tbuffer_load_dwordx4 v[0:3], v20, s[0:3], s8 offen
\ts_barrier
.LBB0_1:
\t{first_wait}
\tds_write_b128 v21, v[4:7]
\tbuffer_load_dwordx4 v[4:7], v20, s[0:3], s9 offen
\tv_mfma_f32_32x32x16_bf16 a[0:15], v[8:11], v[12:15], a[0:15]
{loop_extra}
\ts_barrier
\ts_waitcnt vmcnt(1)
\tds_write_b128 v21, v[0:3]
\tbuffer_load_dwordx4 v[0:3], v20, s[0:3], s8 offen
\ts_barrier
\ts_cbranch_scc1 .LBB0_1
\ts_waitcnt vmcnt(0)
\ts_branch .LBB0_1
.LBB0_2:
\tds_write_b128 v21, v[4:7]
\ts_barrier
\tv_mov_b32_e32 v0, v30
{tail_extra}
\ts_barrier
\tglobal_store_dword v[40:41], v0, off
\ts_endpgm
""".split("\n")


def test_clean_kernel_passes():
    ok, msg = _checker().check("k", _kernel())
    assert ok, msg


def test_register_used_before_its_load_is_waited_for():
    ok, msg = _checker().check("k", _kernel(first_wait="s_waitcnt vmcnt(2)"))
    assert not ok and "ds_write_b128 v21, v[4:7]" in msg


def test_compiler_copy_of_a_register_in_flight():
    ok, msg = _checker().check("k", _kernel(loop_extra="\tv_mov_b32_e32 v31, v5"))
    assert not ok and "v_mov_b32_e32 v31, v5" in msg


def test_scratch_access_inside_the_loop():
    ok, msg = _checker().check("k", _kernel(loop_extra="\tscratch_store_dword off, v30, off"))
    assert not ok and "scratch_store_dword" in msg


def test_load_behind_the_loop():
    ok, msg = _checker().check("k", _kernel(tail_extra="\tbuffer_load_dwordx4 v[4:7], v20, s[0:3], s9 offen"))
    assert not ok and "loads issued behind the loop" in msg


@pytest.mark.parametrize("extra", ["\ts_barrier", "\ts_barrier\n\ts_nop 15\n\tbuffer_load_dwordx4 v[4:7], v20, s[0:3], s9 offen"])
def test_barrier_behind_the_loop(extra):
    """The kernel has five barriers; with another one the positions the checks hang on may be others than meant, and
    what follows it must not go unchecked."""
    ok, msg = _checker().check("k", "\n".join(_kernel()).replace("\tglobal_store", extra + "\n\tglobal_store").split("\n"))
    assert not ok and "expected 5 barriers" in msg


def _loop(n, first_wait="s_waitcnt vmcnt(1)", phase="", outside="", before_exit="", tail="", drain="\ts_waitcnt vmcnt(0)"):
    """One main loop as the compiler lays it out: prologue, two phases, the skipped wait for all loads, the loop's test, the tail; the second phase
    leaves for a block out of line (see _two_loops)."""
    return f"""
.LBB0_{n}0:
\tbuffer_load_dwordx4 v[0:3], v20, s[0:3], s8 offen
\tbuffer_load_dwordx4 v[4:7], v20, s[0:3], s9 offen
\ts_waitcnt vmcnt(1)
\tds_write_b128 v21, v[0:3]
\tbuffer_load_dwordx4 v[0:3], v20, s[0:3], s8 offen
\ts_barrier
\ts_branch .LBB0_{n}2
.LBB0_{n}1:
\ts_cmp_lt_u32 s59, s54
\ts_cbranch_scc0 .LBB0_{n}4
.LBB0_{n}2:
\t{first_wait}
\tds_write_b128 v21, v[4:7]
\tbuffer_load_dwordx4 v[4:7], v20, s[0:3], s9 offen
\ts_barrier
{phase}
\ts_cbranch_scc0 .LBB0_{n}6
.LBB0_{n}3:
\ts_waitcnt vmcnt(1)
\tds_write_b128 v21, v[0:3]
\tbuffer_load_dwordx4 v[0:3], v20, s[0:3], s8 offen
\ts_barrier
\ts_cbranch_scc1 .LBB0_{n}1
{drain}
\ts_branch .LBB0_{n}1
.LBB0_{n}4:
{before_exit}
\tds_write_b128 v21, v[4:7]
\ts_barrier
\tv_mov_b32_e32 v0, v30
{tail}
\ts_barrier
\ts_branch .LBB0_9
.LBB0_{n}6:
\ts_min_i32 s12, s13, s14
{outside}
\ts_branch .LBB0_{n}3
"""


def _two_loops(first=None, second=None, end="", behind_end="", entry="\ts_cbranch_scc1 .LBB0_20"):
    a, b = _loop(1, **(first or {})), _loop(2, **(second or {}))
    return f"""
\ts_load_dwordx4 s[0:3], s[4:5], 0x0
{entry}
{a}{b}
.LBB0_9:
{end}
\ts_nop 15
\ts_nop 15
\tbuffer_load_dwordx4 v[8:11], v20, s[0:3], 0 offen
\ts_waitcnt vmcnt(0)
\tbuffer_store_dwordx4 v[8:11], v20, s[0:3], 0 offen
\ts_endpgm
{behind_end}
""".split("\n")


NT = "kernelILi0ELi0EEE"


def test_two_clean_loops_pass():
    ok, msg = _checker().check(NT, _two_loops())
    assert ok and "2 main loop(s)" in msg, msg


@pytest.mark.parametrize("loop", ["first", "second"])
@pytest.mark.parametrize("fault,found", [
    (dict(first_wait="s_waitcnt vmcnt(2)"), "ds_write_b128 v21, v[4:7]"),                       # a wait too short
    (dict(phase="\tv_mov_b32_e32 v31, v5"), "v_mov_b32_e32 v31, v5"),                           # a register in flight named in the loop
    (dict(phase="\tscratch_store_dword off, v30, off"), "scratch_store_dword"),
    (dict(outside="\tv_add_u32_e32 v2, v30, v31"), "v_add_u32_e32 v2, v30, v31"),               # ... in a block out of line
    (dict(outside="\tscratch_load_dword v40, off, off"), "scratch_load_dword"),
    (dict(before_exit="\tbuffer_load_dwordx4 v[4:7], v20, s[0:3], s9 offen"), "loads issued behind the loop"),
    (dict(tail="\tbuffer_load_dwordx4 v[4:7], v20, s[0:3], s9 offen"), "loads issued behind the loop"),
    (dict(drain="\tv_nop"), "no vmcnt(0) drain"),
])
def test_faults_are_found_in_either_loop(loop, fault, found):
    ok, msg = _checker().check(NT, _two_loops(**{loop: fault}))
    assert not ok and found in msg, msg


def test_load_in_front_of_the_epilogue():
    ok, msg = _checker().check(NT, _two_loops(end="\tbuffer_load_dwordx4 v[60:63], v20, s[0:3], s9 offen"))
    assert not ok and "loads issued behind the loop" in msg and "loads in flight at the epilogue" in msg, msg


def test_block_reached_by_a_far_jump_behind_the_end():
    jump = """\ts_getpc_b64 s[98:99]
.Lpost_getpc0:
\ts_add_u32 s98, s98, (.LBB0_30-.Lpost_getpc0)&4294967295
\ts_addc_u32 s99, s99, (.LBB0_30-.Lpost_getpc0)>>32
\ts_setpc_b64 s[98:99]"""
    for use, good in (("v_mov_b32_e32 v41, v42", True), ("v_mov_b32_e32 v41, v6", False)):
        ok, msg = _checker().check(NT, _two_loops(second=dict(outside=jump), behind_end=f".LBB0_30:\n\t{use}\n\ts_branch .LBB0_23"))
        assert ok == good and (good or use in msg), msg
    ok, msg = _checker().check(NT, _two_loops(second=dict(outside="\ts_setpc_b64 s[98:99]")))
    assert not ok and "without a known target" in msg


def test_the_nt_kernel_has_two_loops():
    """One loop missing, or two in a kernel of one."""
    ok, msg = _checker().check(NT, _kernel())
    assert not ok and "expected 5 barriers" in msg
    ok, msg = _checker().check("kernelILi0ELi1EEE", _two_loops())
    assert not ok and "expected 5 barriers" in msg


def test_generated_code_of_the_built_library_passes():
    asm = os.path.join(ROOT, "paper_2510_03283_amd", "_build", "gemm-hip-amdgcn-amd-amdhsa-gfx950.s")
    if not os.path.exists(asm):
        pytest.skip("library not built in this tree")
    assert _checker().main(asm) == 0


@pytest.mark.parametrize("source", sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h")) and f not in ("gemm.hip", "gemm_w4.h")))
def test_reads_in_asm_end_with_their_wait(source):
    """The compiler takes the outputs of a block of asm as written when the block ends, and may copy or overwrite them
    there; a read still in flight has to be waited for inside.  (The two sources left out count their waits.)"""
    text = open(os.path.join(CSRC, source)).read()
    blocks = [re.findall(r'"((?:[^"\\]|\\.)*)"', b.split("\" :")[0] + '"') for b in re.findall(r"\basm\b[^;]*;", text)]
    for b in ("".join(parts) for parts in blocks):
        if re.search(r"ds_read|buffer_load|global_load|flat_load", b):
            assert "s_waitcnt" in b[max(b.rfind("ds_read"), b.rfind("_load")):], b
