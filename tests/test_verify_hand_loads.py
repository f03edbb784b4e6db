"""The build's check of hand-issued loads in the generated code, on small pieces of assembly text."""
import importlib.util
import os

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
_spec = importlib.util.spec_from_file_location(
    "verify_hand_loads", os.path.join(HERE, "..", "paper_2506_04642_amd", "verify_hand_loads.py"))
v = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(v)

HEAD = "_ZN6tadakv24decode_split_mfma_kernelILi8EEEvNS_10DecodeArgsE:\n"
TAIL = "\ts_endpgm\n.Lfunc_end0:\n"


def kernel(body):
    return HEAD + body + TAIL


GOOD = kernel("""
	;;#ASMSTART
	global_load_dwordx4 a[0:3], v[28:29], off ; by hand
	;;#ASMEND
	v_add_u32_e32 v4, v5, v6
	;;#ASMSTART
	s_waitcnt vmcnt(18)
	;;#ASMEND
	;;#ASMSTART
	; by hand a[0:3]
	;;#ASMEND
	v_accvgpr_read_b32 v10, a0
	;;#ASMSTART
	ds_read_b128 v[40:43], v7 offset:64
	;;#ASMEND
	v_add_u32_e32 v4, v5, v6
	;;#ASMSTART
	s_waitcnt lgkmcnt(0)
	;;#ASMEND
	v_mov_b32_e32 v9, v40
""")


def test_untouched_destinations_pass():
    problems, kernels, n, nl = v.check_text(GOOD)
    assert problems == [] and kernels == 1 and n == 1 and nl == 1


def test_a_copy_before_the_hand_over_is_found():
    # the destination is copied into the accumulation file before the data can be there
    bad = kernel("""
	;;#ASMSTART
	global_load_dwordx4 v[8:11], v[28:29], off ; by hand
	;;#ASMEND
	v_accvgpr_write_b32 a63, v11
	;;#ASMSTART
	s_waitcnt vmcnt(0)
	;;#ASMEND
	;;#ASMSTART
	; by hand v[8:11]
	;;#ASMEND
""")
    problems, _, _, _ = v.check_text(bad)
    assert len(problems) == 1 and "v_accvgpr_write_b32 a63, v11" in problems[0]


def test_a_hand_over_under_another_name_is_found():
    bad = kernel("""
	;;#ASMSTART
	global_load_dwordx4 a[0:3], v[28:29], off ; by hand
	;;#ASMEND
	;;#ASMSTART
	; by hand a[4:7]
	;;#ASMEND
""")
    problems, _, _, _ = v.check_text(bad)
    assert any("which no request names" in p for p in problems)
    assert any("never handed over" in p for p in problems)


def test_scratch_traffic_and_early_use_of_an_lds_read_are_found():
    bad = kernel("""
	;;#ASMSTART
	global_load_dwordx4 a[0:3], v[28:29], off ; by hand
	;;#ASMEND
	scratch_store_dword off, v3, s32
	;;#ASMSTART
	; by hand a[0:3]
	;;#ASMEND
	;;#ASMSTART
	ds_read_b128 v[40:43], v7
	;;#ASMEND
	v_mov_b32_e32 v9, v41
	;;#ASMSTART
	s_waitcnt lgkmcnt(0)
	;;#ASMEND
""")
    problems, _, _, _ = v.check_text(bad)
    assert any("scratch access" in p for p in problems)
    assert any("LDS read" in p for p in problems)


def test_fetches_of_both_forms_in_one_kernel_are_found():
    plain, past = "\tglobal_load_lds_dwordx4 v[2:3], off offset:1024\n", "\tglobal_load_lds_dwordx4 v[2:3], off offset:1024 nt\n"
    for body in (plain * 2, past * 2):
        assert v.check_text(kernel(body))[0] == []
    problems, _, _, _ = v.check_text(kernel(plain + past))
    assert len(problems) == 1 and "both past the caches and not" in problems[0]


def test_a_file_without_hand_loads_is_refused(tmp_path):
    f = tmp_path / "empty.s"
    f.write_text(kernel("\tv_mov_b32_e32 v0, v1\n"))
    with pytest.raises(RuntimeError):
        v.verify(str(f))
    g = tmp_path / "good.s"
    g.write_text(GOOD)
    assert v.verify(str(g)) == (1, 1, 1)


def projection(order):
    """The start of a kernel of 256 tokens x 2 heads with three stages of X and two of W_V, its first fetches in this order of tiles."""
    place = {"X0": 0, "X1": 0x8000, "X2": 0x10000, "W0": 0x18000, "W1": 0x20000}
    body = ["_ZN6tadakv12_GLOBAL__N_121compressv_gemm_kernelILi1ELi2ELi32ELi4ELi64ELi4ELi3ELi2EEEvNS_11ProjectArgsE:"]
    for tile in order.split():
        for i in range(4):
            at = place[tile] + 1024 * i
            body.append("\ts_add_i32 m0, s7, %s" % hex(at) if at else "\ts_mov_b32 m0, s7")
            body.append("\tglobal_load_lds_dwordx4 v[2:3], off")
    return "\n".join(body + ["\ts_waitcnt vmcnt(12)", "\ts_barrier", "\ts_endpgm", ".Lfunc_end0:"])


def test_the_projection_requests_its_stages_in_the_order_its_waits_count_on():
    assert v.check_fetch_order(projection("X0 W0 X1 W1 X2")) == ([], 1)
    # X of the third stage ahead of W_V of the second: the wait for all but four lets the loop read W_V too early
    for order in ("X0 W0 X1 X2 W1", "X0 X1 W0 W1 X2", "X0 W0 X1 W1"):
        problems, kernels = v.check_fetch_order(projection(order))
        assert kernels == 1 and len(problems) == 1, order
    unread = projection("X0 W0 X1 W1 X2").replace("s_mov_b32 m0, s7", "s_lshl_b32 m0, s7, 2")
    assert any("not known" in p for p in v.check_fetch_order(unread)[0])


def test_a_file_without_projection_kernels_is_refused(tmp_path):
    f = tmp_path / "other.s"
    f.write_text(GOOD)
    with pytest.raises(RuntimeError):
        v.verify_fetch_order(str(f))
