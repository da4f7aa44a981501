"""The build's check of the device assembly: a load straight into LDS reads its address from M0 and needs a wait state
behind the scalar write of M0, which the compiler does not insert inside inline assembly."""
from paper_2506_22694_amd import build, inflight_lint

_HEAD = "\t.text\nkern:\n"


def _m0(body):
    bad, loads = inflight_lint.check_m0(_HEAD + body + "\ts_endpgm\n")
    return len(bad), loads


def test_a_load_into_lds_directly_behind_the_write_of_m0_is_reported():
    hand = lambda *lines: "\t;;#ASMSTART\n" + "".join(f"\t{x}\n" for x in lines) + "\t;;#ASMEND\n"
    write, load = "s_mov_b32 m0, s4", "global_load_lds_dwordx4 v1, s[2:3] nt"
    assert _m0(hand(write, load)) == (1, 1)
    assert _m0(hand(write, "s_nop 0", load)) == (0, 1)
    # the write may be the compiler's or sit at the other end of a branch
    assert _m0(f"\t{write}\n" + hand(load)) == (1, 1)
    assert _m0(f"\t{write}\n\ts_add_i32 s5, s5, 1\n" + hand(load)) == (0, 1)
    loop = ".LBB0_1:\n" + hand(load) + f"\ts_add_i32 s5, s5, 1\n\t{write}\n\ts_nop 0\n\ts_cbranch_scc1 .LBB0_1\n"
    assert _m0(loop) == (0, 1)
    assert _m0("\ts_cbranch_scc1 .LBB0_2\n\t" + write + "\n.LBB0_2:\n" + hand(load)) == (1, 1)
    # the next load's own write, and loads into registers, are nobody's hazard
    assert _m0(hand(write, "s_nop 0", load) * 2) == (0, 2)
    assert _m0(hand(write, "global_load_dwordx4 v[4:7], v1, s[2:3]")) == (0, 0)


def test_the_source_with_loads_into_lds_is_checked():
    for name in build.MIN_LDS_LOADS:
        assert name.startswith(build.NO_SCRATCH) and build.MIN_LDS_LOADS[name] > 0
        src = open(f"{build.CSRC}/{name}").read()
        writes = src.count("s_mov_b32 m0")
        assert writes > 0 and src.count("s_mov_b32 m0, %0\\n\\ts_nop 0\\n\\tglobal_load_lds_") == writes


def test_a_function_may_end_in_several_places():
    load, wait = "\t;;#ASMSTART\n\tglobal_load_dwordx4 v[4:7], v1, s[2:3]\n\t;;#ASMEND\n", "\ts_waitcnt vmcnt(0)\n"
    tail = "\ts_cbranch_scc1 .LBB0_2\n\ts_endpgm\n.LBB0_2:\n"
    end = "\ts_endpgm\n.Lfunc_end0:\n\t.size kern, .Lfunc_end0-kern\n"
    other = "other:\n\tv_mov_b32_e32 v40, v4\n\ts_endpgm\n.Lfunc_end1:\n"
    assert inflight_lint.check_asm(_HEAD + load + tail + wait + "\tv_mov_b32_e32 v9, v4\n" + end + other) == ([], 1)
    bad, loads = inflight_lint.check_asm(_HEAD + load + tail + "\tv_mov_b32_e32 v9, v4\n" + wait + end + other)
    assert [b[3] for b in bad] == ["v_mov_b32_e32 v9, v4"] and loads == 1
