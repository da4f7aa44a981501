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


def _offsets(*lines):
    bad, loads = inflight_lint.check_buffer_offsets(_HEAD + "".join(f"\t{x}\n" if not x.startswith(".") else f"{x}\n" for x in lines) + "\ts_endpgm\n")
    return len(bad), loads


def test_a_scalar_offset_beside_a_size_that_is_not_a_constant_is_reported():
    load, at_zero = "buffer_load_dwordx4 v[2:5], v25, s[20:23], s6 offen", "buffer_load_dwordx4 v[6:9], v25, s[20:23], 0 offen"
    constant, variable = "s_mov_b32 s22, 0x10000", "s_lshl_b32 s22, s36, 4"
    assert _offsets(constant, at_zero, load) == (0, 2)
    assert _offsets(variable, at_zero) == (0, 1)
    assert _offsets(variable, at_zero, load) == (1, 2)
    assert _offsets(load) == (1, 1)                                  # (what the caller left there)
    assert _offsets(variable, constant, load) == (0, 1) and _offsets(constant, variable, load) == (1, 1)
    for other in ("s_mov_b64 s[22:23], s[6:7]", "s_load_dwordx4 s[20:23], s[0:1], 0x0", "v_readfirstlane_b32 s22, v7", "s_mov_b32 s22, s9"):
        assert _offsets(constant, other, load) == (1, 1), other
    for other in ("s_cmp_eq_u32 s22, 0", "s_mov_b32 s2, s9", "s_mov_b64 s[20:21], s[6:7]"):
        assert _offsets(constant, other, load) == (0, 1), other
    # the size on one of two paths, and on the way round a loop
    assert _offsets(constant, "s_cbranch_scc1 .LBB0_1", variable, ".LBB0_1:", load) == (1, 1)
    assert _offsets(constant, "s_cbranch_scc1 .LBB0_1", "s_add_i32 s5, s5, 1", ".LBB0_1:", load) == (0, 1)
    assert _offsets(constant, ".LBB0_1:", load, variable, "s_cbranch_scc1 .LBB0_1") == (1, 1)
    assert _offsets(constant, ".LBB0_1:", load, "s_cbranch_scc1 .LBB0_1", variable) == (0, 1)


# A stream's last vectors: a remainder of fewer than 3072 was read up to 48 KiB past the end of the ids
def test_the_count_reads_nothing_past_the_end_of_the_ids():
    for name in build.BUFFER_LOADS:
        bad, loads = inflight_lint.check_buffer_offsets(build.device_assembly(f"{build.CSRC}/{name}"))
        assert loads > 0 and bad == []
