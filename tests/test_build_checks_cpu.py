"""The build's guard for linear_skinny_2bit (csrc/linear_skinny.hip): that kernel retires its LDS-DMA copies with a
counted s_waitcnt, which is right only while copies and weight loads are issued in source order.  The guard reads the
device assembly the shipped object was assembled from; here its parser is run on canned text, good and bad, and on the
assembly of the current build.  So is the one that finds LDS reads outstanding at a barrier: behind it the next copy is
written to the stage that they read."""
import os
import re

import pytest

from paper_2402_17764_amd import build as Bld


def _kernel(params, prologue, loops, name="linear_skinny_2bit"):
    mangled = "_ZN6bitnet%d%sILi%sE" % (len(name), name, "ELi".join(str(p) for p in params))
    copy = "\tbuffer_load_dwordx4 v1, s[4:7], 0 offen lds\n"
    weight = "\tbuffer_load_dwordx4 v[2:5], v6, s[8:11], 0 offen\n"
    emit = lambda seq: "".join(copy if c == "L" else weight for c in seq)
    text = mangled + "EvPKaPKfPK15HIP_vector_typeIjLj4EES4_iilliiiPvNS_7OutTypeE:\n\ts_load_dwordx2 s[0:1], s[4:5], 0x0\n"
    text += emit(prologue) + "\ts_waitcnt vmcnt(3)\n"
    for seg in loops:
        text += "\ts_barrier\n" + emit(seg) + "\tv_mfma_i32_16x16x64_i8 v[0:3], v[4:7], v[8:11], v[0:3]\n"
    return text + "\ts_barrier\n\ts_endpgm\n"


def test_issue_order_parser_accepts_source_order_and_rejects_everything_else():
    p = (2, 2, 2, 4, 2, 2)                      # kMT, kR, kW, kS, kD, kLx: 4 copies then 2 weight loads per step, prologue of 2
    unit = "LLLL" + "WW"
    good = _kernel(p, unit * 2, [unit, unit])
    assert Bld.check_issue_order(good, [p]) == [p]
    # a weight load hoisted above the last copy of the prologue, and one in the loop
    for bad in (_kernel(p, "LLLWLW" + unit, [unit]), _kernel(p, unit * 2, [unit, "LLWLLW"]), _kernel(p, unit, [unit]),
                _kernel(p, unit * 2, [])):
        with pytest.raises(RuntimeError):
            Bld.check_issue_order(bad, [p])
    # an expected instantiation that the assembly does not hold, one it holds unasked, and a truncated kernel
    with pytest.raises(RuntimeError):
        Bld.check_issue_order(good, [p, (1, 1, 1, 8, 2, 2)])
    with pytest.raises(RuntimeError):
        Bld.check_issue_order(good + _kernel((1, 1, 1, 8, 2, 2), "LLLLW" * 2, ["LLLLW"]), [p])
    with pytest.raises(RuntimeError):
        Bld.check_issue_order(good.replace("\ts_endpgm\n", ""), [p])
    with pytest.raises(RuntimeError):
        Bld.check_issue_order("", [p])
    # other kernels in the same file are not its business
    other = _kernel(p, "WWLL", ["WL"], name="linear_skinny_ws_2bit")
    assert Bld.check_issue_order(other + good, [p]) == [p]


def test_dispatched_instantiations_are_read_from_the_launcher():
    src = open(os.path.join(Bld.CSRC, "linear_skinny.hip")).read()
    inst = Bld.skinny_instantiations(src)
    assert len(inst) >= 10 and all(len(t) == 6 for t in inst)
    assert Bld.skinny_instantiations("if (a) SKINNY(1, 2, 3, 4, 5, 6); else SKINNY(1, 2, 3, 4, 5, 6);") == [(1, 2, 3, 4, 5, 6)]


def test_current_build_passes_the_guard():
    asm = os.path.join(Bld.BUILD, "linear_skinny-hip-amdgcn-amd-amdhsa-gfx950.s")
    if not os.path.exists(asm):
        pytest.skip("no build directory here (the library was built elsewhere)")
    src = open(os.path.join(Bld.CSRC, "linear_skinny.hip")).read()
    checked = Bld.check_issue_order(open(asm).read(), Bld.skinny_instantiations(src))
    assert sorted(checked) == Bld.skinny_instantiations(src)
    loader = Bld.skinny_instantiations(src, "SKINNY_WS")
    reads = Bld.check_lds_reads(open(asm).read(), Bld.skinny_instantiations(src), loader)
    assert len(reads) == len(checked) + len(loader) and not any(reads.values())


def _waits(body, name="linear_skinny_ws_2bit", params=(4, 2, 3, 1, 4, 2)):
    head = "_ZN6bitnet%d%sILi%sEEEvPKa:                  ; @kernel\n; %%bb.0:\n" % (len(name), name, "ELi".join(str(p) for p in params))
    lines = {"R": "\tds_read_b128 v[0:3], v4 offset:16", "0": "\ts_waitcnt vmcnt(3) lgkmcnt(0)", "1": "\ts_waitcnt lgkmcnt(1)", "v": "\ts_waitcnt vmcnt(0)",
             "B": "\ts_barrier", "L": ".LBB0_1:                                ; =>This Inner Loop", "J": "\ts_cbranch_scc1 .LBB0_1",
             "S": "\ts_cbranch_execz .LBB0_2", "T": ".LBB0_2:", "E": "\ts_endpgm"}
    return head + "\n".join(lines[c] for c in body) + "\n.Lfunc_end0:\n"


@pytest.mark.parametrize("body,reads", [
    ("RR0BE", 0), ("RR1BE", 1), ("RRvBE", 2), ("BRR0E", 0),
    ("LBRR0JE", 0),                        # a loop that waits before it comes round
    ("LBRR1JE", 1),                        # ... and one whose barrier meets a read of the round before
    ("RSR0TBE", 1),                        # a branch past the wait
    ("RS0TR0BE", 0),
])
def test_outstanding_lds_reads_are_found_on_every_path(body, reads):
    p = (4, 2, 3, 1, 4, 2)
    assert Bld.lds_reads_at_barriers(_waits(body)) == {(True, p): reads}
    if reads:
        with pytest.raises(RuntimeError):
            Bld.check_lds_reads(_waits(body), [], [p])
    else:
        Bld.check_lds_reads(_waits(body), [], [p])
        with pytest.raises(RuntimeError):                  # an instantiation that the assembly does not hold, one that nobody asked for
            Bld.check_lds_reads(_waits(body), [p], [p])
        with pytest.raises(RuntimeError):
            Bld.check_lds_reads(_waits(body), [], [])


def _wide_stores_first(asm):
    """{instantiation: (8-byte stores in front of the first of a single bf16 output, outputs of four that a wave holds)}"""
    found = {}
    for m in re.finditer(r"^_ZN6bitnet\d+(linear_skinny(?:_ws)?_2bit)I((?:Li\d+E)+)E\S*:[^\n]*\n(.*?)^\.Lfunc_end", asm, re.M | re.S):
        p = tuple(int(v) for v in re.findall(r"Li(\d+)E", m.group(2)))
        head = re.split(r"\bglobal_store_(?:short|byte)", m.group(3), maxsplit=1)[0]
        found[m.group(1), p] = (len(re.findall(r"\bglobal_store_dwordx2\b", head)), p[0] * p[1])
    return found


def test_stores_by_the_element_stand_apart():
    """the test for a row's end, and the single stores behind it, in front of every wide store cost short launches 4 %"""
    asm = os.path.join(Bld.BUILD, "linear_skinny-hip-amdgcn-amd-amdhsa-gfx950.s")
    if not os.path.exists(asm):
        pytest.skip("no build directory here (the library was built elsewhere)")
    found = _wide_stores_first(open(asm).read())
    assert len(found) >= 10
    for which, (wide, held) in found.items():
        assert wide >= held, which
