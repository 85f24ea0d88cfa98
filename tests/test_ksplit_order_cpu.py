"""The build's guard for linear_ksplit_2bit (csrc/linear_ksplit.hip), whose waits count the loads younger than a tile's copies: the
parser on canned text, good and bad, and on the assembly of the current build."""
import os

import pytest

from paper_2402_17764_amd import build as Bld

P = (2, 2, 1, 8, 2)                     # kMT, kR, kW, kS, kQ: two weight loads a step, two tiles of four copies, both in LDS
GOOD = "WWLLLLLLLL" "WW" "aRRMRRzMLLLL" "aRRRRzMLLLL" "bRRRRMz" "0RRRRzM"


def _text(events):
    line = {"W": "\tbuffer_load_dwordx4 v[2:5], v6, s[8:11], s3 offen", "L": "\tbuffer_load_dwordx4 v1, s[4:7], 0 offen lds",
            "R": "\tds_read_b128 v[0:3], v4", "M": "\tv_mfma_i32_16x16x64_i8 v[0:3], v[4:7], v[8:11], v[0:3]", "a": "\ts_waitcnt vmcnt(6)",
            "b": "\ts_waitcnt vmcnt(4)", "0": "\ts_waitcnt vmcnt(0)", "9": "\ts_waitcnt vmcnt(9)", "d": "\ts_waitcnt vmcnt(8)",
            "z": "\ts_waitcnt lgkmcnt(0)", "y": "\ts_waitcnt lgkmcnt(1)"}
    return ("_ZN6bitnet18linear_ksplit_2bitILi%sEEEvPKa:                  ; @kernel\n" % "ELi".join(map(str, P)) + "\n".join(line[c] for c in events) +
            "\n\ts_barrier\n\ts_endpgm\n.Lfunc_end0:\n")


def test_order_parser():
    assert Bld.check_ksplit_order(_text(GOOD), [P]) == [P]
    assert Bld.check_ksplit_order(_text(GOOD.replace("LWW", "LdWW")), [P]) == [P]      # the compiler's own wait for the weights
    for bad in (GOOD.replace("LWW", "WLW"), GOOD.replace("aRRMRR", "9RRMRR"), GOOD.replace("aRRM", "RRM"), GOOD.replace("bR", "aR"),
                GOOD.replace("0R", "bR"), GOOD[2:], GOOD[:-7], GOOD.replace("WWaRRMRR", "aRRMRRWW"), "",
                GOOD.replace("aRRRR", "RaRRR"), GOOD.replace("aRRRR", "aRRRRR"), GOOD.replace("LLLLaRRRR", "LLLLRaRRRR"),       # a read in front of its wait, one too many
                GOOD.replace("zMLLLL", "MLLLL", 1), GOOD.replace("zMLLLL", "yMLLLL", 1), GOOD.replace("RRzMLLLLa", "RzRMLLLLa")):     # a copy over a slot that is being read
        with pytest.raises(RuntimeError):
            Bld.check_ksplit_order(_text(bad), [P])
    for expected in ([], [P, P], [(1, 1, 1, 8, 1)]):
        with pytest.raises(RuntimeError):
            Bld.check_ksplit_order(_text(GOOD), expected)
    assert Bld.ksplit_instantiations("KSPLIT(2, 2, 1, 8, 0) KSPLIT(2, 2, 2, 4, 2)") == [(2, 2, 1, 8, 2), (2, 2, 2, 4, 3)]


def test_current_build_passes_the_guard():
    asm = os.path.join(Bld.BUILD, "linear_ksplit-hip-amdgcn-amd-amdhsa-gfx950.s")
    if not os.path.exists(asm):
        pytest.skip("no build directory here (the library was built elsewhere)")
    want = Bld.ksplit_instantiations(open(os.path.join(Bld.CSRC, "linear_ksplit.hip")).read())
    assert len(want) >= 8 and sorted(Bld.check_ksplit_order(open(asm).read(), want)) == want
