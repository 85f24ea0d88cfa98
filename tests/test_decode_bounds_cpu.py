"""Every byte the M <= 16 decode kernel touches stays inside its buffers, for every launch the benchmark makes and for
ragged shapes: a host replica of the kernel's address arithmetic (tests/decode_addr_replica.py) enumerates all
workgroups, lanes and K items of a launch, with the instantiation and the launch geometry taken from the library's own
launch description."""
import pytest

from decode_addr_replica import ceil_div, decode_launch_spans, prefill_any_x_span
from paper_2402_17764_amd import binding as B

_ENTRY = {"LINEAR": B.ENTRY_LINEAR, "LINEAR_FUSED": B.ENTRY_LINEAR_FUSED, "RMSNORM_LINEAR_FUSED": B.ENTRY_RMSNORM_LINEAR_FUSED,
          "SWIGLU_LINEAR_FUSED": B.ENTRY_SWIGLU_LINEAR_FUSED, "FFN_GATE_UP": B.ENTRY_FFN_GATE_UP,
          "FFN_GATE_UP_NORM": B.ENTRY_FFN_GATE_UP_NORM}


def _check(entry, dtype, M, N, K, gstride=0, out_bytes=2):
    d = B.entry_describe(_ENTRY[entry], M, N, K, x_dtype=B.BF16 if dtype != "f32" else B.F32)
    if d["kernel"] not in ("decode", "decode_any", "decode_pair"):
        return None
    kR, kS, kW, kD, xmode = d["params"]
    sp, sizes, lds, grid = decode_launch_spans(kR, kS, kW, kD, xmode, d["kernel"] == "decode_pair", M, N, K,
                                               out_bytes=out_bytes, gstride=gstride)
    assert (grid, 1) == d["grid"] and lds == d["lds"] and d["block"] == 64 * kS * kW, (entry, M, N, K, d, lds, grid)
    for name, span in sp.items():
        assert span.within(sizes[name]), (entry, dtype, M, N, K, d, name, span.lo, span.hi, sizes[name])
    # the stream is read completely: the weight loads reach the last byte of the packed matrix
    assert sp["packed"].lo == 0 and sp["packed"].hi == sizes["packed"]
    return d


def test_every_decode_launch_of_the_benchmark_stays_in_bounds():
    import bench
    seen = set()
    for (leg, entry, dtype, M, N, K) in bench.launch_inventory():
        d = _check(entry, dtype, M, N, K)
        if d:
            seen.add((d["kernel"], tuple(d["params"])))
    assert len(seen) >= 8


def test_ragged_decode_launches_stay_in_bounds():
    import parity_shapes as P
    for (M, N, K) in P.GEMV_SHAPES:
        if K % 16 == 0 and M <= 8:
            for ob in (2, 4):
                _check("LINEAR", "int8", M, N, K, gstride=M % 2, out_bytes=ob)
    for dtype in ("bf16", "f32"):
        for (M, N, K) in P.FUSED_SHAPES:
            _check("LINEAR_FUSED", dtype, M, N, K, gstride=1)
        for (M, N, K) in P.NORM_FUSED_SHAPES:
            _check("RMSNORM_LINEAR_FUSED", dtype, M, N, K)
        for (M, N, F) in P.SWIGLU_FUSED_SHAPES:
            _check("SWIGLU_LINEAR_FUSED", dtype, M, N, F)
        for (M, F, K) in P.FFN_GATE_UP_SHAPES:
            _check("FFN_GATE_UP", dtype, M, F, K, gstride=1)
            _check("FFN_GATE_UP_NORM", dtype, M, F, K)


ANY_SHAPES = [(1, 300, 4097), (2, 16400, 259), (16, 33, 1001), (16, 16401, 77), (5, 300, 15), (3, 100, 255), (17, 130, 35), (32, 70, 333),
              (33, 100, 4863), (40, 1900, 3900), (77, 1003, 2050), (8192, 16, 33), (1, 40, 81407)]


@pytest.mark.parametrize("M,N,K", ANY_SHAPES)
def test_decode_launches_on_rows_of_any_length_stay_in_bounds(M, N, K):
    """x_q is read at byte alignment, sixteen bytes at a time past the row's end into the next one: to the last byte of x_q and
    no further, whatever the last token tile holds."""
    for ob in (2, 4):
        d = _check("LINEAR", "int8", M, N, K, gstride=1, out_bytes=ob)
        assert d["kernel"] == "decode_any"
    sp, sizes, _, _ = decode_launch_spans(*d["params"], False, M, N, K)
    assert sp["x"].lo == 0 and sp["x"].hi == sizes["x"] == M * K and sp["y"].hi == sizes["y"]
    # K a multiple of 16 comes here with an x_q that is not 16-byte aligned (described as if it were): the same form
    sp, sizes, _, _ = decode_launch_spans(*d["params"], False, M, N, ceil_div(K, 16) * 16)
    assert all(span.within(sizes[name]) for name, span in sp.items()) and sp["x"].hi == sizes["x"]


@pytest.mark.parametrize("M,N,K", [(200, 1000, 3333), (1030, 2500, 301), (700, 25000, 77), (3000, 1100, 3), (8193, 16, 33), (64, 5000, 255), (65, 9000, 272),
                                   (2000, 9000, 256), (17, 16, 200001)])
def test_prefill_launches_on_rows_of_any_length_read_x_q_to_its_end(M, N, K):
    d = B.linear_describe(M, N, K)
    assert K % 16 == 0 or (d["kernel"] == "prefill_any" and d["params"][0] == 64)
    sp = prefill_any_x_span(2, M, K)
    assert sp.lo == 0 and sp.hi == M * K
    assert K % 16 == 0 or prefill_any_x_span(2, M, K, bounded=False).hi > M * K          # what the bound is for


def test_the_replica_catches_a_planted_overrun():
    """the check itself: a launch whose LDS allocation is one fold slot short, and one with a row block too many"""
    sp, sizes, lds, grid = decode_launch_spans(1, 4, 1, 4, 0, False, 1, 3200, 3200)
    assert sp["lds"].within(sizes["lds"]) and not sp["lds"].within(sizes["lds"] - 16)
    sp, sizes, _, _ = decode_launch_spans(1, 4, 1, 4, 0, False, 1, 3200, 3200)
    assert not sp["packed"].within(sizes["packed"] - 16) and not sp["y"].within(sizes["y"] - 2)
