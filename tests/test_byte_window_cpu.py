"""The address rule of the 16-byte loads from rows of any length (csrc/byte_window.hpp, compiled for the host): every load lies in the
matrix, and what a kernel puts in LDS for a column below K is that column's byte -- also where the kernel moves pulled-back pieces
only in tiles that have some."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

from paper_2402_17764_amd.build import CSRC

SHIM = """
#include "byte_window.hpp"
using bitnet::ByteSpan;
extern "C" void span(int64_t first, int64_t left, int* lead, int* bytes) { const ByteSpan s(first, left); *lead = s.lead; *bytes = s.bytes; }
extern "C" int whole(int64_t first, int64_t left) { return ByteSpan(first, left).whole(); }
extern "C" int at(int64_t first, int64_t left, int off) { return ByteSpan(first, left).at(off); }
extern "C" int moved(int64_t first, int64_t left, int off) { return ByteSpan(first, left).moved(off); }
extern "C" int pulls_back(int64_t first, int64_t left, int rows, int K) { return ByteSpan(first, left).pulls_back(rows, K); }
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("byte_window")
    src, lib = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, src, "-o", lib])
    so = ctypes.CDLL(lib)
    for name in ("span", "whole", "at", "moved", "pulls_back"):
        getattr(so, name).argtypes = [ctypes.c_int64, ctypes.c_int64] + {"span": [ctypes.POINTER(ctypes.c_int)] * 2, "whole": []}.get(
            name, [ctypes.c_int] * (2 if name == "pulls_back" else 1))
    return so


def window(rule, first, left):
    lead, size = ctypes.c_int(), ctypes.c_int()
    rule.span(first, left, ctypes.byref(lead), ctypes.byref(size))
    return first - lead.value, size.value


def piece(rule, x, first, left, base, off, move):
    """the 16 bytes that land in LDS; the load itself has to lie in the matrix"""
    start = base + rule.at(first, left, off)
    assert 0 <= start and start + 16 <= len(x)
    down = rule.moved(first, left, off) if move else 0
    got = np.zeros(16, dtype=np.int64)
    if down < 16:
        got[:16 - down] = x[start + down:start + 16]
    return got


def test_loads_stay_in_the_matrix_and_hold_its_bytes(rule):
    rng = random.Random(11)
    for _ in range(300):
        M, K = rng.randint(1, 40), rng.choice([1, 3, 7, 15, 16, 17, 31, 255, 256, 257, 333])
        x = np.arange(M * K, dtype=np.int64) % 251 + 1
        row0 = rng.randrange(M)
        first, left = row0 * K, (M - row0) * K
        base, size = window(rule, first, left)
        assert rule.whole(first, left) == (size >= 16)
        if size < 16:
            assert left < 16                                 # such a matrix is read byte by byte
            continue
        for row in range(row0, M):
            for col in range(0, (K + 255) // 256 * 256, 16):
                off = (row - row0) * K + col
                want = np.zeros(16, dtype=np.int64)
                rest = x[row0 * K + off:row0 * K + off + 16]
                want[:len(rest)] = rest
                assert np.array_equal(piece(rule, x, first, left, base, off, True), want)


@pytest.mark.parametrize("tokens", [64, 96, 128])
def test_tiles_that_skip_the_move_hold_their_rows_all_the_same(rule, tokens):
    """the prefill form: a tile's pieces are moved in the last K step, and only if the tile has one that is pulled back"""
    skipped = 0
    for K in list(range(1, 18)) + [31, 100, 255, 256, 257, 300, 513]:
        for M in [1, 5, tokens - 1, tokens] + [tokens + r for r in range(1, 17)] + [3 * tokens + 1]:
            x = (np.arange(M * K, dtype=np.int64) * 7) % 251 + 1
            steps = (K + 255) // 256
            for row0 in range(0, M, tokens):
                rows, first, left = min(tokens, M - row0), row0 * K, (M - row0) * K
                base, size = window(rule, first, left)
                if size < 16:
                    continue
                pulls = rule.pulls_back(first, left, rows, K)
                skipped += not pulls
                for row in sorted({0, rows // 2} | set(range(max(0, rows - 18), rows))):
                    for step in sorted({0, steps - 1}):
                        for col in range(step * 256, min(step * 256 + 256, K), 16):
                            off = row * K + col
                            n = min(16, K - col)                 # bytes behind the row meet zero codes
                            got = piece(rule, x, first, left, base, off, pulls and step == steps - 1)
                            assert np.array_equal(got[:n], x[first + off:first + off + n]), (M, K, row0, row, col)
    assert skipped > 100
