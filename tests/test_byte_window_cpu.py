"""The address rule of the 16-byte loads from rows of any length, replicated: every load lies in the matrix, and what is moved to
its place is what a load that stops at the end would hold."""
import random

import numpy as np


def window(first, left):
    lead = 16 if first >= 16 else 0
    return first - lead, lead, min(left + lead, 1 << 30)


def test_loads_stay_in_the_matrix_and_hold_its_bytes():
    rng = random.Random(11)
    for _ in range(300):
        M, K = rng.randint(1, 40), rng.choice([1, 3, 7, 15, 16, 17, 31, 255, 256, 257, 333])
        x = np.arange(M * K, dtype=np.int64) % 251 + 1
        row0 = rng.randrange(M)
        base, lead, size = window(row0 * K, (M - row0) * K)
        if size < 16:
            assert (M - row0) * K < 16                       # such a matrix is read byte by byte
            continue
        for row in range(row0, M):
            for col in range(0, (K + 255) // 256 * 256, 16):
                off = (row - row0) * K + col
                at = min(lead + off, size - 16)
                assert 0 <= at and 0 <= base + at and base + at + 16 <= M * K
                moved = lead + off - at
                got = np.zeros(16, dtype=np.int64)
                if moved < 16:
                    got[:16 - moved] = x[base + at + moved:base + at + 16]
                want = np.zeros(16, dtype=np.int64)
                rest = x[row0 * K + off:row0 * K + off + 16]
                want[:len(rest)] = rest
                assert np.array_equal(got, want)
