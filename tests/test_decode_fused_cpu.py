"""The fused decode launches of one to four tokens (csrc/decode_kernel.hpp), on the CPU: a replica of the kernel's address
arithmetic, with launch shape and LDS allocation from the library's own launch description, shows that every byte of the packed
matrix is requested exactly once and by nobody past its end, and that LDS reads and writes stay inside the allocation."""
import random

import numpy as np
import pytest

from decode_addr_replica import ceil_div
from paper_2402_17764_amd import binding as B

HEADER, MAX_AT, EXACT_AT = 512, 0, 256
ENTRIES = {"rows": B.ENTRY_LINEAR_FUSED, "norm": B.ENTRY_RMSNORM_LINEAR_FUSED, "pair": B.ENTRY_FFN_GATE_UP, "norm_pair": B.ENTRY_FFN_GATE_UP_NORM}


def vecs(K, threads, bf16):
    return ceil_div(K, threads * (8 if bf16 else 4))


def check(entry, bf16, M, N, K):
    """None where another kernel serves the call, else the form."""
    d = B.entry_describe(ENTRIES[entry], M, N, K, x_dtype=B.BF16 if bf16 else B.F32)
    pair, norm = entry.endswith("pair"), entry.startswith("norm")
    kR, kS, kW, kD, xmode = d["params"]
    threads, waves = 64 * kS * kW, kS * kW
    if M > 4 or vecs(K, threads, bf16) > 4:
        return None
    assert xmode == (4 if norm else 2) + (0 if bf16 else 1) and d["block"] == threads <= 1024 and (kR == 2 or not pair)
    steps, rb = ceil_div(K, 256), ceil_div(N, 16)
    kT, kV, kE = (1, 2, 4, 4)[M - 1], vecs(K, threads, bf16), 8 if bf16 else 4
    row, lds = steps * 256, d["lds"]
    items = ceil_div(ceil_div(steps, kS), kD) * kD
    # LDS
    assert MAX_AT + kT * 16 * 4 <= EXACT_AT and EXACT_AT + 2 * 16 * 8 <= HEADER and HEADER + kT * waves * 8 <= lds
    written = np.arange(kV * threads, dtype=np.int64) * kE
    written = written[written < row]
    assert written.max() + kE == row                                   # whole rows, zero padding included
    rows_end = HEADER + M * row
    assert rows_end <= lds
    last_read = (min(kT, M) - 1) * row + 3 * 64 + min(kS - 1 + (items - 1) * kS, steps - 1) * 256 + 3 * 16 + 16
    assert HEADER + last_read <= rows_end
    need = (kS - 1) * kW * kR * 256
    assert (rows_end if rows_end + need <= lds else HEADER) + need <= lds
    # weights: chunk of (step, row block) -> [first, first + bytes)
    halves = 2 if pair else 1
    step_bytes, last = rb * halves * 1024, (ceil_div(K, 64) - 4 * (steps - 1)) * 256
    wg = np.arange(d["grid"][0], dtype=np.int64)[:, None, None]
    ww, ws = np.arange(kW)[None, :, None], np.arange(kS)[None, None, :]
    first = (wg * kW + ww) if pair else (wg * kW + ww) * kR
    total, end = 0, 0
    for item in range(items):
        step = ws + item * kS
        nbytes = np.where(step < steps - 1, 1024, np.where(step == steps - 1, last, 0))
        for a in range(kR):
            r = first + (a * rb if pair else a)
            n = np.where(first < rb if pair else r < rb, nbytes, 0)
            total += int(n.sum())
            end = max(end, int(np.where(n > 0, step * step_bytes + r * nbytes + n, 0).max()))
    size = 16 * rb * halves * 64 * ceil_div(K, 64) // 4
    assert total == size and end == size, (entry, M, N, K, d)
    # output rows: all of them, none twice
    n = first[..., 0:1] * 16 + np.arange(16 * (1 if pair else kR))
    assert int((n < N).sum()) == N
    return (entry, bf16, kR, kS, kW, kD, kV, kT)


@pytest.mark.parametrize("entry", list(ENTRIES))
def test_fused_decode_launches_stay_in_bounds_and_read_the_matrix_once(entry):
    rng, seen = random.Random(4), set()
    for _ in range(1500):
        M, bf16 = rng.choice([1, 1, 2, 3, 4]), rng.random() < 0.6
        N = rng.choice([16, 96, 256, 1504, 4096, 4112, 8192, 8208, 9600, 11008, 16384, 16400, 24576, 32768, 32784, 40000, 49152, 49168, 57344])
        N = N if entry.endswith("pair") else N - rng.choice([0, 0, 1, 15])
        K = 16 * rng.choice([1, 4, 5, 16, 17, 48, 64, 65, 80, 100, 128, 129, 144, 160, 200, 256, 257, 320, 368, 400, 512, 513, 540, 688, 750, 768, 1024, 1025, 1153, 1280, 1536, 1792])
        if 512 + M * ceil_div(K, 256) * 256 <= 65536:
            seen.add(check(entry, bf16, M, N, K))
    forms = {f[2:6] for f in seen if f}
    assert len(forms) >= (8 if entry.endswith("pair") else 13), sorted(forms)
    assert {f[6] for f in seen if f} == {1, 2, 3, 4} and {f[7] for f in seen if f} == {1, 2, 4} and None in seen


@pytest.mark.parametrize("entry", list(ENTRIES))
def test_every_size_that_fits_is_served(entry):
    """what the acceptance rule lets through has a kernel: every K step with its first and last K, in every class of row blocks"""
    for rb in (1, 256, 257, 400, 512, 513, 640, 641, 1024, 1025, 2048, 2049, 3072, 3073, 4096):
        for M in (1, 2, 3, 4):
            for steps in range(1, (65536 - HEADER) // (256 * M) + 1):
                for K in (256 * steps - 240, 256 * steps):
                    for dtype in (B.BF16, B.F32):
                        B.entry_describe(ENTRIES[entry], M, 16 * rb, K, x_dtype=dtype)          # raises for an error status
