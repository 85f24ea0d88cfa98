"""The packing passes of the weight quantizer where a row is no whole number of 16-byte loads, starts on none, or the matrix is
smaller than one: the codes are integers and gamma one rounding of an exact sum, so everything is compared for equality."""
import numpy as np
import pytest
import torch

import oracle
from layout_ref import decode_2bit, decode_trit5

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (3, 1), (4, 1), (7, 1), (8, 1), (1, 2), (1, 3), (1, 7), (2, 3), (2, 5), (3, 5), (17, 1), (33, 2), (16, 320), (17, 321), (15, 319),
          (16, 313), (31, 648), (5, 327), (40, 511), (18, 513), (16, 1028), (100, 1001), (2100, 324), (700, 2563)]


def weights(N, K, dtype, offset, seed):
    """[N, K] on the GPU, `offset` elements into a larger buffer whose other elements would change every result."""
    rng = np.random.default_rng(seed)
    W = torch.from_numpy(rng.standard_normal((N, K), dtype=np.float32) * np.float32(0.02)).to(dtype)
    buf = torch.full((N * K + offset + 16,), 3.0e4, dtype=dtype, device="cuda")
    view = buf[offset:offset + N * K].view(N, K)
    view.copy_(W)
    return view, W.float().numpy()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("offset", [0, 1, 3, 4])
@pytest.mark.parametrize("N,K", SHAPES)
def test_five_trit_packing_at_the_edges(gpu_lib, N, K, offset, dtype):
    B = gpu_lib
    W, Wf = weights(N, K, dtype, offset, 1000 * N + K)
    codes, gamma = oracle.quantize_weights(Wf)
    packed, g = B.quantize_weights(W, B.PACK_TRIT5)
    assert g.cpu().numpy()[0].tobytes() == np.float32(gamma).tobytes()
    got, pad_zero = decode_trit5(packed.cpu().numpy(), N, K)
    assert pad_zero and np.array_equal(got, codes)
    p2, g2 = B.quantize_weights_sharded(W, B.abs_sum(W).view(1, 2), N, B.PACK_TRIT5)
    assert torch.equal(p2, packed) and torch.equal(g2, g)


@pytest.mark.parametrize("K", [640, 645])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_five_trit_packing_of_nan_and_infinity(gpu_lib, dtype, K):
    """What rounding and clipping the quotients gives: a NaN gamma makes every quotient NaN, which clips to -1 (padding included: all
    digits 0); an infinite one, here of a sum beyond fp32, makes a finite weight's quotient 0 and an infinite weight's NaN."""
    B, N = gpu_lib, 40
    W, _ = weights(N, K, dtype, 0, 5)
    W[3, 7] = float("nan")
    packed, g = B.quantize_weights(W, B.PACK_TRIT5)
    assert torch.isnan(g).all() and not packed.any()
    W[3, 7] = float("inf")
    W[39, K - 1] = float("-inf")
    sums = torch.tensor([[1e300, 0.0]], dtype=torch.float64, device="cuda")
    packed, g = B.quantize_weights_sharded(W, sums, N, B.PACK_TRIT5)
    want = np.zeros((N, K), dtype=np.int8)
    want[3, 7] = want[39, K - 1] = -1
    got, pad_zero = decode_trit5(packed.cpu().numpy(), N, K)
    assert torch.isinf(g).all() and pad_zero and np.array_equal(got, want)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("offset", [0, 1, 3, 4])
@pytest.mark.parametrize("N,K", SHAPES + [(16, 64), (17, 255), (31, 257), (16, 520), (40, 1023), (33, 1032)])
def test_two_bit_packing_at_the_edges(gpu_lib, N, K, offset, dtype):
    B = gpu_lib
    W, Wf = weights(N, K, dtype, offset, 1000 * N + K)
    codes, gamma = oracle.quantize_weights(Wf)
    packed, g = B.quantize_weights(W)
    assert g.cpu().numpy()[0].tobytes() == np.float32(gamma).tobytes()
    got, pad_zero = decode_2bit(packed.cpu().numpy(), N, K)
    assert pad_zero and np.array_equal(got, codes)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("rows,K", [((16, 3), 1), ((32, 16, 5), 3), ((16, 48, 16), 321), ((160, 32, 7), 1001), ((64, 64), 520)])
def test_segments_end_where_the_next_one_starts(gpu_lib, rows, K, offset, dtype):
    """Each segment's last rows are read up to their end, whatever follows, and the last one's tail is no whole row block."""
    B, N = gpu_lib, sum(rows)
    W, Wf = weights(N, K, dtype, offset, 7 * N + K)
    packed, g = B.quantize_weights_segmented(W, list(rows))
    got, pad_zero = decode_2bit(packed.cpu().numpy(), N, K)
    at, blocks = 0, g.cpu().numpy()
    for n in rows:
        codes, gamma = oracle.quantize_weights(Wf[at:at + n])
        assert np.array_equal(got[at:at + n], codes)
        assert all(b.tobytes() == np.float32(gamma).tobytes() for b in blocks[at // 16:(at + n + 15) // 16])
        at += n
    assert pad_zero
