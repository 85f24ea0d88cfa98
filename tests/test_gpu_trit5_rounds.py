"""GPU tests of the 5-trit launches whose row blocks per workgroup are chosen to put one on every CU (five, six, seven and eight): row
counts at the edges of each, K walks that end within a wave's round, one to sixteen tokens; against the exact product."""
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("RB", [1025, 1280, 1281, 1536, 1537, 1792, 1793, 2048])
@pytest.mark.parametrize("K", [320, 2896, 3200, 4176, 6400])
def test_row_blocks_per_workgroup(gpu_lib, RB, K):
    N = 16 * RB - 5 * (RB % 2)
    g = torch.Generator(device="cuda").manual_seed(RB + K)
    packed, gamma = B.quantize_weights(torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g), B.PACK_TRIT5)
    codes = B.unpack_weights(packed, N, K, B.PACK_TRIT5).float()
    for M in (1, 3, 4, 5, 8, 9, 16):
        xq, sx = B.quantize_acts(torch.randn((M, K), device="cuda", generator=g))
        want = (xq.float() @ codes.t()).to(torch.int32)            # |sums| < 2^24: exact in fp32
        print("trit5 rounds", RB, K, M, flush=True)
        assert K * 127 < 2 ** 24
        assert torch.equal(B.linear(xq, sx, packed, gamma, N, fmt=B.PACK_TRIT5, y_dtype=B.I32), want)
