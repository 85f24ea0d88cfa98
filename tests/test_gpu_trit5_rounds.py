"""GPU tests of the 5-trit launches whose row blocks per workgroup are chosen to put one on every CU (five, six, seven and eight): row
counts at the edges of each, K walks that end within a wave's round, one to sixteen tokens; against the exact product."""
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# K waves, row blocks per workgroup, prefetch depth, groups of eight tokens
FORMS = {(1025, 3200, 5): [4, 1, 2, 1], (1025, 4176, 5): [2, 5, 2, 1], (1280, 6400, 16): [2, 5, 2, 2], (1281, 4176, 8): [2, 6, 2, 1], (1536, 3200, 9): [2, 6, 2, 2],
         (1537, 320, 1): [1, 7, 4, 1], (1792, 6400, 4): [1, 7, 4, 1], (1793, 2896, 3): [1, 8, 4, 1], (2048, 6400, 4): [1, 8, 4, 1],
         (1537, 6400, 5): [1, 8, 4, 1], (1025, 320, 9): [1, 8, 4, 2], (2048, 6400, 16): [1, 8, 4, 2]}


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
        if (RB, K, M) in FORMS:
            assert B.linear_describe(M, N, K, B.PACK_TRIT5)["params"] == FORMS[RB, K, M]
        assert K * 127 < 2 ** 24
        assert torch.equal(B.linear(xq, sx, packed, gamma, N, fmt=B.PACK_TRIT5, y_dtype=B.I32), want)
