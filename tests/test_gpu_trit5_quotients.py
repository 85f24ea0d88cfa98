"""GPU test of the 5-trit decode kernel that works on quotients: every launch shape of its selection, K from a part of a step on, both
groups of eight tokens, rows that do and do not allow four outputs in a store -- accumulators exact, outputs to the bit."""
import numpy as np
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,K", [(250, 6416), (4096, 8000), (4500, 2576), (6400, 7200), (9600, 960), (9601, 3216), (12800, 6560), (16400, 2560), (16400, 6416),
                                 (24600, 336), (27648, 1280), (33000, 2576), (50001, 3200)])
def test_quotients(gpu_lib, N, K):
    g = torch.Generator(device="cuda").manual_seed(N + K)
    W = torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g)
    W[: N // 3] = W[: N // 3].abs() + 0.05                               # rows of ones, of minus ones: every quotient at its largest
    W[N // 3: N // 2] = -W[N // 3: N // 2].abs() - 0.05
    packed, gamma = B.quantize_weights(W, B.PACK_TRIT5)
    codes = B.unpack_weights(packed, N, K, B.PACK_TRIT5).float()
    x = torch.randint(-127, 128, (16, K), device="cuda", generator=g, dtype=torch.int32).to(torch.int8)
    x[0], x[1], x[9] = 127, -127, 127
    sx = torch.rand(16, device="cuda", generator=g) + 0.5
    for M in (1, 3, 4, 5, 8, 9, 16):
        print("quotients", M, N, K, flush=True)
        xm, sm = x[:M].contiguous(), sx[:M].contiguous()
        want = (xm.float() @ codes.t()).to(torch.int32)                  # |sums| < 2^24: exact in fp32
        assert torch.equal(B.linear(xm, sm, packed, gamma, N, fmt=B.PACK_TRIT5, y_dtype=B.I32), want)
        scale = (gamma.cpu().numpy() * sm.cpu().numpy()) / np.float32(127.0)
        y = want.float() * torch.from_numpy(scale).cuda()[:, None]
        assert torch.equal(B.linear(xm, sm, packed, gamma, N, fmt=B.PACK_TRIT5), y)
        room = torch.full((M * N + 9,), 77, dtype=torch.bfloat16, device="cuda")
        for off in (0, 1):
            out = room[off:off + M * N].view(M, N)
            B.linear(xm, sm, packed, gamma, N, fmt=B.PACK_TRIT5, y_dtype=B.BF16, y=out)
            assert torch.equal(out, y.to(torch.bfloat16)) and (room[M * N + 1:] == 77).all()
