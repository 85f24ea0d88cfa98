"""GPU tests of the batched-decode kernels' ends: K walks of every length around the steps that stand behind the loop, and outputs
that can and cannot be stored four at a time."""
import numpy as np
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# one form per (tokens, row blocks) class of the selection, with and without a loader wave; K from one step to past two whole walks
@pytest.mark.parametrize("M,N", [(9, 4096), (13, 9000), (29, 4096), (20, 12288), (30, 22016), (64, 4000), (50, 8200), (40, 22016), (64, 40000), (100, 4096), (200, 5120)])
@pytest.mark.parametrize("K", [16, 256, 528, 768, 1296, 2048, 2320, 4112, 8208])
def test_k_walks_and_output_rows(gpu_lib, M, N, K):
    assert B.linear_describe(M, N, K)["kernel"].startswith("batched_decode")
    g = torch.Generator(device="cuda").manual_seed(M * N + K)
    packed, gamma = B.quantize_weights(torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g))
    xq, sx = B.quantize_acts(torch.randn((M, K), device="cuda", generator=g))
    codes = B.unpack_weights(packed, N, K)
    want = (xq.float() @ codes.float().t()).to(torch.int32) if K * 127 < 2 ** 24 else (xq.double() @ codes.double().t()).to(torch.int32)
    print("batched", M, N, K, flush=True)
    acc = B.linear(xq, sx, packed, gamma, N, y_dtype=B.I32)
    assert torch.equal(acc, want)
    for y_dtype, dtype in ((B.I32, torch.int32), (B.F32, torch.float32), (B.BF16, torch.bfloat16)):
        y = B.linear(xq, sx, packed, gamma, N, y_dtype=y_dtype)
        if y_dtype != B.I32:
            # numpy divides as IEEE has it (torch multiplies by the reciprocal of a scalar divisor)
            scale = (gamma.cpu().numpy() * sx.cpu().numpy()) / np.float32(127.0)
            scaled = want.float() * torch.from_numpy(scale).cuda()[:, None]
            assert torch.equal(y, scaled.to(dtype))
        # a base one output past an aligned one: the narrow stores, nothing written around them
        room = torch.full((M * N + 9,), 77, dtype=dtype, device="cuda")
        B.linear(xq, sx, packed, gamma, N, y_dtype=y_dtype, y=room[1:1 + M * N].view(M, N))
        assert torch.equal(room[1:1 + M * N].view(M, N), y) and (room[:1] == 77).all() and (room[1 + M * N:] == 77).all()
