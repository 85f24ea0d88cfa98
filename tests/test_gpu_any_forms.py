"""GPU tests of the launch shapes for activation rows of any length (decode_any): each of them at tokens, rows and K that do and do not fill
it, against the exact product, one gamma and a gamma per row block."""
import numpy as np
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FORMS = [(1, 300, 4097, [1, 8, 1, 1]), (16, 4090, 17, [1, 8, 1, 1]), (33, 1001, 2049, [1, 8, 1, 1]), (77, 1003, 600, [2, 4, 1, 1]), (16, 9001, 1001, [2, 4, 1, 1]),
         (2, 30001, 130, [2, 4, 1, 1]), (40, 1900, 1900, [2, 8, 1, 1]), (5, 8177, 1283, [2, 8, 1, 1]), (77, 1003, 2050, [2, 8, 1, 2]), (16, 8190, 4001, [2, 8, 1, 2]),
         (9, 12001, 2305, [2, 4, 2, 2]), (4, 20003, 1539, [2, 4, 2, 2]), (3, 8205, 2050, [1, 4, 1, 4]), (6, 9000, 1400, [1, 4, 1, 4]), (1, 16401, 2055, [2, 4, 1, 1]),
         (2, 17001, 4099, [1, 2, 2, 4])]


@pytest.mark.parametrize("M,N,K,form", FORMS)
def test_forms_against_the_exact_product(gpu_lib, M, N, K, form):
    d = B.linear_describe(M, N, K)
    assert (d["kernel"], d["params"][:4]) == ("decode_any", form)
    g = torch.Generator(device="cuda").manual_seed(M * N + K)
    rows = [(N + 31) // 32 * 16, N - (N + 31) // 32 * 16]
    packed, gamma_rb = B.quantize_weights_segmented(torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g), rows)
    xq, sx = B.quantize_acts(torch.randn((M, K), device="cuda", generator=g))
    want = (xq.float() @ B.unpack_weights(packed, N, K).float().t()).to(torch.int32)      # |sums| < 2^24: exact in fp32
    print("any", M, N, K, flush=True)
    assert torch.equal(B.linear(xq, sx, packed, torch.ones(1, device="cuda"), N, y_dtype=B.I32), want)
    # in the kernel's association: (gamma s_x) / 127, IEEE (torch multiplies by a reciprocal)
    scale = (gamma_rb.repeat_interleave(16)[:N].cpu().numpy()[None, :] * sx.cpu().numpy()[:, None]) / np.float32(127.0)
    assert torch.equal(B.linear_segmented(xq, sx, packed, gamma_rb, N, y_dtype=B.F32), want.float() * torch.from_numpy(scale).cuda())
