"""Prefill on rows of a few bytes, with a few tokens behind a whole tile of 64: the last pieces of the tile in front of the last one
reach the end of x_q too.  Integer products: exact."""
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("M,N", [(1025, 1024), (1026, 1030), (1030, 1024), (1039, 1500), (129, 8000), (131, 16000), (65, 20000), (71, 20001), (4097, 4096)])
def test_rows_of_a_few_columns(gpu_lib, M, N):
    served = 0
    for K in range(1, 18):
        if B.linear_describe(M, N, K)["kernel"] != "prefill_any":
            continue
        served += 1
        g = torch.Generator(device="cuda").manual_seed(M + N + K)
        packed, gamma = B.quantize_weights(torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g))
        xq = torch.randint(-127, 128, (M, K), device="cuda", generator=g, dtype=torch.int32).to(torch.int8)
        want = (xq.float() @ B.unpack_weights(packed, N, K).float().t()).to(torch.int32)
        print("few columns", M, N, K, flush=True)
        assert torch.equal(B.linear(xq, torch.ones(M, device="cuda"), packed, gamma, N, y_dtype=B.I32), want), K
    assert served >= 5
