"""GPU tests of the fused decode launches of one to four tokens: every launch shape at the edges of its range (row blocks and K
steps where the selection changes, remainders of both, the last vectors a thread holds), bit for bit against the kernels that
serve more tokens or int8 input, which the oracle pins."""
import pytest

import oracle
from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# N x K (the pair: F x K): 2 ... 3126 row blocks, 1 ... 64 steps
SHAPES = [(17, 16), (250, 2048), (4096, 2064), (4090, 4096), (100, 4112), (300, 8640), (33, 12304), (4112, 1024), (8192, 1040), (8190, 2048), (5000, 2064),
          (8192, 5120), (8208, 1024), (9600, 2560), (9600, 3200), (16384, 4112), (16400, 272), (20000, 5120), (32784, 1280), (33000, 6144), (49168, 528), (50001, 2576), (50001, 6160)]


def inputs(M, N, K, bf16, seg):
    g = torch.Generator(device="cuda").manual_seed(N * 31 + K)
    W = torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g)
    x = torch.randn((M, K), device="cuda", generator=g)
    x[:, :: 97] *= 20.0
    x[:, -1] = 30.0                                          # the last column of a row decides its scale
    gain = 1.0 + 0.1 * torch.randn(K, device="cuda", generator=g)
    w = B.quantize_weights_segmented(W, [N - N // 2 // 16 * 16, N // 2 // 16 * 16]) if seg else B.quantize_weights(W)
    return x.to(torch.bfloat16) if bf16 else x, w, gain


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("N,K", SHAPES)
def test_rows(gpu_lib, N, K, bf16):
    seg = N % 64 == 0
    x, w, gain = inputs(4, N, K, bf16, seg)
    lin, fused = (B.linear_segmented, B.linear_fused_segmented) if seg else (B.linear, B.linear_fused)
    for M in (1, 2, 3, 4):
        xm = x[4 - M:].contiguous()
        q, qn, qg = B.quantize_acts(xm), B.rmsnorm_quantize(xm, None, 1e-6), B.rmsnorm_quantize(xm, gain, 1e-5)
        # eps = 0, with three tokens beside a fourth that is not there
        assert torch.equal(B.rmsnorm_linear_fused(xm, gain, 0.0, *w, N, segmented=seg), lin(*B.rmsnorm_quantize(xm, gain, 0.0), *w, N))
        for y in (B.F32, B.BF16, B.I32):
            print("rows", M, N, K, bf16, y, flush=True)
            assert torch.equal(fused(xm, *w, N, y_dtype=y), lin(*q, *w, N, y_dtype=y))
            assert torch.equal(B.rmsnorm_linear_fused(xm, None, 1e-6, *w, N, y_dtype=y, segmented=seg), lin(*qn, *w, N, y_dtype=y))
            assert torch.equal(B.rmsnorm_linear_fused(xm, gain, 1e-5, *w, N, y_dtype=y, segmented=seg), lin(*qg, *w, N, y_dtype=y))


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("F,K", [(N // 16 * 16, K) for (N, K) in SHAPES if N <= 33000 and 5 * K <= 64000] + [(8640, 8208), (1504, 9216), (4096, 6144), (12320, 6160), (12320, 8208)])
def test_pairs(gpu_lib, F, K, bf16):
    """five tokens go through the kernel that serves more than four: their first rows"""
    seg = F % 64 == 0
    x, w, gain = inputs(5, 2 * F, K, bf16, seg)
    for norm, g in ((False, None), (True, None), (True, gain)):
        for h in (B.F32, B.BF16):
            want = B.ffn_gate_up_fused(x, *w, F, norm=norm, g=g, eps=1e-6, gamma_per_block=seg, h_dtype=h)
            for M in (1, 2, 3, 4):
                print("pairs", M, F, K, bf16, norm, h, flush=True)
                assert torch.equal(B.ffn_gate_up_fused(x[:M].contiguous(), *w, F, norm=norm, g=g, eps=1e-6, gamma_per_block=seg, h_dtype=h), want[:M])


@pytest.mark.parametrize("F,K", [(8208, 18448), (11008, 20480), (16384, 24576)])
def test_pairs_of_rows_beyond_64_steps(gpu_lib, F, K):
    """the most vectors a thread of twelve or sixteen waves holds, and three tokens beyond that: the gate applied to the outputs of the
    plain fused launch, bit for bit"""
    x, w, gain = inputs(3, 2 * F, K, True, False)
    for M in (1, 2, 3):
        if 512 + M * ((K + 255) // 256) * 256 > 65536:
            continue
        xm = x[:M].contiguous()
        for norm in (False, True):
            print("long pairs", M, F, K, norm, flush=True)
            y = B.rmsnorm_linear_fused(xm, gain, 1e-6, *w, 2 * F) if norm else B.linear_fused(xm, *w, 2 * F)
            h = B.ffn_gate_up_fused(xm, *w, F, norm=norm, g=gain if norm else None, eps=1e-6)
            assert h.cpu().numpy().tobytes() == oracle.swiglu_quantize(y.cpu().numpy())[2].tobytes()
