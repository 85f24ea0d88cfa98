"""GPU tests of the batched-decode kernel whose waves share out the K steps (csrc/linear_ksplit.hip): every built form at tokens and
rows that fill its tiles and that do not, K from one step (seven waves without any) over as many as there are waves to a whole round
and one, a last step of one to four quads; against the exact integer product."""
import numpy as np
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (tokens, rows) -> token tiles, row blocks as two factors, waves as kS groups of kW
FORMS = [(9, 4096, [1, 1, 1, 8]), (48, 30, [1, 1, 1, 8]), (30, 4000, [1, 1, 2, 4]), (16, 9999, [1, 2, 2, 4]), (57, 4090, [1, 2, 2, 4]),
         (17, 260, [2, 1, 1, 8]), (200, 250, [2, 1, 1, 8]), (140, 1530, [2, 1, 2, 4]), (29, 12288, [2, 2, 2, 4]), (128, 4093, [2, 2, 2, 4]),
         (20, 17000, [2, 6, 1, 8]), (190, 3300, [2, 6, 1, 8]), (63, 441, [4, 1, 1, 8]), (110, 8010, [4, 4, 1, 8]), (211, 4000, [4, 4, 1, 8]),
         (67, 12900, [5, 4, 1, 8]), (300, 4096, [5, 4, 1, 8])]


@pytest.mark.parametrize("M,N,form", FORMS)
@pytest.mark.parametrize("K", [16, 64, 144, 1872, 2048, 2064, 4160, 6224, 11008])
def test_forms_against_the_exact_product(gpu_lib, M, N, form, K):
    d = B.linear_describe(M, N, K)
    if form[0] != 5 or K > 1536:                           # tiles of 80 tokens are taken from seven K steps on
        assert (d["kernel"], d["params"][:4]) == ("batched_decode", form)
    g = torch.Generator(device="cuda").manual_seed(M * N + K)
    rows = [(N + 31) // 32 * 16, N - (N + 31) // 32 * 16] if N > 32 else [N]
    packed, gamma_rb = B.quantize_weights_segmented(torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g), rows)
    xq, sx = B.quantize_acts(torch.randn((M, K), device="cuda", generator=g))
    want = (xq.double() @ B.unpack_weights(packed, N, K).double().t()).to(torch.int32)
    print("ksplit", M, N, K, flush=True)
    one = torch.ones(1, device="cuda")
    assert torch.equal(B.linear(xq, sx, packed, one, N, y_dtype=B.I32), want)
    # a gamma per row block, in the kernel's association: (gamma s_x) / 127 (the prefill kernel: gamma (s_x / 127)), IEEE (torch multiplies by a reciprocal)
    gamma = gamma_rb.repeat_interleave(16)[:N].cpu().numpy()
    sxn = sx.cpu().numpy()[:, None]
    scale = gamma[None, :] * (sxn / np.float32(127.0)) if d["kernel"] == "prefill" else (gamma[None, :] * sxn) / np.float32(127.0)
    assert torch.equal(B.linear_segmented(xq, sx, packed, gamma_rb, N, y_dtype=B.F32), want.float() * torch.from_numpy(scale).cuda())
    # outputs that cannot be stored four at a time, and nothing written around them
    room = torch.full((M * N + 9,), 77, dtype=torch.bfloat16, device="cuda")
    B.linear(xq, sx, packed, one, N, y_dtype=B.BF16, y=room[1:1 + M * N].view(M, N))
    assert torch.equal(room[1:1 + M * N].view(M, N), B.linear(xq, sx, packed, one, N, y_dtype=B.BF16))
    assert (room[:1] == 77).all() and (room[1 + M * N:] == 77).all()


@pytest.mark.parametrize("M,N,K,kernel", [(257, 1024, 2048, "batched_decode"), (480, 2048, 2048, "batched_decode"), (300, 4096, 4096, "batched_decode"),
                                          (280, 4096, 256, "prefill"), (280, 4096, 1552, "batched_decode"), (300, 2700, 2048, "prefill"), (257, 4096, 4096, "prefill")])
def test_short_k_beyond_256_tokens(gpu_lib, M, N, K, kernel):
    """where these kernels are taken without a split-K form: forced ones go to the prefill kernel, KERNEL_GEMV stays refused"""
    assert B.linear_describe(M, N, K)["kernel"] == kernel
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    packed, gamma = B.quantize_weights(torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g))
    xq, sx = B.quantize_acts(torch.randn((M, K), device="cuda", generator=g))
    want = (xq.double() @ B.unpack_weights(packed, N, K).double().t()).to(torch.int32)
    print("short k", M, N, K, flush=True)
    assert torch.equal(B.linear(xq, sx, packed, gamma, N, y_dtype=B.I32), want)
    ws = torch.empty(2 * M * N * 4, dtype=torch.uint8, device="cuda")
    assert torch.equal(B.linear_ws(xq, sx, packed, gamma, N, ws, y_dtype=B.I32), want)
    if K >= 512:
        assert torch.equal(B.linear_ws(xq, sx, packed, gamma, N, ws, y_dtype=B.I32, kernel=B.KERNEL_GEMM_SPLITK[2]), want)
    with pytest.raises(B.BitnetError):
        B.linear(xq, sx, packed, gamma, N, y_dtype=B.I32, kernel=B.KERNEL_GEMV)
