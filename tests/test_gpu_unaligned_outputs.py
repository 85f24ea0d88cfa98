"""GPU tests of output rows at every alignment: N that is no multiple of the 16-byte stores, and a base one output past an aligned one,
through every product kernel -- the exact integers, and nothing written outside of them."""
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [("prefill", 300, 9601, 1536, B.PACK_2BIT), ("prefill", 200, 22019, 528, B.PACK_2BIT), ("prefill", 600, 6150, 768, B.PACK_2BIT),
         ("prefill", 520, 5123, 5120, B.PACK_2BIT), ("prefill", 1024, 15357, 512, B.PACK_2BIT), ("prefill", 130, 70001, 256, B.PACK_2BIT),
         ("batched_decode", 30, 5127, 1024, B.PACK_2BIT), ("batched_decode", 8, 20003, 512, B.PACK_2BIT), ("batched_decode_loader", 64, 30001, 768, B.PACK_2BIT),
         ("decode", 3, 4099, 2048, B.PACK_2BIT), ("decode", 7, 517, 1024, B.PACK_2BIT), ("decode_any", 77, 1003, 1025, B.PACK_2BIT),
         ("prefill_any", 300, 2501, 515, B.PACK_2BIT), ("trit5_decode", 4, 4097, 640, B.PACK_TRIT5), ("trit5_decode", 9, 27645, 3200, B.PACK_TRIT5)]


@pytest.mark.parametrize("kernel,M,N,K,fmt", CASES)
def test_rows_at_every_alignment(gpu_lib, kernel, M, N, K, fmt):
    assert B.linear_describe(M, N, K, fmt=fmt)["kernel"] == kernel
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    packed, gamma = B.quantize_weights(torch.empty((N, K), device="cuda").normal_(0.0, 0.02, generator=g), fmt)
    xq, sx = B.quantize_acts(torch.randn((M, K), device="cuda", generator=g))
    want = (xq.double() @ B.unpack_weights(packed, N, K, fmt).double().t()).to(torch.int32)
    print("unaligned", kernel, M, N, K, flush=True)
    for y_dtype, dtype in ((B.I32, torch.int32), (B.F32, torch.float32), (B.BF16, torch.bfloat16)):
        y = B.linear(xq, sx, packed, gamma, N, fmt=fmt, y_dtype=y_dtype)
        if y_dtype == B.I32:
            assert torch.equal(y, want)
        else:
            # three fp32 roundings (gamma s_x, its quotient by 127, the product), and bf16's own: eight significant bits, so half a spacing is
            # up to 2^-8 of a value
            scaled = want.double() * (gamma.double() * sx.double() / 127.0)[:, None]
            assert ((y.double() - scaled).abs() <= scaled.abs() * (4 * 2.0 ** -24 + (2.0 ** -8 if y_dtype == B.BF16 else 0.0))).all()
        for off in (1, 3):
            room = torch.full((M * N + 16,), 77, dtype=dtype, device="cuda")
            B.linear(xq, sx, packed, gamma, N, fmt=fmt, y_dtype=y_dtype, y=room[off:off + M * N].view(M, N))
            assert torch.equal(room[off:off + M * N].view(M, N), y) and (room[:off] == 77).all() and (room[off + M * N:] == 77).all()
