"""The constant table of silu's bf16 values against the arithmetic of the fp32 form: the bits of every entry.  A token with one nonzero
gate has that value as its scale, and up = 2^16 lifts it over the scale's floor exactly."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,per_call", [(9216, 170), (16640, 94)])
def test_every_entry_of_the_silu_table(gpu_lib, F, per_call):
    B = gpu_lib
    low, high = (127 - 15) << 7, (127 + 8) << 7
    bits = torch.cat([torch.tensor([0]), torch.arange(low, high + 1)])
    bits = torch.cat([bits, bits | 0x8000]).to(torch.int32)
    values = (bits << 16).view(torch.float32).bfloat16()
    assert torch.equal(values.view(torch.int16).int() & 0xFFFF, bits)
    for at in range(0, len(values), per_call):
        v = values[at:at + per_call].cuda()
        gu = torch.zeros(len(v), 2 * F, dtype=torch.bfloat16, device="cuda")
        col = torch.arange(at, at + len(v), device="cuda") % F
        rows = torch.arange(len(v), device="cuda")
        gu[rows, col] = v
        gu[:, F:] = 2.0 ** 16
        hq, sh = B.swiglu_quantize(gu)
        hq32, sh32 = B.swiglu_quantize(gu.float())
        assert torch.equal(sh, sh32) and torch.equal(hq, hq32)
