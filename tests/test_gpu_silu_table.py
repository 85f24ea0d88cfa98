"""The constant table of silu's bf16 values against the arithmetic of the fp32 form: the bits of every entry.  A token with one nonzero
gate has that value as its scale, lifted over the scale's floor by a power of two: 2^16, and 2^120 for the gates below -20, whose
values are down to 2^-119."""
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
        gu[:, F:] = torch.where(v < -20.0, 2.0 ** 120, 2.0 ** 16).to(torch.bfloat16)[:, None]
        hq, sh = B.swiglu_quantize(gu)
        hq32, sh32 = B.swiglu_quantize(gu.float())
        assert torch.equal(sh, sh32) and torch.equal(hq, hq32)
        # nothing hides under the floor: the scale is the value, and its code the largest
        seen = v != 0
        assert (sh[seen] > 1e-5).all() and (hq[rows, col].abs()[seen] == 127).all()
