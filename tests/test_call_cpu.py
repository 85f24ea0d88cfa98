"""The native argument marshalling of the binding refuses what it always refused, with the same exception types: here as far
as that can be seen without a GPU (every tensor argument has to be on one)."""
import pytest
import torch

from paper_2402_17764_amd import binding as B

CPU_X = torch.zeros(2, 64)
CPU_Q = torch.zeros(2, 64, dtype=torch.int8)


@pytest.mark.parametrize("call", [
    lambda t: B.quantize_acts(t), lambda t: B.rmsnorm_quantize(t), lambda t: B.swiglu_quantize(t),
    lambda t: B.linear(t, t, t, t, 16), lambda t: B.linear_segmented(t, t, t, t, 16), lambda t: B.linear_ws(t, t, t, t, 16, None),
    lambda t: B.linear_fused(t, t, t, 16), lambda t: B.linear_fused_segmented(t, t, t, 16),
    lambda t: B.rmsnorm_linear_fused(t, None, 1e-6, t, t, 16), lambda t: B.swiglu_linear_fused(t, t, t, 16),
    lambda t: B.ffn_gate_up_fused(t, t, t, 16)])
@pytest.mark.parametrize("arg", [CPU_X, CPU_Q, None, 3, "x"])
def test_only_gpu_tensors(call, arg):
    with pytest.raises(TypeError, match="must be a CUDA/HIP tensor"):
        call(arg)
