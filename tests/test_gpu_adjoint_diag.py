"""The operator on diag(g): the first-point pass that forms its own input, over the plans that launch it differently."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# Two orders of the same four passes: 4 (2 log2 N + 3) <= 68 roundings of eps/2 on a way, far below 100 eps of the largest
# value (the errors are independent, and most values are much smaller than the largest).
TOL = {torch.complex64: 100 * 2.0 ** -23, torch.complex128: 100 * 2.0 ** -52}


# column chunks: the plan's own (0), one launch each, pairs of launches, pairs and ends
@pytest.mark.parametrize("n,chunks", [(2, 0), (8, 0), (32, 0)] + [(n, c) for n in (64, 128) for c in (0, 1, 2, 8)])
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
def test_formed_input_equals_embedded(gpu_lib, n, dtype, chunks):
    real = torch.float32 if dtype == torch.complex64 else torch.float64
    g = torch.randn((n, n), generator=torch.Generator().manual_seed(n), dtype=torch.float64).to(real).cuda()
    ref = gpu_lib.propagate_adjoint(gpu_lib.diag_embed(g, dtype), 2e-5, 633e-9, 0.3, False)
    if chunks:
        plan = gpu_lib.get_plan(n, dtype)
        gpu_lib.set_plan(n, dtype, plan["fused_slab"], plan["slab_chunk"], n * n // chunks)
    try:
        out = gpu_lib.propagate_adjoint_diag(g, 2e-5, 633e-9, 0.3, False, dtype=dtype)
    finally:
        if chunks:
            gpu_lib.set_plan(n, dtype)
    assert (out - ref).abs().max() <= TOL[dtype] * ref.abs().max()
