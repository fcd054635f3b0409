"""S without the rest of the propagated array against the propagation and its diagonal, under every schedule."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("farfield", [False, True])
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n,plan", [(2, None), (4, None), (8, None), (16, None), (32, None), (64, None), (128, None),
                                    (64, (1, 0, 512)), (64, (0, 128, 512)), (64, (3, 0, 4096, 16))])
def test_density_equals_diagonal(gpu_lib, n, plan, dtype, farfield):
    """The same sums in the same order: no difference."""
    g = torch.Generator(device="cuda").manual_seed(n)
    w = torch.view_as_complex(torch.randn((n, n, n, n, 2), generator=g, device="cuda", dtype=torch.float32)).to(dtype)
    if plan and plan[0] == 1 and dtype == torch.complex128:
        plan = (3,) + plan[1:]
    if plan:
        gpu_lib.set_plan(n, dtype, *plan)
    try:
        ref = gpu_lib.spectral_density(gpu_lib.propagate(w.clone(), 2e-5, 633e-9, 0.3, farfield)[0])
        s = gpu_lib.propagate_density(w, 2e-5, 633e-9, 0.3, farfield)
    finally:
        if plan:
            gpu_lib.set_plan(n, dtype)
    assert torch.equal(s, ref)
