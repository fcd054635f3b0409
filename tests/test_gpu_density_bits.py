"""S alone has the bits of the propagated array's diagonal at every size, N = 256 among them, and under the schedules of N = 128."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def fill(w, seed):
    g = torch.Generator(device="cuda")
    v = torch.view_as_real(w)
    for i in range(w.shape[0]):
        v[i] = torch.randn(v[i].shape, generator=g.manual_seed(seed + i), device="cuda", dtype=torch.float32)


@pytest.mark.parametrize("farfield", [False, True])
@pytest.mark.parametrize("n,dtype,plan", [(256, torch.complex64, None), (256, torch.complex128, None),
                                          (128, torch.complex64, (3, 0, 1024)), (128, torch.complex64, (1, 0, 16384)),
                                          (128, torch.complex64, (0, 256, 512)), (128, torch.complex128, (3, 2048, 1024)),
                                          (128, torch.complex128, (0, 256, 16384)), (32, torch.complex64, (0, 64, 256))])
def test_density_bits(gpu_lib, n, dtype, plan, farfield):
    w = torch.empty((n,) * 4, dtype=dtype, device="cuda")
    if plan:
        gpu_lib.set_plan(n, dtype, *plan)
    try:
        fill(w, n)
        s = gpu_lib.propagate_density(w, 2e-5, 633e-9, 0.3, farfield)
        fill(w, n)
        gpu_lib.propagate(w, 2e-5, 633e-9, 0.3, farfield, out=w)
        ref = gpu_lib.spectral_density(w)
    finally:
        if plan:
            gpu_lib.set_plan(n, dtype)
    assert torch.equal(s, ref)
    del w
    torch.cuda.empty_cache()
