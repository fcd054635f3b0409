"""The centred chirp-z transforms of the common-grid sum on the FFT grid against the propagation operator, on a source without
any symmetry, at every number of threads that a row takes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P, LZ = 20e-6, 600e-9 * 0.3


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n,k", [(2, 1), (2, 3), (4, 2), (8, 1), (16, 5), (32, 3), (64, 1), (128, 1)])
def test_fft_grid_equals_operator(gpu_lib, n, k, dtype):
    """Pairs of one product lambda z share the grid of pitch lambda z / (N P). Sums of N^4 random terms, rounded as in the
    operator by a few u of their root sum of squares: 100 u, and in FP64 10^-12 for the chain of 2 N factors."""
    g = torch.Generator(device="cuda").manual_seed(n)
    w = torch.view_as_complex(torch.randn((n, n, n, n, 2), generator=g, device="cuda", dtype=torch.float32)).to(dtype)
    lam = 600e-9 * (1 + 0.1 * np.arange(k))
    z, wt = LZ / lam, 1.0 + 0.5 * np.arange(k)
    s, mu = gpu_lib.propagate_polychromatic(w, P, lam, z, wt, LZ / (n * P), ip=n - 1, jp=n // 2, floor_rel=1e-2)
    total = 0
    for i in range(k):
        total = total + wt[i] * gpu_lib.propagate_fresnel(w.to(torch.complex128), P, lam[i], z[i])[0]
    sref = gpu_lib.spectral_density(total)
    u = 2.0 ** -24 if dtype == torch.complex64 else 2.0 ** -53
    assert float((s.double() - sref).norm() / sref.norm()) < max(100 * u, 1e-12)
    mref = gpu_lib.degree_of_coherence(total, n - 1, n // 2, 1e-2)
    both = (mu != 0) & (mref != 0)
    if bool(both.any()):
        assert float((mu - mref)[both].norm() / mref[both].norm()) < max(2e4 * u, 1e-10)
