"""The one-launch mu slice (N <= 64) and the three-launch one above it equal the same row of the full mu bit for bit."""
from __future__ import annotations

import pytest
import torch

import wolf_inputs as WI

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n", [2, 4, 10, 32, 62, 64, 66])
def test_slice_is_a_row_of_the_full_mu(gpu_lib, n, dtype):
    g = torch.Generator(device="cuda").manual_seed(n)
    w = torch.view_as_complex(torch.randn((n, n, n, n, 2), generator=g, device="cuda", dtype=torch.float32)).to(dtype)
    d = torch.arange(n * n, device="cuda")
    w.view(n * n, n * n)[d, d] = torch.rand(n * n, generator=g, device="cuda").to(dtype) - 0.2  # some S below zero
    for floor in (0.0, 0.3):
        full = gpu_lib.degree_of_coherence(w, -1, -1, floor)
        s = gpu_lib.spectral_density(w)
        top, low = divmod(int(s.argmax()), n), divmod(int(s.argmin()), n)
        for ip, jp in ((0, 0), (n - 1, n - 1), top, low):
            got = gpu_lib.degree_of_coherence(w, ip, jp, floor)
            assert torch.equal(got, full[ip, jp])
            assert torch.equal(got != 0, (full[ip, jp] != 0))
        assert bool((gpu_lib.degree_of_coherence(w, *top, floor) != 0).any())
        assert not bool((gpu_lib.degree_of_coherence(w, *low, floor) != 0).any())
    w.view(n * n, n * n)[d, d] = float("nan")
    assert torch.equal(gpu_lib.degree_of_coherence(w, 0, 1, 0.1) != 0, gpu_lib.degree_of_coherence(w, -1, -1, 0.1)[0, 1] != 0)
