"""S_B and its gradients in complex128 as sums over point differences, against the array passes of the same library."""
from __future__ import annotations

import math

import pytest
import torch

import wolf_inputs as WI
from paper_2203_02734_amd import autograd as A

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("farfield", [False, True])
@pytest.mark.parametrize("n", [2, 4, 8, 16, 32, 64, 128])  # 64 on: four outputs per thread; up to 4: fewer rows
def test_fit_sums_match_the_arrays(gpu_lib, n, farfield):
    """Both sides sum N^4 FP64 products: S_B, dL/dI and dL/dsigma to 1e-11 (the float32 d_imap to its rounding)."""
    p, z, lam, sg = 20e-6, 0.3, WI.LAMBDA_HENE, 0.08e-3
    imap = torch.from_numpy(WI.intensity_map(n, p, seed=n, env_sigma_m=p * n / 4)).cuda()
    w = gpu_lib.build_source(A._map_source(imap, sg), n, p, torch.complex128)
    gpu_lib.propagate(w, p, lam, z, farfield, out=w)
    s_ref = gpu_lib.spectral_density(w)
    s, corr = gpu_lib.fit_forward(imap, p, sg, lam, z, farfield)
    assert float((s - s_ref).norm() / s_ref.norm()) < 1e-11
    g = torch.from_numpy(WI.rng(n).standard_normal((n, n))).cuda()
    di_ref, ds_ref = gpu_lib.fit_gradient(gpu_lib.propagate_adjoint_diag(g, p, lam, z, farfield, dtype=torch.complex128),
                                          imap, p, sg)
    di, ds = gpu_lib.fit_backward(g, imap, corr, p, sg, lam, z, farfield)
    assert float((di.double() - di_ref.double()).norm() / di_ref.double().norm()) < 2.0 ** -23
    # dL/dsigma is a sum of N^4 terms of both signs: its rounding is relative to the sum of their sizes, at most
    # |g| S of the incoherent map, here bounded through |S_B| and the largest |delta|^2.
    scale = float(g.abs().sum() * s_ref.abs().max()) * 2 * (n * p) ** 2 / sg ** 3
    assert abs(float(ds - ds_ref)) < 1e-11 * scale


def test_fit_sums_limits(gpu_lib):
    n, p, lam, z = 16, 20e-6, WI.LAMBDA_HENE, 0.3
    imap = torch.from_numpy(WI.intensity_map(n, p, seed=1)).cuda()
    w = gpu_lib.build_source(A._map_source(imap, math.inf), n, p, torch.complex128)
    gpu_lib.propagate_fresnel(w, p, lam, z, out=w)
    s, corr = gpu_lib.fit_forward(imap, p, math.inf, lam, z)  # a fully coherent source
    assert float((s - gpu_lib.spectral_density(w)).norm() / s.norm()) < 1e-11
    with pytest.raises(gpu_lib.WolfError):
        gpu_lib.fit_backward(s, imap, corr, p, math.inf, lam, z)
    with pytest.raises(gpu_lib.WolfError):
        gpu_lib.fit_forward(imap, p, -1.0, lam, z)
    with pytest.raises(ValueError):
        gpu_lib.fit_forward(imap[:8], p, 1e-4, lam, z)
    with pytest.raises(gpu_lib.WolfError):
        gpu_lib.fit_forward(torch.ones((6, 6), device="cuda"), p, 1e-4, lam, z)
    big = torch.ones((256, 256), device="cuda")
    s, corr = gpu_lib.fit_forward(big, p, 1e-4, lam, z)
    assert bool(torch.isfinite(s).all())
    with pytest.raises(gpu_lib.WolfError):
        gpu_lib.fit_backward(s, big, corr, p, 1e-4, lam, z)
