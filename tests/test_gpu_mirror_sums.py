"""The mirrored contractions of the batch and of the common-grid sum against the propagation operator, on a source without
any symmetry: each size of the pair tiles, both precisions, probe points at the edges of the grid."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import wolf_inputs as WI

pytestmark = pytest.mark.gpu

P, LAM = 20e-6, 600e-9
# (N, pairs, probe): pair tiles of 16, 32 and 64 with ragged counts, two groups; the corner, the middle, the last point.
CASES = [(32, 2, (0, 0)), (32, 33, (16, 31)), (64, 16, (31, 1)), (64, 17, (0, 32)), (64, 65, (63, 63)), (128, 3, (64, 0)),
         (128, 40, (127, 5))]


def source(n, dtype):
    """Random complex entries, fixed over the cases of one N."""
    g = torch.Generator(device="cuda").manual_seed(n)
    w = torch.randn((n, n, n, n, 2), generator=g, device="cuda", dtype=torch.float32)
    return torch.view_as_complex(w).to(dtype)


def pairs_of(k):
    i = np.arange(k)
    return LAM * (0.8 + 0.4 * ((7 * i) % 11) / 11), 0.05 + 0.4 * ((5 * i) % 13) / 13, 0.5 + (i % 3)


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n,k,probe", CASES)
def test_batch_without_symmetry(gpu_lib, n, k, probe, dtype):
    """S of three pairs against the operator; W(P, .) through mu where S is not small. Each S is a sum of N^4 random terms
    whose rounding is u times the root of the sum of their squares, as the sum itself is: a few u sqrt(log N^4), with the
    FP32 chain of up to 4 N terms 40 u at most."""
    w = source(n, dtype)
    lam, z, wt = pairs_of(k)
    s, mu = gpu_lib.propagate_batch(w, P, lam, z, wt, ip=probe[0], jp=probe[1], floor_rel=1e-2)
    u = 2.0 ** -24 if dtype == torch.complex64 else 2.0 ** -53
    for q in {0, k // 2, k - 1}:
        wb, _ = gpu_lib.propagate_fresnel(w.to(torch.complex128), P, lam[q], z[q])
        sref = wt[q] * gpu_lib.spectral_density(wb)
        assert float((s[q].double() - sref).norm() / sref.norm()) < max(100 * u, 1e-12)
        mref = gpu_lib.degree_of_coherence(wb, *probe, 1e-2)
        both = (mu[q] != 0) & (mref != 0)
        if bool(both.any()):
            d = (mu[q] - mref)[both]
            assert float(d.norm() / mref[both].norm()) < max(2e4 * u, 1e-10)
        assert int((both != (mref != 0)).sum()) <= n  # points at the floor may fall on either side


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n,k", [(64, 2), (64, 33), (128, 5), (128, 64)])
def test_poly_equals_batch_without_symmetry(gpu_lib, n, k, dtype):
    """Pairs of one product lambda z share their FFT grid: the common-grid S is the sum of the batch's."""
    w = source(n, dtype)
    lam, _, wt = pairs_of(k)
    z = LAM * 0.3 / lam
    s, _ = gpu_lib.propagate_batch(w, P, lam, z, wt, ip=1, jp=n - 1)
    sp, _ = gpu_lib.propagate_polychromatic(w, P, lam, z, wt, LAM * 0.3 / (n * P), ip=1, jp=n - 1)
    ref = s.double().sum(0)
    tol = 100 * 2.0 ** -24 if dtype == torch.complex64 else 1e-12
    assert float((sp.double() - ref).norm() / ref.norm()) < tol
