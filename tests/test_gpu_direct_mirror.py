"""The mirrored form of the exact-kernel direct sum (N >= 16) on an input without any symmetry, in place and out of
place, against the FP64 oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as O
import wolf_inputs as WI
from tests.test_gpu_direct import fp32_bound, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n", [8, 16, 32])  # 8: the plain products; 16: one ragged tile per class; 32: several
def test_direct_no_symmetry_in_place(gpu_lib, n, dtype):
    p, z, lam = 20e-6, 4e-3, WI.LAMBDA_HENE
    w = WI.random_complex((n, n, n, n), seed=70 + n)
    ref, _ = O.propagate_direct(w, n, p, lam, z, O.KIND_SECONDARY)
    a = torch.from_numpy(w).to(dtype).cuda()
    keep = a.clone()
    out, _ = gpu_lib.propagate_direct(a, p, lam, z)
    torch.cuda.synchronize()
    assert torch.equal(a, keep)
    # complex64: the product bound, and one rounding more per folded and unfolded axis (8 u of the result).
    tol = 1e-12 if dtype == torch.complex128 else fp32_bound(w, n, p, z, O.KIND_SECONDARY) + 8 * 2.0 ** -24
    assert rel(out.cpu().numpy(), ref) < tol
    gpu_lib.propagate_direct(a, p, lam, z, out=a)
    torch.cuda.synchronize()
    assert torch.equal(out, a)
