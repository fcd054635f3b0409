"""The order of the complex64 sums behind S and mu of the batch and S of the common-grid sum, pinned by its bits.

mu is zero where S <= floor_rel max S. In FP32 a sum of N^4 products carries 1e-7 of max S, so any other order of the same sums
moves points whose S lies there to the other side of the floor, and mu at them jumps between zero and its value. The bits of S
are therefore part of what a caller sees. The digests are those of the register-ring and LDS-staged 3M products; the inputs are
twelve-bit numbers formed by integer arithmetic, the same bits everywhere."""
from __future__ import annotations

import hashlib

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P, LAM, FLOOR = 20e-6, 600e-9, 0.75


def source(n, dtype=torch.complex64):
    """Twelve-bit entries without any symmetry, and a diagonal that keeps S positive and within a few per cent of its mean."""
    w = torch.empty((n * n, n * n, 2), dtype=torch.float32, device="cuda")
    c = torch.arange(2 * n * n, dtype=torch.int64, device="cuda")
    for p in range(n * n):
        w[p] = ((((c + p * 2 * n * n) * 2654435761 % 4294967296) >> 20).to(torch.float32) / 2048 - 1).reshape(n * n, 2)
    d = torch.arange(n * n, device="cuda")
    w[d, d, 0] += 8
    return torch.view_as_complex(w).reshape(n, n, n, n).to(dtype)


def pairs_of(k):
    i = np.arange(k)
    return LAM * (0.8 + 0.4 * ((7 * i) % 11) / 11), 0.05 + 0.4 * ((5 * i) % 13) / 13, 0.5 + (i % 3)


def observe(lib, kind, n, k, floor=FLOOR):
    w = source(n)
    lam, z, wt = pairs_of(k)
    if kind == "batch":
        return lib.propagate_batch(w, P, lam, z, wt, ip=n // 2 + 1, jp=n // 2 - 2, floor_rel=floor)
    return lib.propagate_polychromatic(w, P, lam, z, wt, LAM * 0.3 / (n * P), ip=n // 2 + 1, jp=n // 2 - 2, floor_rel=floor)


def digest(t):
    return hashlib.sha256(t.cpu().numpy().tobytes()).hexdigest()[:16]


# (kind, N, pairs): S. The tiles of 16, 32 and 64 pairs at the two sizes that have kernels of their own, ragged counts.
S_BITS = {
    ("batch", 64, 2): "18b1c1a4a8e4aa35", ("batch", 64, 20): "0093866745fe65ba", ("batch", 64, 40): "caf0f4c16fc46ed5",
    ("batch", 128, 5): "95cd81dd0a39a534", ("batch", 128, 20): "008fe4f40607f8d8", ("batch", 128, 40): "87c46e8fa3846175",
    ("poly", 64, 3): "edbe91b7b274b589", ("poly", 64, 20): "70623c337f558f99", ("poly", 64, 40): "1b8d0a3ba8ae76ad",
    ("poly", 128, 5): "a4a484a035b0c23a", ("poly", 128, 20): "a93c891252ead889", ("poly", 128, 40): "f76629e709fb072c",
}


@pytest.mark.parametrize("kind,n,k", sorted(S_BITS))
def test_s_keeps_its_bits(gpu_lib, kind, n, k):
    assert digest(observe(gpu_lib, kind, n, k)[0]) == S_BITS[kind, n, k]


# (N, pairs): mu of the batch above a floor of zero. Its row sums take phase times chirp as one FP64-built weight; rounding the
# two by themselves, and W again on the way, made W(P, .) of a beam at N = 128 up to a quarter less exact.
MU_BITS = {
    (32, 3): "6cb0e81c58d69826", (32, 33): "ebf421d20ef70c11", (64, 20): "2855c58834da01b4", (64, 40): "9349f45b33291c54",
    (128, 5): "4ed41074817165d0", (128, 20): "4f0e342c91edadfb", (128, 40): "e59332bee57ca986",
}


@pytest.mark.parametrize("n,k", sorted(MU_BITS))
def test_batch_mu_keeps_its_bits(gpu_lib, n, k):
    s, mu = observe(gpu_lib, "batch", n, k, 0.0)
    assert int((mu != 0).sum()) > 0.9 * mu.numel()
    assert digest(mu) == MU_BITS[n, k]
