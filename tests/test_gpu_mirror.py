"""The mirrored dense passes (any N_z without an FFT split) against the FP64 separable oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as O
import wolf_inputs as WI
from tests.gpu_util import separable_rel

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
# N at the ends of the buckets of contraction steps (c = N/2 in 4 KJ - 4 .. 4 KJ - 1 at KJ = 5, 9, .., 33), of the
# output tiles (c + 1 = 16, 17), and the smallest and largest; N_z odd, even, N itself and the largest.
C64 = [(2, 3), (4, 5), (14, 14), (30, 31), (32, 33), (38, 45), (40, 41), (70, 71), (72, 90), (102, 2047), (104, 104),
       (134, 134), (136, 150), (166, 166), (168, 170), (198, 203), (230, 230), (232, 240), (256, 300)]
C128 = [(2, 3), (30, 30), (38, 46), (40, 42), (70, 2046), (72, 75), (102, 103), (104, 110), (134, 134), (136, 140),
        (166, 167), (200, 202), (232, 234), (256, 258)]


@pytest.mark.parametrize("n,nz,dtype", [(*c, torch.complex64) for c in C64] + [(*c, torch.complex128) for c in C128])
def test_mirror_passes(gpu_lib, n, nz, dtype):
    """W = wx wy with random complex factors, in place. The rounding error of a sum of N random terms taken in order,
    relative to the sum, is about u sqrt(N / 6) rms; four passes and the O(1) roundings of the chirps stay below
    8 u sqrt(N) + 20 u."""
    p, z, lam = 20e-6, 0.4, WI.LAMBDA_HENE
    wx, wy = WI.random_complex((n, n), 31 + n), WI.random_complex((n, n), 32 + n)
    bx, by = O.propagate_separable(wx, wy, n, p, lam, z, n_fft=nz)
    w = torch.empty((n,) * 4, dtype=dtype, device="cuda")
    tx, ty = torch.from_numpy(wx).cuda(), torch.from_numpy(wy).cuda()
    for i in range(n):
        w[i] = tx[i][None, :, None] * ty[:, None, :]
    work = torch.empty_like(w)
    gpu_lib.propagate_padded(w, p, lam, z, nz, out=w, work=work)
    tol = 1e-12 if dtype == torch.complex128 else 8 * U32 * n ** 0.5 + 20 * U32
    assert separable_rel(w, bx, by) < tol
    del w, work
    torch.cuda.empty_cache()


def test_mirror_out_of_place(gpu_lib):
    """Out of place equals in place bit for bit and leaves the input as it was (N = 90: one group of planes)."""
    n = 90
    w = torch.from_numpy(WI.random_complex((n, n, 4, 1), 7).astype(np.complex64)).cuda().expand(n, n, 4, n)
    w = w.repeat(1, 1, 23, 1)[:, :, :n].contiguous()
    keep = w.clone()
    out, _ = gpu_lib.propagate_padded(w, 20e-6, WI.LAMBDA_HENE, 0.4, 90)
    torch.cuda.synchronize()
    assert torch.equal(w, keep)
    gpu_lib.propagate_padded(w, 20e-6, WI.LAMBDA_HENE, 0.4, 90, out=w)
    torch.cuda.synchronize()
    assert torch.equal(out, w)
