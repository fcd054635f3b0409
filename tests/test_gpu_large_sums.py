"""N = 256, and probes whose S is certainly positive: the contractions of the batch, the common-grid sum and the fit against
references that need no N^4 array of the oracle."""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

import oracle as O
import wolf_inputs as WI
from tests.test_gpu_mirror_sums import pairs_of

pytestmark = pytest.mark.gpu

P, LAM = 20e-6, 600e-9
U = {torch.complex64: 2.0 ** -24, torch.complex128: 2.0 ** -53}


# ---------------------------------------------------------------------------------------------------------
# Sources without mirror symmetry and with S > 0 everywhere, so that mu is compared at every point.
# ---------------------------------------------------------------------------------------------------------
def positive_source(n, dtype):
    """Random complex entries (no symmetry) on a diagonal of 4: S is 4 N^2 and a random part of about 0.7 N^2."""
    g = torch.Generator(device="cuda").manual_seed(n)
    w = torch.view_as_complex(torch.randn((n * n, n * n, 2), generator=g, device="cuda", dtype=torch.float32))
    d = torch.arange(n * n, device="cuda")
    w *= 0.5
    w[d, d] += 4
    return w.reshape(n, n, n, n).to(dtype)


def mu_reference(w, lam, z, probe):
    """S and mu(P, .) of one pair from the complex128 operator."""
    n = w.shape[0]
    wb, _ = WOLF.propagate_fresnel(w.to(torch.complex128), P, lam, z)
    s = WOLF.spectral_density(wb)
    return s, wb[probe[0], probe[1]] / torch.sqrt(s[probe[0], probe[1]] * s)


WOLF = None


@pytest.fixture(autouse=True)
def _library(gpu_lib):
    global WOLF
    WOLF = gpu_lib


# Pair tiles of 16, 32 and 64 with ragged counts; probes at the corner, the edges and the middle.
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n,k,probe", [(32, 2, (0, 0)), (32, 33, (16, 31)), (64, 16, (31, 1)), (64, 17, (0, 32)),
                                       (64, 65, (63, 63)), (128, 3, (64, 0)), (128, 20, (0, 127)), (128, 40, (127, 5))])
def test_batch_mu_at_every_point(gpu_lib, n, k, probe, dtype):
    """W(P, m) is a sum of N^4 products of random terms: its rounding against the sum is that of a product tree, 100 u at most
    (S: the same). |W| is about 0.12 S here, so mu carries W's 100 u and half of S's and S(P)'s, 200 u together; in FP64 the
    phases' own error, 10^-12, is the larger."""
    w = positive_source(n, dtype)
    lam, z, wt = pairs_of(k)
    s, mu = gpu_lib.propagate_batch(w, P, lam, z, wt, ip=probe[0], jp=probe[1], floor_rel=1e-2)
    for q in sorted({0, k // 2, k - 1}):
        sref, mref = mu_reference(w, lam[q], z[q], probe)
        assert float(sref.min()) > 0.05 * float(sref.max())
        assert float((s[q].double() - wt[q] * sref).norm() / (wt[q] * sref).norm()) < max(100 * U[dtype], 1e-12)
        assert bool((mu[q] != 0).all())
        assert float((mu[q] - mref).norm() / mref.norm()) < max(200 * U[dtype], 1e-12)


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("n,k,probe", [(2, 1, (1, 0)), (8, 3, (7, 4)), (16, 5, (0, 15)), (32, 3, (31, 16)), (64, 1, (5, 63)),
                                       (64, 20, (32, 0)), (128, 5, (127, 64))])
def test_poly_mu_at_every_point(gpu_lib, n, k, probe, dtype):
    """Pairs of one product lambda z share their FFT grid: S and W(P, .) are the weighted sums of the operator's. Bounds as above."""
    w = positive_source(n, dtype)
    lam = LAM * (1 + 0.02 * np.arange(k))
    z, wt = LAM * 0.3 / lam, 1.0 + 0.5 * (np.arange(k) % 3)
    s, mu = gpu_lib.propagate_polychromatic(w, P, lam, z, wt, LAM * 0.3 / (n * P), ip=probe[0], jp=probe[1], floor_rel=1e-2)
    total = 0
    for i in range(k):
        total = total + wt[i] * gpu_lib.propagate_fresnel(w.to(torch.complex128), P, lam[i], z[i])[0]
    sref = gpu_lib.spectral_density(total)
    assert float(sref.min()) > 0.05 * float(sref.max())
    mref = total[probe] / torch.sqrt(sref[probe] * sref)
    assert float((s.double() - sref).norm() / sref.norm()) < max(100 * U[dtype], 1e-12)
    assert bool((mu != 0).all())
    assert float((mu - mref).norm() / mref.norm()) < max(200 * U[dtype], 1e-12)


# ---------------------------------------------------------------------------------------------------------
# Separable sources W = wx(i1, i2) wy(j1, j2): W_B = bx by, b = conj(h) w h^T per axis in numpy.
# ---------------------------------------------------------------------------------------------------------
def psd_axis(n, seed):
    """Hermitian, positive and without mirror symmetry: A A^H of rank 3 with random A, and a diagonal."""
    a = WI.random_complex((n, 3), seed)
    return a @ a.conj().T / 3 + np.eye(n)


def stored(wx, wy, dtype):
    n = wx.shape[0]
    tx, ty = torch.from_numpy(wx).cuda().to(dtype), torch.from_numpy(wy).cuda().to(dtype)
    w = torch.empty((n,) * 4, dtype=dtype, device="cuda")
    for i in range(n):
        w[i] = tx[i][None, :, None] * ty[:, None, :]
    return w


def axis_kernel(n, lz, out_pitch, farfield=False):
    i = np.arange(n) - n / 2
    x, xi = out_pitch * i[:, None], P * i[None, :]
    c = (x * x - 2 * x * xi) / lz if farfield else (x - xi) ** 2 / lz
    return np.exp(1j * np.pi * np.remainder(c, 2.0))


def observed(wx, wy, lz, out_pitch, probe, farfield=False):
    """(S, W(P, .)) without the weight, the scale 1 / (lambda z)^2 P^4 included (secondary source)."""
    h = axis_kernel(wx.shape[0], lz, out_pitch, farfield)
    bx, by = h.conj() @ wx @ h.T, h.conj() @ wy @ h.T
    c = P ** 4 / lz ** 2
    return c * np.outer(np.diag(bx).real, np.diag(by).real), c * np.outer(bx[probe[0]], by[probe[1]])


def check(s, mu, sref, wref, probe, dtype):
    """S and mu where S is above 5 % of its maximum: 200 u of the FP32 sums as above; FP64 phases of up to 10^2 turns, 10^-11."""
    tol = max(200 * U[dtype], 1e-11)
    assert np.linalg.norm(s - sref) / np.linalg.norm(sref) < tol
    inside = sref > 0.05 * sref.max()
    assert inside[probe] and inside.mean() > 0.02
    mref = wref / np.sqrt(np.where(inside, sref, 1.0) * sref[probe])
    assert np.all(mu[inside] != 0)
    assert np.linalg.norm((mu - mref)[inside]) / np.linalg.norm(mref[inside]) < tol


@pytest.mark.parametrize("n,k,dtype", [(64, 5, torch.complex64), (64, 20, torch.complex128), (128, 17, torch.complex64),
                                       (128, 40, torch.complex128), (256, 3, torch.complex64), (256, 1, torch.complex64)])
def test_poly_off_the_fft_grid(gpu_lib, n, k, dtype):
    """A common grid whose pitch is no FFT pitch of any pair, several products lambda z."""
    wx, wy = psd_axis(n, 11 + n), psd_axis(n, 12 + n)
    w = stored(wx, wy, dtype)
    lam, z, wt = pairs_of(k)
    op = 0.77 * LAM * 0.25 / (n * P)
    sref, best = 0.0, None
    probe = (n // 2 + 3, n // 2 - 2)
    parts = [observed(wx, wy, lam[q] * z[q], op, probe) for q in range(k)]
    sref = sum(wt[q] * parts[q][0] for q in range(k))
    probe = np.unravel_index(np.argmax(sref), sref.shape)  # a point of high S
    wref = sum(wt[q] * observed(wx, wy, lam[q] * z[q], op, probe)[1] for q in range(k))
    s, mu = gpu_lib.propagate_polychromatic(w, P, lam, z, wt, op, ip=int(probe[0]), jp=int(probe[1]), floor_rel=1e-2)
    check(s.double().cpu().numpy(), mu.to(torch.complex128).cpu().numpy(), sref, wref, probe, dtype)


@pytest.mark.parametrize("k,dtype", [(17, torch.complex64), (40, torch.complex64), (2, torch.complex128), (20, torch.complex128),
                                     (40, torch.complex128)])
def test_batch_at_256(gpu_lib, k, dtype):
    n = 256
    wx, wy = psd_axis(n, 21), psd_axis(n, 22)
    w = stored(wx, wy, dtype)
    lam, z, wt = pairs_of(k)
    probe = (n // 2 + 1, n // 2 - 2)
    first = observed(wx, wy, lam[0] * z[0], lam[0] * z[0] / (n * P), probe)[0]
    probe = tuple(int(v) for v in np.unravel_index(np.argmax(first), first.shape))
    s, mu = gpu_lib.propagate_batch(w, P, lam, z, wt, ip=probe[0], jp=probe[1], floor_rel=1e-3)
    for q in sorted({0, k // 2, k - 1}):
        lz = lam[q] * z[q]
        sref, wref = observed(wx, wy, lz, lz / (n * P), probe)
        got = s[q].double().cpu().numpy() / wt[q]
        if sref[probe] > 0.05 * sref.max():
            check(got, mu[q].to(torch.complex128).cpu().numpy(), sref, wref, probe, dtype)
        else:
            assert q > 0
            assert np.linalg.norm(got - sref) / np.linalg.norm(sref) < max(200 * U[dtype], 1e-11)
    del w
    torch.cuda.empty_cache()


@pytest.mark.parametrize("farfield", [False, True])
def test_fit_forward_at_256(gpu_lib, farfield):
    """A separable map: S_B = sx sy with s = diag(conj(h) (a a^T mu_g) h^T) per axis. FP64 sums of N^4 terms: 10^-11."""
    n, lam, z, sg = 256, 633e-9, 0.5, 3e-4
    r = np.random.default_rng(5)
    ax, ay = (np.round(2.0 ** 5 * (0.5 + r.random(n))) / 2.0 ** 5 for _ in range(2))  # 6 bits: float32 holds a^2 a^2
    imap = torch.from_numpy(np.outer(ax * ax, ay * ay).astype(np.float32)).cuda()
    assert (imap.double().cpu().numpy() == np.outer(ax * ax, ay * ay)).all()
    x = P * (np.arange(n) - n / 2)
    g = np.exp(-(x[:, None] - x[None, :]) ** 2 / (2 * sg * sg))
    h = axis_kernel(n, lam * z, lam * z / (n * P), farfield)
    sx, sy = (np.einsum("ma,ab,mb->m", h.conj(), a[:, None] * g * a[None, :], h, optimize=True).real for a in (ax, ay))
    sref = P ** 4 / (lam * z) ** 2 * np.outer(sx, sy)
    s, _ = gpu_lib.fit_forward(imap, P, sg, lam, z, farfield)
    assert np.linalg.norm(s.cpu().numpy() - sref) / np.linalg.norm(sref) < 1e-11


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
def test_formed_diagonal_at_256(gpu_lib, dtype):
    """The operator on diag(gx gy) is separable: A = a_x a_y with a = h^T diag(g) conj(h) per axis; passes of
    4 (2 log2 N + 3) roundings, 200 u of the largest value; FP64 phases of up to 10^2 turns, 10^-11."""
    n, lam, z = 256, 633e-9, 0.5
    r = np.random.default_rng(6)
    gx, gy = r.standard_normal(n), r.standard_normal(n)
    real = torch.float32 if dtype == torch.complex64 else torch.float64
    g = torch.from_numpy(np.outer(gx, gy)).to(real).cuda()
    h = axis_kernel(n, lam * z, lam * z / (n * P))
    a = [h.T @ (v[:, None] * h.conj()) for v in (gx, gy)]
    out = gpu_lib.propagate_adjoint_diag(g, P, lam, z, dtype=dtype)
    c = P ** 4 / (lam * z) ** 2
    tx, ty = torch.from_numpy(c * a[0]).cuda(), torch.from_numpy(a[1]).cuda()
    worst = 0.0
    for i in range(n):
        ref = tx[i][None, :, None] * ty[:, None, :]
        worst = max(worst, float((out[i].to(torch.complex128) - ref).abs().max()))
    assert worst <= max(200 * U[dtype], 1e-11) * float(tx.abs().max() * ty.abs().max())
    del out
    torch.cuda.empty_cache()
