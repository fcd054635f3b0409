"""Rounding of the complex128 sums of the batch and of the fit against long double."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P, LAM = 20e-6, 600e-9
L, CL = np.longdouble, np.clongdouble
PI = L("3.14159265358979323846264338327950288")


def cis(turns):
    """e^{2 pi i turns} in long double."""
    a = 2 * PI * (turns - np.rint(turns))
    return np.cos(a) + 1j * np.sin(a)


def beam_axis(n, width, coherence, curve):
    """One axis of a partially coherent beam with a curved wavefront, rounded to 20 bits: products of two are exact."""
    x, h = np.arange(n) - n / 2, n / 2
    f = np.exp(-(x[:, None] ** 2 + x[None, :] ** 2) / (4 * (width * h) ** 2)
               - (x[:, None] - x[None, :]) ** 2 / (2 * (coherence * h) ** 2)).astype(complex)
    f *= np.exp(1j * np.pi * curve * (x[None, :] ** 2 - x[:, None] ** 2))
    return (np.round(f.real * 2.0 ** 20) + 1j * np.round(f.imag * 2.0 ** 20)) / 2.0 ** 20


# The register-tiled 3M sums (twelve chunks of b at N = 128) are 2.33e-16 to 2.43e-16 off on these inputs: a tenth above that.
# A plain chain of N additions, near d = 0 all of one sign, is 3.7e-16 to 4.2e-16 off at N = 128.
FORMER = 2.43e-16


@pytest.mark.parametrize("n,k,probe", [(64, 5, (33, 30)), (64, 40, (34, 31)), (128, 5, (65, 62)), (128, 23, (3, 123)),
                                       (128, 40, (66, 63))])
def test_batch_s_of_a_beam(gpu_lib, n, k, probe):
    """S in the 2-norm, root mean square over pairs of the group."""
    fx, fy = beam_axis(n, 0.3, 0.1, 0.2 / n), beam_axis(n, 0.25, 0.13, -0.3 / n)
    tx, ty = torch.from_numpy(fx).cuda(), torch.from_numpy(fy).cuda()
    w = torch.empty((n,) * 4, dtype=torch.complex128, device="cuda")
    for i in range(n):
        w[i] = tx[i][None, :, None] * ty[:, None, :]
    i = np.arange(k)
    lam, z = LAM * (0.8 + 0.4 * ((7 * i) % 11) / 11), 0.1 + 0.8 * ((5 * i) % 13) / 13
    s, _ = gpu_lib.propagate_batch(w, P, lam, z, np.ones(k), ip=probe[0], jp=probe[1], floor_rel=0.0)
    s = s.cpu().numpy().astype(L)
    d = (np.arange(n) - n // 2).astype(L)
    sq = []
    for q in range(0, k, max(1, k // 6)):
        lz = lam[q] * z[q]
        h = cis(-(d[:, None] * d[None, :]) / n) * cis(d * d * L(P * P / lz) / 2)[None, :]
        bx, by = h.conj() @ fx.astype(CL) @ h.T, h.conj() @ fy.astype(CL) @ h.T
        ref = L(1.0 / (lz * lz) * P * P * P * P) * np.outer(np.diag(bx).real, np.diag(by).real)
        sq.append(float(((s[q] - ref) ** 2).sum() / (ref ** 2).sum()))
    assert np.sqrt(np.mean(sq)) < 1.1 * FORMER


def fit_reference(b, inv, scale, moment=0):
    """scale sum_d e^{2 pi i <m - c, d> / N} D[d] from the differences of b, in long double: S_B. moment = 2: with |d|^2 D[d]."""
    n = b.shape[0]
    dd = np.zeros((n, n), CL)
    for di in range(n):
        for dj in range(-n + 1, n):
            if di == 0 and dj < 0:
                continue
            j0, j1 = max(0, dj), min(n, n + dj)
            c = (b[di:, j0:j1].conj() * b[:n - di, j0 - dj:j1 - dj]).sum() * np.exp(-L(di * di + dj * dj) * L(inv))
            if moment:
                c *= di * di + dj * dj
            dd[di % n, dj % n] += c
            if di or dj:
                dd[-di % n, -dj % n] += c.conj()
    k = np.arange(n)
    f = cis(((k[:, None] - n // 2) * k[None, :]).astype(L) / n)
    return L(scale) * (f @ dd @ f.T).real


# The passes over the propagated array are 1.47e-16 to 1.55e-16 off on these inputs: a tenth above that. Plain chains in the two
# transforms of the difference sums are 3.0e-16 to 3.9e-16 off.
FORMER_FIT = 1.55e-16


@pytest.mark.parametrize("farfield", [False, True])
@pytest.mark.parametrize("n,seeds", [(32, 8), (64, 4)])
def test_fit_s(gpu_lib, n, seeds, farfield):
    """S_B of the custom-map source in the 2-norm, root mean square over seeds; sqrt(I) is exact."""
    sq = []
    for seed in range(seeds):
        r = np.random.default_rng(100 * n + seed)
        sg, z, lam = r.uniform(0.06, 0.15) * P * n / 2, r.uniform(0.4, 0.6), LAM * r.uniform(0.9, 1.1)
        x = np.arange(n) - n / 2
        im = (0.02 + np.exp(-(x[:, None] ** 2 + x[None, :] ** 2) / (2 * (0.4 * n / 2) ** 2))) * np.exp(
            0.3 * r.standard_normal((n, n)))
        a = np.round(np.sqrt(im) * 2 ** 11) / 2 ** 11
        s, _ = gpu_lib.fit_forward(torch.from_numpy((a * a).astype(np.float32)).cuda(), P, sg, lam, z, farfield)
        d = np.arange(n) - n // 2
        t = cis((d * d).astype(L) * L(0.0 if farfield else P * P / (lam * z)) / 2)
        ref = fit_reference(a.astype(L) * t[:, None] * t[None, :], P * P / (2.0 * sg * sg),
                            1.0 / ((lam * z) * (lam * z)) * P * P * P * P)
        sq.append(float(((s.cpu().numpy().astype(L) - ref) ** 2).sum() / (ref ** 2).sum()))
    assert np.sqrt(np.mean(sq)) < 1.1 * FORMER_FIT


@pytest.mark.parametrize("farfield", [False, True])
@pytest.mark.parametrize("n", [16, 32])
def test_fit_dsigma(gpu_lib, n, farfield):
    """dL/dsg = f sum_m g[m] T[m], T the transform of |d|^2 D[d], with random g. The library takes it as f sum_d Re G conj(D2):
    G carries 2 u of its root mean square from two transforms, D2 4 u from table, product, weight and sums, the final sum u, against
    the sum of the sizes |G D2|: 8 u of it."""
    r = np.random.default_rng(n)
    sg, z, lam = 0.1 * P * n / 2, 0.5, LAM
    x = np.arange(n) - n / 2
    a = np.round((0.2 + np.exp(-(x[:, None] ** 2 + x[None, :] ** 2) / (n / 2) ** 2)) * np.exp(
        0.2 * r.standard_normal((n, n))) * 2 ** 11) / 2 ** 11
    g = np.round(64 * r.standard_normal((n, n))) / 64
    imap = torch.from_numpy((a * a).astype(np.float32)).cuda()
    gs = torch.from_numpy(g).cuda()
    s, corr = gpu_lib.fit_forward(imap, P, sg, lam, z, farfield)
    _, ds = gpu_lib.fit_backward(gs, imap, corr, P, sg, lam, z, farfield)
    d = np.arange(n) - n // 2
    t = cis((d * d).astype(L) * L(0.0 if farfield else P * P / (lam * z)) / 2)
    scale = 1.0 / ((lam * z) * (lam * z)) * P * P * P * P
    tm = fit_reference(a.astype(L) * t[:, None] * t[None, :], P * P / (2.0 * sg * sg), scale, 2)
    f = L(P * P / (sg * sg * sg))
    k = np.arange(n)
    w = cis(((k[:, None] - n // 2) * k[None, :]).astype(L) / n)
    sizes = np.abs(w.conj().T @ g.astype(CL) @ w.conj()) * np.abs(w.conj().T @ tm.astype(CL) @ w.conj()) / (n * n)
    ref = f * (g.astype(L) * tm).sum()
    assert abs(float(L(float(ds)) - ref)) < 8 * 2.0 ** -53 * float(f * sizes.sum())
