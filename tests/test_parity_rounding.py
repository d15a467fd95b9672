"""FP64 recursion vectors of the row pipelines carry no larger rounding errors
than those of the one-step kernels: a_{n-2} comes off last, after Ht a_{n-1}
has been summed up."""
from fractions import Fraction

import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_common import DEV, gpu_moments, maxdiff

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -53


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _emulated_row(w, a, N):
    """Doubling moments of site 1 of a three-site open row: vectors rounded as
    the one-step kernels round them, sums exact."""
    de = [float(v) for v in (w.eps - w.mu_c) / a]
    dr = [float(v) for v in np.asarray(w.delta) / a]
    th = w.t / a
    ce, ch, pe, ph = [-th, de[1], -th], [0.0, dr[1], 0.0], [0.0, 1.0, 0.0], [0.0] * 3
    ee, he = np.zeros(N), np.zeros(N)
    ee[0], ee[1], he[1] = 1.0, de[1], dr[1]
    ee[2] = 2.0 * float(sum(Fraction(v) ** 2 for v in ce + ch)) - 1.0
    for m in range(2, N // 2 + 1):
        ne, nh = [], []
        for x in range(3):
            se = (ce[x - 1] if x > 0 else 0.0) + (ce[x + 1] if x < 2 else 0.0)
            sh = (ch[x - 1] if x > 0 else 0.0) + (ch[x + 1] if x < 2 else 0.0)
            ne.append(_fma(2.0, _fma(de[x], ce[x], _fma(dr[x], ch[x], -(th * se))), -pe[x]))
            nh.append(_fma(2.0, _fma(-de[x], ch[x], _fma(dr[x], ce[x], th * sh)), -ph[x]))
        s0 = sum(Fraction(v) ** 2 for v in ne + nh)
        s1 = sum(Fraction(u) * Fraction(v) for u, v in zip(ne + nh, ce + ch))
        s2 = sum(Fraction(ne[i]) * Fraction(ch[i]) - Fraction(nh[i]) * Fraction(ce[i]) for i in range(3))
        if 2 * m < N:
            ee[2 * m] = float(2 * s0 - 1)
        if 2 * m - 1 < N:
            ee[2 * m - 1] = float(2 * s1 - Fraction(ee[1]))
            he[2 * m - 1] = float((-2 if m & 1 else 2) * s2 - Fraction(he[1]))
        pe, ph, ce, ch = ce, ch, ne, nh
    return ee, he


@pytest.mark.parametrize("seed", [1, 2])
def test_real_pipeline_rounds_as_the_one_step_kernels(seed):
    """Errors of the vectors grow over 4000 steps (to 1.4e-14 in the moments
    where the sums begin with a_{n-2}); those of the sums do not.  A sum of
    three lanes takes at most four roundings of terms adding up to 1 at most,
    a moment is twice a sum and one difference, on either side: 12 roundings."""
    N = 8000
    w = W.small_random(3, 1, N, seed=seed)
    op, ee, he = gpu_moments(w, sites=[1], N=N, tile=1, algorithm=2, fixed=(7.0, 0.0))
    op.close()
    r_ee, r_he = _emulated_row(w, 7.0, N)
    assert maxdiff(ee[0], r_ee) <= 12 * ULP and maxdiff(he[0], r_he) <= 12 * ULP


def _run_nb(w, op):
    import paper_1007_1609_amd as P
    sites = torch.as_tensor(w.start_sites, device=DEV)
    return [t.cpu().numpy() for t in P.chebyshev_moments_nb(op, sites, w.N, len(sites))[:2]]


@pytest.mark.parametrize("cplx", [False, True])
def test_general_pipeline_rounds_uniform_operators_as_the_one_step_kernels(cplx):
    import paper_1007_1609_amd as P
    w = W.small_random(41, 20, 256, seed=8, complex_=cplx, n_sites=40)
    op = P.Operator.from_workload(w, DEV)
    ee, he = _run_nb(w, op)
    op.close()
    op, d_ee, d_he = gpu_moments(w, tile=40, algorithm=1)
    op.close()
    assert np.array_equal(ee, d_ee) and np.array_equal(he, d_he)


def _local_moments_80bit(w, a):
    """mu_ee, mu_he of the start sites from recursion vectors in 80 bits."""
    L, C = np.longdouble, np.clongdouble
    sh, n, k = (w.Ly, w.Lx), len(w.start_sites), np.arange(len(w.start_sites))
    de = ((w.eps - w.mu_c) / a).reshape(sh).astype(L)

    def scaled(z):
        z = np.asarray(z, dtype=np.complex128)
        return (z.real / a + 1j * (z.imag / a)).astype(C)

    dl, b = scaled(w.delta).reshape(sh), scaled(w.delta_bond).reshape((2,) + sh)
    th = np.zeros((2,) + sh) if w.peierls is None else np.asarray(w.peierls).reshape((2,) + sh)
    t = (w.t * np.cos(th) / a + 1j * (w.t * np.sin(th) / a)).astype(C)
    for z in (t, b):
        z[0, :, -1] = 0.0
        z[1, -1, :] = 0.0

    def apply(v):
        e, h = v[..., 0], v[..., 1]
        oe, oh = de * e + dl * h, np.conj(dl) * e - de * h
        for ax, d in ((0, 2), (1, 1)):
            ef, hf, eb, hb = np.roll(e, -1, d), np.roll(h, -1, d), np.roll(e, 1, d), np.roll(h, 1, d)
            tb, bb = np.roll(np.conj(t[ax]), 1, d - 1), np.roll(b[ax], 1, d - 1)
            oe = oe - t[ax] * ef + b[ax] * hf - tb * eb + bb * hb
            oh = oh + np.conj(b[ax]) * ef + np.conj(t[ax]) * hf + np.conj(bb) * eb + np.conj(tb) * hb
        return np.stack([oe, oh], -1)

    y, x = w.start_sites // w.Lx, w.start_sites % w.Lx
    p = np.zeros((n,) + sh + (2,), C)
    p[k, y, x, 0] = 1.0
    q = apply(p)
    mu = np.zeros((n, w.N, 2), C)
    mu[:, 0], mu[:, 1] = p[k, y, x], q[k, y, x]
    for m in range(2, w.N):
        p, q = q, 2 * apply(q) - p
        mu[:, m] = q[k, y, x]
    return mu[..., 0].real, mu[..., 1]


@pytest.mark.parametrize("cplx,flux", [(False, 0.0), (True, 1.0 / 16.0)])
def test_general_pipeline_rounds_per_bond_operators_no_worse(cplx, flux):
    """rms error of the local moments against 80-bit vectors, relative to the
    one-step kernels': sums begun with a_{n-2} double it, so the line lies at
    the square root of two."""
    import paper_1007_1609_amd as P
    w = W.small_random(33, 24, 300, seed=6, complex_=cplx, bond=True, flux=flux, n_sites=24)
    op = P.Operator.from_workload(w, DEV, fixed=(8.0, 0.0))
    ee, he = _run_nb(w, op)
    op.close()
    op, d_ee, d_he = gpu_moments(w, tile=24, algorithm=1, fixed=(8.0, 0.0))
    op.close()
    r_ee, r_he = _local_moments_80bit(w, 8.0)

    def rms(e, h):
        return float(np.sqrt(np.mean((e - r_ee) ** 2) + np.mean(np.abs(h - r_he) ** 2)))

    print("rms error: pipeline %.2e, one-step kernels %.2e" % (rms(ee, he), rms(d_ee, d_he)))
    assert rms(ee, he) <= np.sqrt(2.0) * rms(d_ee, d_he)
