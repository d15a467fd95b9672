"""FP64 recursion vectors of the row pipeline carry no larger rounding errors
than those of the one-step kernels: a_{n-2} comes off last, after Ht a_{n-1}
has been summed up."""
from fractions import Fraction

import numpy as np
import pytest

import workloads as W
from tests.gpu_common import gpu_moments, maxdiff

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
