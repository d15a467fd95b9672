"""The pipelined recursion (real operators with uniform hopping, moment
doubling): row widths at the edges of every lane width and of the two column
halves, pass lengths around a whole pass, passes that wrap a periodic
direction, row segments of few vectors; against the direct algorithm (other
kernels, one moment per step), FP64 to 1e-12 and FP32 to 2e-5 as elsewhere."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import gpu_moments, maxdiff

pytestmark = pytest.mark.gpu

WIDTHS = [1, 5, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 383, 384, 385, 511, 512]


def _check(w, N, tile, precision, tol):
    op, ee, he = gpu_moments(w, N=N, tile=tile, precision=precision, algorithm=2)
    op.close()
    op, d_ee, d_he = gpu_moments(w, N=N, tile=tile, algorithm=1)
    op.close()
    assert maxdiff(ee, d_ee) <= tol and maxdiff(he, d_he) <= tol
    assert np.all(he[:, 0::2] == 0)


@pytest.mark.parametrize("precision,tol", [(0, 1e-12), (1, 2e-5)])
@pytest.mark.parametrize("bcx", [0, 1])
@pytest.mark.parametrize("Lx", WIDTHS)
def test_widths(Lx, bcx, precision, tol):
    if bcx and Lx < 3:
        pytest.skip("a periodic direction has at least three sites")
    w = W.small_random(Lx, 31, N=90, seed=Lx + bcx, bc_x=bcx, bc_y=Lx % 2, n_sites=min(260, 31 * Lx))
    _check(w, 90, 260, precision, tol)


@pytest.mark.parametrize("Lx,L", [(64, 20), (192, 24), (384, 12)])
@pytest.mark.parametrize("off", [-2, -1, 0, 1, 2, 3])
def test_pass_lengths(Lx, L, off):
    # passes take the steps 2 .. N/2: one and two whole passes and their neighbours
    for passes in (1, 2):
        N = 2 * (passes * L + 1) + off
        _check(W.small_random(Lx, 40, N=N, seed=N, n_sites=257), N, 257, 0, 1e-12)


@pytest.mark.parametrize("Lx,Ly,bcx,bcy,n", [
    (64, 200, 0, 0, 3), (64, 200, 0, 1, 3), (100, 150, 1, 1, 20), (256, 130, 0, 0, 1), (300, 90, 0, 1, 9),
    (16, 3, 1, 1, 48), (64, 61, 0, 1, 300), (128, 43, 1, 1, 300),
])
def test_segments_and_wrapping(Lx, Ly, bcx, bcy, n):
    w = W.small_random(Lx, Ly, N=161, seed=Lx + Ly, bc_x=bcx, bc_y=bcy, n_sites=n)
    _check(w, 161, n, 0, 1e-12)
    _check(w, 161, n, 1, 2e-5)


def test_ragged_tiles_and_invalid_sites():
    w = W.small_random(70, 33, N=64, seed=5, n_sites=300)
    sites = w.start_sites.copy()
    sites[[0, 17, 299]] = [-1, 70 * 33, 1 << 30]
    op, ee, he = gpu_moments(w, sites=sites, N=64, tile=128, algorithm=2)
    op.close()
    bad = np.isnan(ee).all(axis=1) & np.isnan(he).all(axis=1)
    assert list(np.flatnonzero(bad)) == [0, 17, 299]
    op, d_ee, d_he = gpu_moments(w, sites=sites, N=64, tile=300, algorithm=1)
    op.close()
    ok = ~bad
    assert maxdiff(ee[ok], d_ee[ok]) <= 1e-12 and maxdiff(he[ok], d_he[ok]) <= 1e-12
